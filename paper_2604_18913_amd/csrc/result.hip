// Result side of logoskg_khop: per-query reached counts, the query-major
// (entity, hop, predecessor edge) lists, and the per-query traversed-edge
// counts.
//
// The level planes are entity-major bit matrices; the lists are their
// transpose.  Entities are cut into tiles of 64 (one wavefront of lanes), super
// tiles of 16 tiles and mega tiles of 64 super tiles.  A wavefront owns one
// word (64 queries) of a tile: lane v holds that word of entity 64*tile+v, and
// for each query a ballot gives the mask of tile entities the query reached -
// its popcount is the tile's count, the population below a lane is the
// entity's rank inside the tile's run of the query's list.
//
//   count : per (query, tile) counts -> nested exclusive prefixes -> offsets
//           (of the visited plane, or of one level plane for the per-level lists)
//   lists : one block per super tile compacts the (entity, hop) entries of each
//           query in LDS and writes them as whole 64-lane stores; entity lists
//           of 16-word planes a wavefront per word of a tile, lane = entity
//   pred  : the predecessor edge (smallest edge id whose subject sits one hop
//           closer and whose relation the query allows - the first active
//           triple of Eq. 5-7 in edge-id order) is found by walking the object
//           row of the entity with a mask of still unresolved queries, so every
//           (query, entity) pair is written once.  Object rows of up to 32
//           entries belong to the tile kernels that walk them in ascending
//           edge id and write the entity and hop lists as well (k_fetch_narrow
//           on planes of one and four words, the pair k_pred_walk / k_pred_emit
//           on 16-word planes with k <= 6; k_pred, beside k_lists, for deeper
//           searches there); rows of 33 .. hub_min-1 entries belong to
//           k_pred_wave and longer ones to k_pred_row, whose lanes claim in
//           parallel and keep the minimum, or, where a line has one or four
//           words or the fetched queries sit in one, two or four aligned words
//           of it, to k_narrow_wave and k_narrow_row with a lane per entry.  A
//           level with a small frontier is taken from the subject side for the
//           longer rows of 16-word planes (k_pred_push).
#include <algorithm>
#include <climits>
#include <cstdlib>

#include "common.h"

namespace lkg {

// Tiles.  A tile is 64 entities.  Without a list (tile_ent == NULL) tile i holds the ids
// 64 i .. 64 i + 63; with the list of a result's active entities (those with a bit in any level,
// ascending, built by k_active_*) tile i holds entries 64 i .. 64 i + 63 of the list, so that the
// tiles carry no entity that no query reached (-1 pads the last tile).
__device__ __forceinline__ long long tile_entity(const int32_t *__restrict__ tile_ent, long long tile, int i,
                                                 int32_t E) {
    if (tile_ent) return tile_ent[tile * 64 + i];
    const long long e = tile * 64 + i;
    return e < E ? e : -1;
}

template <int W>
__device__ __forceinline__ unsigned long long stage_word(unsigned long long (*stage)[W + 1],
                                                         const unsigned long long *__restrict__ plane,
                                                         const int32_t *__restrict__ tile_ent, long long tile,
                                                         int32_t E, int wave) {
    // Lane v takes word `wave` of the tile's entity v.  Lines of one and four words are read that way (a
    // wavefront's lanes cover neighbouring 8- or 32-byte lines), without LDS and without a barrier (a caller
    // whose wavefronts share something needs one of its own), so a caller's loads over several tiles are in
    // flight together; through LDS with two barriers each, they were a chain of 64 dependent rounds in a block
    // of the list kernel (31 us for the lists of one query on 407,000 entities, 27 us without).  A 16-word line is 128 bytes: loaded with W
    // consecutive lanes per line and handed over through LDS.
    if constexpr (W <= 4) {
        const long long e = tile_entity(tile_ent, tile, lane(), E);
        return e >= 0 ? plane[(size_t)e * W + wave] : 0ull;
    }
    const int t = threadIdx.x;
    const long long e = tile_entity(tile_ent, tile, t / W, E);
    __syncthreads();
    stage[t / W][t % W] = e >= 0 ? plane[(size_t)e * W + t % W] : 0ull;
    __syncthreads();
    return stage[lane()][wave];
}

// ---------------------------------------------------------------- list of the active entities
// act holds one bitmap per level (one bit per entity with a non-zero line); their union marks the
// entities some query reached.  Chunks of 2,048 entities (64 bitmap words, one wavefront):
// k_active_count counts a chunk, k_active_scan turns the counts into exclusive offsets and the
// total, k_active_fill writes the ids (ascending) and every listed entity's position.
constexpr int kActChunkWords = 64;

__device__ __forceinline__ uint32_t active_word(const uint32_t *__restrict__ act, long long actw, int levels,
                                                long long word) {
    uint32_t u = 0;
    if (word < actw)
        for (int h0 = 0; h0 < levels; h0 += 4)  // four levels requested together (the last one again where there are fewer)
#pragma unroll
            for (int i = 0; i < 4; ++i) u |= act[(size_t)min(h0 + i, levels - 1) * actw + word];
    return u;
}

__global__ void __launch_bounds__(256)
k_active_count(const uint32_t *__restrict__ act, long long actw, int levels, long long nchunks, uint32_t *chunk_cnt) {
    const long long chunk = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (chunk >= nchunks) return;
    const uint32_t u = active_word(act, actw, levels, chunk * kActChunkWords + lane());
    const long long c = wave_sum((long long)__popc(u));
    if (lane() == 0) chunk_cnt[chunk] = (uint32_t)c;
}

// one block: exclusive prefix over the chunk counts (in place), total to *n_active, and -1 in the
// 64 list entries behind the last id
__global__ void __launch_bounds__(1024)
k_active_scan(long long nchunks, uint32_t *chunk_cnt, unsigned long long *n_active, int32_t *tile_ent) {
    __shared__ unsigned long long part[2][1024];
    const int t = threadIdx.x;
    const long long per = (nchunks + 1023) / 1024, lo = (long long)t * per, hi = min(nchunks, lo + per);
    unsigned long long sum = 0;
    for (long long i = lo; i < hi; ++i) sum += chunk_cnt[i];
    int cur = 0;
    part[0][t] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        unsigned long long x = part[cur][t];
        if (t >= d) x += part[cur][t - d];
        part[cur ^ 1][t] = x;
        cur ^= 1;
        __syncthreads();
    }
    unsigned long long run = part[cur][t] - sum;
    for (long long i = lo; i < hi; ++i) {
        const uint32_t c = chunk_cnt[i];
        chunk_cnt[i] = (uint32_t)run;
        run += c;
    }
    const unsigned long long total = part[cur][1023];
    if (t == 0) *n_active = total;
    if (t < 64) tile_ent[total + t] = -1;
}

// The ids and positions of a chunk, its first listed entity at place `at`; lane l holds bitmap word first + l.  64 entities at a
// time, lane = entity, so that both stores are contiguous: a lane that walks the bits of its own word stores to 64 places
// of the list at once (20M entities: 320 us, 407,000 in one launch: 16 us).
__device__ __forceinline__ void write_listed(uint32_t u, long long first, long long at, int32_t *tile_ent, int32_t *cpos) {
    int total;
    const int rank = wave_excl_scan(__popc(u), total);
    if (total == 0) return;
#pragma unroll 4
    for (int i = 0; i < kActChunkWords; i += 2) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)u, i), hi = (uint32_t)__builtin_amdgcn_readlane((int)u, i + 1);
        const unsigned long long m = ((unsigned long long)hi << 32) | lo;
        if (m == 0) continue;
        const long long place = at + __builtin_amdgcn_readlane(rank, i) + __popcll(m & ((1ull << lane()) - 1ull));
        const int32_t e = (int32_t)((first + i) * 32) + lane();
        if ((m >> lane()) & 1ull) {
            tile_ent[place] = e;
            cpos[e] = (int32_t)place;
        }
    }
}

// SUM: the chunks' counts are still that, and a block adds up those before its own (instead of a launch of k_active_scan
// between: 4 us and its gap).  What the blocks read together grows with the square of the graph, so it ends at kActSumChunks,
// well before that shows: us of a search of one question by entities, with the scan / without: 1M 1,380 / 1,376, 16M 1,587 /
// 1,586, 33M 1,835 / 1,829, 100M 2,959 / 2,953 (1.2 GB through the L2s).
constexpr long long kActSumChunks = 16384;  // 33M entities: 0.13 GB

template <bool SUM>
__global__ void __launch_bounds__(256)
k_active_fill(const uint32_t *__restrict__ act, long long actw, int levels, long long nchunks,
              const uint32_t *__restrict__ chunk_base, unsigned long long *n_active, int32_t *tile_ent, int32_t *cpos) {
    __shared__ uint32_t part[4];
    const int wave = threadIdx.x >> 6;
    const long long chunk0 = (long long)blockIdx.x * 4, chunk = chunk0 + wave, first = chunk * kActChunkWords;
    const uint32_t mine = active_word(act, actw, levels, first + lane());  // (0 behind the last chunk)
    long long at = 0;
    if constexpr (SUM) {
        uint32_t sum = 0;
        for (long long i = threadIdx.x; i < chunk0; i += 256) sum += chunk_base[i];
        sum = (uint32_t)wave_sum(sum);
        if (lane() == 0) part[wave] = sum;
        __syncthreads();
        at = (long long)part[0] + part[1] + part[2] + part[3];
        for (long long c = chunk0; c < min(chunk, nchunks); ++c) at += chunk_base[c];
        if (blockIdx.x + 1 == gridDim.x && wave == 3) {  // behind this block's last chunk
            const long long end = at + (chunk < nchunks ? chunk_base[chunk] : 0u);
            if (lane() == 0) *n_active = (unsigned long long)end;
            tile_ent[end + lane()] = -1;
        }
    }
    if (chunk >= nchunks) return;
    if constexpr (!SUM) at = chunk_base[chunk];
    write_listed(mine, first, at, tile_ent, cpos);
}

// The three in one launch: a block (a thread per bitmap word) counts what lies before it by itself.  The blocks' common
// reading grows with the square of the graph and with the levels, so only bitmaps of few words go this way.  Searches of one
// question, one launch less three, us, by entities and levels: 16,384 x 4 -4, x 32 -3; 65,536 x 8 -2, x 16 +7; 131,072 x 4
// -1, x 12 +5; 262,144 x 4 0, x 8 +7; 407,000 x 4 +4, x 12 +19; 1M x 2 +14, x 32 +129.
constexpr long long kActiveOneLaunch = 1ll << 19;  // entities times levels
inline bool active_in_one_launch(long long Epad, int levels) { return Epad * levels <= kActiveOneLaunch; }
constexpr int kActiveListThreads = 256;

__global__ void __launch_bounds__(kActiveListThreads)
k_active_list(const uint32_t *__restrict__ act, long long actw, int levels, unsigned long long *n_active, int32_t *tile_ent,
              int32_t *cpos) {
    constexpr int NT = kActiveListThreads;
    __shared__ int before_part[NT / 64], own_part[NT / 64];
    const int t = threadIdx.x, wave = t >> 6;
    const long long first = (long long)blockIdx.x * NT;
    int before = 0;
    constexpr int U = 8;  // bitmap words requested together (one at a time, the reading is a chain)
    for (long long i0 = 2 * t; i0 < first; i0 += 2 * NT * U) {  // (first and actw are even, the bitmaps 8-byte aligned)
        unsigned long long u[U] = {};
        for (int h0 = 0; h0 < levels; h0 += 4)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t *row = act + (size_t)min(h0 + i, levels - 1) * actw;
#pragma unroll
                for (int x = 0; x < U; ++x)  // (in range for every lane, counted only before the block)
                    u[x] |= *reinterpret_cast<const unsigned long long *>(row + min(i0 + 2 * NT * x, first - 2));
            }
#pragma unroll
        for (int x = 0; x < U; ++x) before += i0 + 2 * NT * x < first ? __popcll(u[x]) : 0;
    }
    const uint32_t mine = active_word(act, actw, levels, first + t);
    const int own = (int)wave_sum(__popc(mine));
    before = (int)wave_sum(before);
    if (lane() == 0) {
        before_part[wave] = before;
        own_part[wave] = own;
    }
    __syncthreads();
    long long at = 0, end = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        at += before_part[w] + (w < wave ? own_part[w] : 0);
        end += before_part[w] + own_part[w];
    }
    write_listed(mine, first + 64 * wave, at, tile_ent, cpos);
    if (blockIdx.x + 1 == gridDim.x) {  // nothing lies behind this block
        if (t == 0) *n_active = (unsigned long long)end;
        if (t < 64) tile_ent[end + t] = -1;
    }
}

// blocks are dealt round-robin to the 8 XCDs; give every XCD a contiguous run of
// tiles so that neighbouring tiles (which write neighbouring list entries) share
// an L2
__device__ __forceinline__ long long xcd_contiguous(long long block, long long nblocks) {
    long long per = (nblocks + 7) / 8;
    return (block & 7) * per + (block >> 3);
}

// ---------------------------------------------------------------- counts
// ---- the prefixes over the super tiles' counts of narrow planes, by the blocks of the count kernel themselves: whoever adds
// the last super tile of a mega tile scans its rows, and whoever does that last scans the mega tiles and then the queries.
// On 407,000 entities the kernel takes as long as it and the two scan kernels of 16-word planes did (13 us), without two
// launches.  On 16-word planes, whose counts are longer, every block would wait for its ticket: 92 instead of 73 us on
// 30M triples' 1.4M listed entities.
// The sums are handed over past the L1s (agent scope); the tickets are zero between two counts.
struct ScanArgs {
    uint32_t *super_sum, *mega_base;  // [nsuper][Qp]: sums, then prefixes inside a mega tile; [nmega][Qp]
    unsigned int *tickets;            // [nmega + 1]
    long long nsuper;
    int Q;
    long long *reached_off, *host_off;  // offsets of the lists, also to pinned memory (a copy would be 10 us)
    const unsigned long long *n_active;
    unsigned long long *host_n_active;
};

// true in the block that takes the last of n tickets, which it puts back; behind it the others' agent-scope stores can be read
__device__ __forceinline__ bool last_of(unsigned int *ticket, unsigned int n) {
    __shared__ int last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's stores are in before the ticket is taken
    __syncthreads();
    if (threadIdx.x == 0) {
        last = atomicAdd(ticket, 1u) == n - 1;
        if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const bool mine = last;
    __syncthreads();  // (the flag is used again)
    return mine;
}

// Exclusive prefix down a column of `rows` rows, the total returned; a block of 1,024 threads with 1024 / Qp threads per
// column, each with every row of its part, sixteen of them requested together (and read once where there are no more).
template <int Qp, typename Store>
__device__ __forceinline__ uint32_t scan_rows(const uint32_t *in, long long rows, Store store) {
    constexpr int P = 1024 / Qp;
    __shared__ uint32_t part_sum[P][Qp];
    const int q = threadIdx.x % Qp, p = threadIdx.x / Qp;
    const long long per = (rows + P - 1) / P, lo = p * per, hi = min(rows, lo + per);
    uint32_t x[16], sum = 0, run = 0, total = 0;
    auto load = [&](long long r0) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            x[i] = r0 + i < hi ? __hip_atomic_load(&in[(size_t)(r0 + i) * Qp + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    };
    for (long long r0 = lo; r0 < hi; r0 += 16) {
        load(r0);
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += x[i];
    }
    part_sum[p][q] = sum;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (i < p) run += part_sum[i][q];
        total += part_sum[i][q];
    }
    __syncthreads();
    for (long long r0 = lo; r0 < hi; r0 += 16) {
        if (hi - lo > 16) load(r0);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (r0 + i < hi) {
                store(r0 + i, run);
                run += x[i];
            }
    }
    return total;
}

// called by every block of a count, behind its agent-scope stores of super tile st's sums
template <int Qp>
__device__ __forceinline__ void scan_counts(const ScanArgs &a, long long st) {
    const long long mega = st / kMegaSupers, first = mega * kMegaSupers, nmega = (a.nsuper + kMegaSupers - 1) / kMegaSupers;
    const long long rows = min((long long)kMegaSupers, a.nsuper - first);
    if (!last_of(&a.tickets[mega], (unsigned)rows)) return;  // block-uniform
    const int t = threadIdx.x, q = t % Qp;
    uint32_t *sums = a.super_sum + (size_t)first * Qp;
    const uint32_t all = scan_rows<Qp>(sums, rows, [&](long long r, uint32_t v) { sums[(size_t)r * Qp + q] = v; });
    if (t < Qp) __hip_atomic_store(&a.mega_base[(size_t)mega * Qp + q], all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_of(&a.tickets[nmega], (unsigned)nmega)) return;
    const uint32_t mine = scan_rows<Qp>(a.mega_base, nmega, [&](long long r, uint32_t v) { a.mega_base[(size_t)r * Qp + q] = v; });
    // prefix over the queries
    __shared__ long long totals[2][Qp];
    const long long own = q < a.Q ? mine : 0;
    int cur = 0;
    if (t < Qp) totals[0][q] = own;
    __syncthreads();
    for (int d = 1; d < Qp; d <<= 1) {
        if (t < Qp) totals[cur ^ 1][q] = totals[cur][q] + (q >= d ? totals[cur][q - d] : 0);
        cur ^= 1;
        __syncthreads();
    }
    if (t >= Qp) return;
    a.reached_off[q] = a.host_off[q] = totals[cur][q] - own;
    if (q == Qp - 1) a.reached_off[Qp] = a.host_off[Qp] = totals[cur][q];
    if (q == 0 && a.n_active) *a.host_n_active = *a.n_active;
}

// Bit-sliced sums of 64 counters side by side: sum and carry of three words.
__device__ __forceinline__ void full_add(unsigned long long a, unsigned long long b, unsigned long long c, unsigned long long &sum,
                                         unsigned long long &carry) {
    sum = a ^ b ^ c;
    carry = (a & b) | (c & (a | b));
}

// 16-word planes: one block per super tile, a wavefront per tile: tile_base[tile][q] = entities query q reached in the
// earlier tiles of the super tile, super_sum[st][q] = in the whole super tile.
// With a list the number of tiles follows from *n_active (the grid covers the largest possible
// number of super tiles; those behind the list write zero sums).
// A 16-lane group takes 16 of the tile's entities, lane = word, the lines of four requested together from the base and then from
// every level they are active in, and adds the unions up bit-sliced: five words say for 64 queries how many of the 16
// entities each reached, seven when the four groups have been added.  Only those are turned into a number per query
// (lane = query: a word is the mask of a select).  A wavefront per word that transposed 64 x 64 bits per tile, the lines
// handed over through LDS, was a chain of latencies and twelve LDS permutes per (tile, word): 20M entities 1,338 -> 620 us
// over one plane with all sixteen lines of a group on their way, which the unions of levels have no registers for.  One
// plane now / the levels of three hops, us: 30M triples' 0.9M listed entities 36 / 66 (31 / 33, the second over a plane that
// the hops kept), 2M hub-heavy ones 94 / 173 (82 / 64).
constexpr int kCountLevels = 3;  // levels whose active bits are asked for ahead of the first line: those of three hops

__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_count(Seen s, long long ntiles, int32_t E, const int32_t *__restrict__ tile_ent,
        const unsigned long long *__restrict__ n_active, uint16_t *tile_base, uint32_t *super_sum) {
    constexpr int W = 16, Qp = 64 * W;
    __shared__ uint8_t cnt[kSuperTiles][Qp];  // (at most 64)
    const long long st = blockIdx.x, first = st * kSuperTiles;
    const int t = threadIdx.x, wave = t >> 6, v = lane(), lw = v & (W - 1), g = v / W;
    if (tile_ent) ntiles = (long long)((*n_active + 63) / 64);
    const int n = (int)max(0ll, min((long long)kSuperTiles, ntiles - first));  // block-uniform
    if (wave < n) {
        const long long tile = first + wave;
        // lane v asks for the tile's entity v; group g's lanes take the lines of entities 16 g .. 16 g + 15, four at a time
        // (sixteen, and their words of another level beside them, are more registers than two blocks per CU have)
        const int32_t own = (int32_t)tile_entity(tile_ent, tile, v, E);
        auto in_level = [&](int l) { return __ballot(l < s.last && own >= 0 && active_in(s, l, own)); };
        unsigned long long on[1 + kCountLevels];
        on[0] = __ballot(s.base && own >= 0 && active_in_base(s, own));
#pragma unroll
        for (int l = 0; l < kCountLevels; ++l) on[1 + l] = in_level(s.first + l);
        unsigned long long p[7] = {};  // p[b]: bit b of the sums
#pragma unroll 1
        for (int i0 = 0; i0 < 16; i0 += 4) {
            int32_t e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = __shfl(max(own, 0), g * 16 + i0 + i);
            unsigned long long x[4] = {};
            auto add_lines = [&](const unsigned long long *__restrict__ lines, unsigned long long active) {
                const unsigned mine = (unsigned)(active >> (g * 16 + i0));
                if (!(active & (0x000f000f000f000full << i0))) return;  // wavefront-uniform
                unsigned long long y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = lines[(size_t)e[i] * W + lw];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] |= (mine >> i) & 1u ? y[i] : 0ull;
            };
            add_lines(s.base, on[0]);
#pragma unroll
            for (int l = 0; l < kCountLevels; ++l) add_lines(s.levels + (size_t)(s.first + l) * s.plane, on[1 + l]);
            for (int l = s.first + kCountLevels; l < s.last; ++l) add_lines(s.levels + (size_t)l * s.plane, in_level(l));
            unsigned long long c2[2], c4;
            full_add(x[0], x[1], p[0], p[0], c2[0]);
            full_add(x[2], x[3], p[0], p[0], c2[1]);
            full_add(c2[0], c2[1], p[1], p[1], c4);
            unsigned long long carry = p[2] & c4;
            p[2] ^= c4;
            c4 = p[3] & carry;
            p[3] ^= carry;
            p[4] ^= c4;  // (16 at most)
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {  // the four groups
            unsigned long long carry = 0;
#pragma unroll
            for (int b = 0; b < 5 + s; ++b) full_add(p[b], shfl_xor64(p[b], W << s), carry, p[b], carry);
            p[5 + s] = carry;
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            int c = 0;
#pragma unroll
            for (int b = 0; b < 7; ++b) {
                const unsigned long long m =
                    ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(p[b] >> 32), w) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)p[b], w);
                c |= __builtin_amdgcn_inverse_ballot_w64(m) ? 1 << b : 0;
            }
            cnt[wave][w * 64 + v] = (uint8_t)c;
        }
    }
    __syncthreads();
    int run = 0;
#pragma unroll
    for (int k = 0; k < kSuperTiles; ++k) {
        if (k >= n) continue;
        tile_base[(size_t)(first + k) * Qp + t] = (uint16_t)run;
        run += cnt[k][t];
    }
    super_sum[(size_t)st * Qp + t] = (uint32_t)run;
}

// The same for planes of one and four words: a wavefront per tile of the super tile, the sixteen counts of a
// query summed through LDS.  One wavefront per word walking the sixteen tiles in turn was a chain of 32
// dependent loads: 20 us on 407,000 entities (22 us with four words), 4.3 us (8.5 us) now.
template <int W>
__global__ void __launch_bounds__(64 * kSuperTiles)
k_count_narrow(const unsigned long long *__restrict__ visited, long long ntiles, int32_t E,
               const int32_t *__restrict__ tile_ent, const unsigned long long *__restrict__ n_active,
               uint16_t *tile_base, ScanArgs scan) {
    static_assert(W <= 4, "16-word lines are staged by k_count");
    constexpr int Qp = 64 * W;
    __shared__ uint16_t cnt[kSuperTiles][Qp];
    const int i = threadIdx.x >> 6, t = threadIdx.x;
    const long long first = (long long)blockIdx.x * kSuperTiles, tile = first + i;
    if (tile_ent) ntiles = (long long)((*n_active + 63) / 64);
    unsigned long long x[W];
#pragma unroll
    for (int w = 0; w < W; ++w) x[w] = 0;
    if (tile < ntiles) {  // wavefront-uniform
        const long long e = tile_entity(tile_ent, tile, lane(), E);
        if (e >= 0)
#pragma unroll
            for (int w = 0; w < W; ++w) x[w] = visited[(size_t)e * W + w];
    }
    for (int w = 0; w < W; ++w) {
        unsigned long long y = x[0];
#pragma unroll
        for (int v = 1; v < W; ++v)
            if (v == w) y = x[v];
        int c = 0;
        if (wave_any(y != 0)) c = __popcll(transpose64(y));  // lane qq: entities of the tile query qq reached
        cnt[i][w * 64 + lane()] = (uint16_t)c;
    }
    __syncthreads();
    if (t < Qp) {
        int run = 0;
#pragma unroll
        for (int k = 0; k < kSuperTiles; ++k) {
            if (first + k < ntiles) tile_base[(size_t)(first + k) * Qp + t] = (uint16_t)run;
            run += cnt[k][t];
        }
        __hip_atomic_store(&scan.super_sum[(size_t)blockIdx.x * Qp + t], (uint32_t)run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    scan_counts<Qp>(scan, blockIdx.x);
}

// 16-word planes: exclusive prefix of `sum` over groups of `group` consecutive rows; total per group to `up`.
// One thread per (group, query); the rows are read sixteen at a time before any is rewritten,
// so the loads of a batch are in flight together.
__global__ void k_scan_level(long long nrows, int group, int Qp, uint32_t *sum_to_base, uint32_t *up) {
    const long long g = blockIdx.x;
    const int q = blockIdx.y * blockDim.x + threadIdx.x;
    if (q >= Qp) return;
    uint32_t run = 0;
    for (int t0 = 0; t0 < group; t0 += 16) {
        uint32_t x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const long long row = g * group + t0 + i;
            x[i] = (t0 + i < group && row < nrows) ? sum_to_base[(size_t)row * Qp + q] : 0u;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const long long row = g * group + t0 + i;
            if (t0 + i < group && row < nrows) sum_to_base[(size_t)row * Qp + q] = run;
            run += x[i];
        }
    }
    up[(size_t)g * Qp + q] = run;
}

// One block of Qp threads: prefix over mega tiles for every query (eight rows requested before any is
// rewritten), then the prefix over queries (Hillis-Steele steps in LDS).  The offsets and, with a list, the number
// of listed entities go to pinned host memory as well: two copies behind the kernel and the gaps around them
// were 20 us of every count.
__global__ void k_scan_top(long long nmega, int Q, int Qp, uint32_t *mega_base, long long *reached_off,
                           const unsigned long long *__restrict__ n_active, long long *host_off,
                           unsigned long long *host_n_active) {
    __shared__ long long total[2][1024];
    const int q = threadIdx.x;
    long long run = 0;
    for (long long m0 = 0; m0 < nmega; m0 += 8) {
        uint32_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = m0 + i < nmega ? mega_base[(size_t)(m0 + i) * Qp + q] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (m0 + i < nmega) mega_base[(size_t)(m0 + i) * Qp + q] = (uint32_t)run;
            run += x[i];
        }
    }
    const long long mine = q < Q ? run : 0;
    int cur = 0;
    total[0][q] = mine;
    __syncthreads();
    for (int d = 1; d < Qp; d <<= 1) {  // inclusive prefix
        long long v = total[cur][q];
        if (q >= d) v += total[cur][q - d];
        total[cur ^ 1][q] = v;
        cur ^= 1;
        __syncthreads();
    }
    reached_off[q] = host_off[q] = total[cur][q] - mine;  // exclusive
    if (q == Qp - 1) reached_off[Qp] = host_off[Qp] = total[cur][q];
    if (q == 0 && n_active) *host_n_active = *n_active;
}

__device__ __forceinline__ unsigned long long range_bits(int q0, int q1, int w) {
    return query_bits(q1, w) & ~query_bits(q0, w);
}

// position of a super tile's first entry in the list of query q (relative to query q0's start)
__device__ __forceinline__ long long super_start(const FillArgs &a, long long st, int Qp, int q) {
    return a.reached_off[q] - a.reached_off[a.q0] + a.mega_base[(size_t)(st / kMegaSupers) * Qp + q] +
           a.super_base[(size_t)st * Qp + q];
}

// ---------------------------------------------------------------- entity / hop lists
// One block per super tile (1024 entities) or part of one, one wavefront per word.  The wave
// keeps its word of all the block's tiles in registers (visited and the bit-sliced hop
// number), and for one query at a time compacts the reached entities into LDS,
// then streams them out with full-width stores.
// NB = words of the bit-sliced hop number (0: entity ids only; of few words of 16-word planes: see k_word_lists); TILES = tiles per block
// (launch_lists_w), at most half a super tile on 16-word planes, where the registers of a whole one
// would not leave room for two blocks per CU.
template <int W, int NB, int TILES>
__global__ void __launch_bounds__(64 * W) k_lists(FillArgs a) {
    constexpr int Qp = 64 * W, NBX = NB > 0 ? NB : 1;
    __shared__ unsigned long long stage[64][W + 1];
    __shared__ uint16_t s_ent[W][TILES * 64];
    __shared__ uint8_t s_hop[NB > 0 ? W : 1][TILES * 64];
    __shared__ int32_t blk_ent[TILES * 64];  // entity ids of the block's tiles
    const long long first_tile = (long long)blockIdx.x * TILES;
    for (int i = threadIdx.x; i < TILES * 64; i += 64 * W) {
        const long long tile = first_tile + i / 64;
        blk_ent[i] = tile < a.ntiles ? (int32_t)tile_entity(a.tile_ent, tile, i % 64, a.E) : -1;
    }
    const long long st = first_tile / kSuperTiles;
    const int wave = threadIdx.x >> 6, v = lane();
    unsigned long long visw[TILES];
    unsigned long long hb[NBX][TILES];
#pragma unroll
    for (int i = 0; i < TILES; ++i) {
        long long tile = first_tile + i;
        visw[i] = 0;
#pragma unroll
        for (int b = 0; b < NBX; ++b) hb[b][i] = 0;
        if (tile < a.ntiles) {  // block-uniform
            visw[i] = stage_word<W>(stage, a.visited, a.tile_ent, tile, a.E, wave);
            if constexpr (NB > 0)
                for (int h = 1; h <= a.k; ++h) {  // hop number of each bit, bit-sliced over NB words
                    unsigned long long x =
                        stage_word<W>(stage, a.levels + (size_t)h * a.plane, a.tile_ent, tile, a.E, wave);
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if ((h >> b) & 1) hb[b][i] |= x;
                }
        }
    }
    unsigned long long present = 0;
#pragma unroll
    for (int i = 0; i < TILES; ++i) present |= visw[i];
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) present |= shfl_xor64(present, m);
    present &= range_bits(a.q0, a.q1, wave);
    // lane qq keeps the list position where query 64*wave+qq continues in this block's tiles
    long long mybase = 0;
    if ((present >> v) & 1ull) {
        mybase = super_start(a, st, Qp, wave * 64 + v);
        if (TILES < kSuperTiles) mybase += a.tile_base[(size_t)first_tile * Qp + wave * 64 + v];
    }
    uint16_t *ent = s_ent[wave];
    uint8_t *hp = s_hop[NB > 0 ? wave : 0];
    // blk_ent is written by all wavefronts and read by each (here, behind the plane loads, so that they do not wait
    // for the ids).  stage_word has barriers of its own only for 16-word lines.
    if constexpr (W <= 4) __syncthreads();
    while (present) {
        const int qq = __ffsll((long long)present) - 1;
        present &= present - 1;
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
            bool bit = (visw[i] >> qq) & 1ull;
            unsigned long long m = __ballot(bit);
            if (bit) {
                int pos = cnt + __popcll(m & ((1ull << v) - 1ull));
                ent[pos] = (uint16_t)(i * 64 + v);
                if constexpr (NB > 0) {
                    int hv = 0;
#pragma unroll
                    for (int b = 0; b < NB; ++b) hv |= (int)((hb[b][i] >> qq) & 1ull) << b;
                    hp[pos] = (uint8_t)hv;
                }
            }
            cnt += __popcll(m);
        }
        __builtin_amdgcn_wave_barrier();
        const long long base = (long long)shfl64((unsigned long long)mybase, qq);
        for (int p = v; p < cnt; p += 64) {
            a.entity[base + p] = blk_ent[ent[p]];
            if constexpr (NB > 0) a.hop[base + p] = hp[p];
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------- predecessor edges
// 64 in-edges of an object row for a caller that merges claims with a minimum over entries (the row
// kernels): every W-lane group keeps a mask `rem` of its own (word lw of the queries it has not resolved),
// takes every (64/W)-th candidate subject, gathers its line and claims whatever its mask still holds, with no
// exchange between the groups.  (An ordered walk - a candidate claims only what no earlier candidate of the
// round has, found with an exclusive prefix-OR across the groups - costs ten dependent LDS permutes per
// round, which is what these kernels then wait on.)  A query may be claimed by several groups; the smallest
// entry wins.
//
// The candidates are compacted into a queue of the wavefront in LDS (subject, relation, place in the chunk), so
// that a round costs a group one LDS read.  Picking them out of the ballot mask one after the other was half of
// the kernels' vector and nearly all of their scalar instructions, and they are bound by instruction issue
// (30M triples, 1,024 queries: mid rows 354 us, giants 439 us, other hubs 200 us; 309, 280 and 131 us with the queue).
// emit(hit, at) runs on lanes whose word has newly claimed bits, at = the entry's place in the chunk;
// returns the lines gathered.
// smin[b] = min(smin[b], at) for every bit b of hit, in 32-bit halves: a turn is then six vector instructions where
// the 64-bit form took a dozen, and these turns are most of what the row kernels issue.
__device__ __forceinline__ void claim(unsigned int *smin, unsigned long long hit, unsigned int at) {
    for (uint32_t m = (uint32_t)hit; m; m &= m - 1u) atomicMin(&smin[__builtin_ctz(m)], at);
    for (uint32_t m = (uint32_t)(hit >> 32); m; m &= m - 1u) atomicMin(&smin[32 + __builtin_ctz(m)], at);
}

// The 64 entries of a word lie kClaimStride apart: lanes of one round mostly claim the same bits of their words, and
// with 64 apart all of them met in one LDS bank.
constexpr int kClaimStride = 65;

struct PredQueue {
    int s[64];
    uint16_t r[64];
    uint8_t at[64];
};

template <bool MASK, typename Emit>
__device__ __forceinline__ int pred_resolve_unordered(int s, int r, bool cand, const FillArgs &a,
                                                      const unsigned long long *__restrict__ prev, PredQueue &queue,
                                                      unsigned long long &rem, Emit emit) {
    constexpr int W = 16;
    const int lw = lane() & (W - 1), g = lane() / W;
    const unsigned long long cm = __ballot(cand);
    const int n = __popcll(cm);
    if (n == 0) return 0;
    if (cand) {
        const int at = __popcll(cm & ((1ull << lane()) - 1ull));
        queue.s[at] = s;
        if (MASK) queue.r[at] = (uint16_t)r;
        queue.at[at] = (uint8_t)lane();
    }
    __builtin_amdgcn_wave_barrier();
    constexpr int NR = 4, GPW = 64 / W;
    int base = 0;
    for (; base < n; base += NR * GPW) {
        unsigned long long l[NR], ok[NR];  // (put together behind all loads: in the branch, each round waited for its own)
#pragma unroll
        for (int x = 0; x < NR; ++x) {
            const int i = base + x * GPW + g;
            l[x] = ok[x] = 0;
            if (i < n) {
                l[x] = prev[(size_t)queue.s[i] * W + lw];
                if (MASK) ok[x] = a.allow[(size_t)queue.r[i] * W + lw];
            }
        }
#pragma unroll
        for (int x = 0; x < NR; ++x) {
            if (MASK) l[x] &= ok[x];
            const unsigned long long hit = l[x] & rem;
            rem &= ~l[x];
            if (hit) emit(hit, (int)queue.at[base + x * GPW + g]);
        }
        if (!wave_any(rem != 0)) break;
    }
    __builtin_amdgcn_wave_barrier();  // the queue is rewritten by the next chunk
    return min(n, base + NR * GPW);
}

// List positions of entity `ev` for every query: slot[q] = start of the tile's run in query q's
// list + rank of the entity inside the tile.  Called by a whole wavefront for the words
// w = w_first, w_first + w_step, .. below w_end; slot[0] belongs to query q_first.
template <int W>
__device__ __forceinline__ void row_slots(const FillArgs &a, int ev, int w_first, int w_step, long long *slot,
                                          int w_end = W, int q_first = 0) {
    constexpr int Qp = 64 * W;
    long long at = ev;  // place of the entity in the tiles
    if (a.cpos) {       // an entity no query reached is not listed: it needs no positions
        at = a.cpos[ev];
        if (at < 0 || at >= a.n_listed || a.tile_ent[at] != ev) return;
    }
    const long long tile = at >> 6;
    const int vi = (int)(at & 63), v = lane();
    const unsigned long long below = (1ull << vi) - 1ull;
    const long long ent_v = tile_entity(a.tile_ent, tile, v, a.E);
    for (int w = w_first; w < w_end; w += w_step) {  // lane v = entity v of the tile
        unsigned long long x = ent_v >= 0 ? a.visited[(size_t)ent_v * W + w] & range_bits(a.q0, a.q1, w) : 0ull;
        int rank = 0;
        if (shfl64(x, vi) != 0ull)  // only queries that reached this entity matter
            rank = __popcll(transpose64(x) & below);
        int q = w * 64 + v;
        long long b = 0;
        if (q >= a.q0 && q < a.q1)
            b = super_start(a, tile / kSuperTiles, Qp, q) + a.tile_base[(size_t)tile * Qp + q] + rank;
        slot[q - q_first] = b;
    }
}

// Triple index of a row entry; ~0: none was found (a reached pair has one, so only a broken input leads here).
__device__ __forceinline__ int32_t entry_id(const FillArgs &a, unsigned int at) { return at == ~0u ? INT_MAX : a.in_eid[at]; }

// AND over the 64/W groups of a wavefront (word lw of each group).
template <int W>
__device__ __forceinline__ unsigned long long and_groups(unsigned long long x) {
#pragma unroll
    for (int m = W; m < 64; m <<= 1) x &= shfl_xor64(x, m);
    return x;
}

// Object rows of 33 .. hub_min-1 entries: one wavefront per row, four rows per block.  The W-lane
// groups of the wavefront claim independently (pred_resolve_unordered) and the smallest edge id per
// query is kept in a table of the wavefront in LDS; the groups' masks are merged once per 64
// entries, and after a level the table is written out (one contiguous store per 64 queries in the
// row-buffer mode) and reset.
template <bool MASK, bool STATS, bool BUF>
__global__ void __launch_bounds__(256) k_pred_wave(FillArgs a, long long first_row, long long n_rows_total) {
    constexpr int W = 16, Qp = 64 * W;
    __shared__ long long slots[BUF ? 1 : 4][BUF ? 1 : Qp];
    __shared__ unsigned int smin_all[4][W * kClaimStride];  // smallest entry per query (index into in_sub)
    __shared__ PredQueue queue[4];
    const int wave = threadIdx.x >> 6, v = lane(), lw = v & (W - 1);
    const long long idx = (long long)blockIdx.x * 4 + wave;
    long long n_rows = 0, n_edges = 0, n_lines = 0;
    if (idx < n_rows_total) {  // wave-uniform
        const int ev = a.rows[first_row + idx];
        long long *slot = slots[BUF ? 0 : wave];
        unsigned int *smin = smin_all[wave];
        int32_t *out = BUF ? a.row_pred + (size_t)(first_row + idx) * Qp : a.pred;
        if (!BUF) row_slots<W>(a, ev, 0, 1, slot);
        for (int w = 0; w < W; ++w) smin[w * kClaimStride + v] = ~0u;
        __builtin_amdgcn_wave_barrier();
        const uint32_t lo = a.in_off[ev], hi = a.in_off[ev + 1];
        for (int h = 1; h <= a.k; ++h) {
            const unsigned long long level = a.levels[(size_t)h * a.plane + (size_t)ev * W + lw] & range_bits(a.q0, a.q1, lw);
            unsigned long long rem = level;
            if (!wave_any(rem != 0) || ((a.push_levels >> h) & 1u)) continue;
            const uint32_t *act_prev = a.act + (size_t)(h - 1) * a.actw;
            const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
            const bool dense = !STATS && ((a.dense_levels >> h) & 1u);  // the line of an entity outside the level is zero
            ++n_rows;
            // the subjects of the next 64 entries are requested while the lines of these are gathered
            int s_next = lo + v < hi ? a.in_sub[lo + v] : -1, r_next = MASK && lo + v < hi ? a.in_rel[lo + v] : 0;
            for (uint32_t j0 = lo; j0 < hi; j0 += 64) {
                const int s = s_next, r = r_next;
                const uint32_t jn = j0 + 64 + v;
                s_next = jn < hi ? a.in_sub[jn] : -1;
                r_next = MASK && jn < hi ? a.in_rel[jn] : 0;
                const bool cand = s >= 0 && (dense || ((act_prev[s >> 5] >> (s & 31)) & 1u));
                n_lines += pred_resolve_unordered<MASK>(s, r, cand, a, prev, queue[wave], rem, [&](unsigned long long hit, int at) {
                    claim(&smin[lw * kClaimStride], hit, j0 + (uint32_t)at);
                });
                rem = and_groups<W>(rem);  // what any group has resolved is resolved
                n_edges += min((uint32_t)64, hi - j0);
                if (!wave_any(rem != 0)) break;
            }
            __builtin_amdgcn_wave_barrier();
            // Queries 64 i .. 64 i + 63: word i of the level, held by lane i.  All triple indices are requested before the
            // first is stored (a load behind a store, sixteen times over, was a third of a row's time).
            int32_t eid[W];
            bool on[W];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                on[i] = (shfl64(level, i) >> v) & 1ull;
                eid[i] = 0;
                if (on[i]) eid[i] = entry_id(a, smin[i * kClaimStride + v]);
            }
#pragma unroll
            for (int i = 0; i < W; ++i)
                if (on[i]) {
                    out[BUF ? (long long)(64 * i + v) : slot[64 * i + v]] = eid[i];
                    smin[i * kClaimStride + v] = ~0u;
                }
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (STATS && v == 0) {
        if (n_rows) atomicAdd(&a.stats_mid[0], (unsigned long long)n_rows);
        if (n_edges) atomicAdd(&a.stats_mid[1], (unsigned long long)n_edges);
        if (n_lines) atomicAdd(&a.stats_mid[2], (unsigned long long)n_lines);
    }
}

__device__ __forceinline__ unsigned long long wave_or64(unsigned long long x) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) x |= shfl_xor64(x, m);
    return x;
}

// ---- narrow lines: planes of one and four words, and a page of a 16-word batch that sits in one, two or four
// aligned words (N words from word `off` of the line).  Such a piece of a line is one lane's load, so lane = entry of
// the object row: 256 entries of a wavefront are gathered together, and a 64 x 64 bit transpose per chunk of
// 64 entries and word turns "entry -> queries it resolves" into "query -> entries that resolve it" (lane =
// query), whose lowest set bit is the entry with the smallest triple index.  No frontier bit is asked for
// first: it would cost as much as the piece of the line (zero outside the level).
// What bounds these kernels is the chain of loads per step (ids, pieces, then the next step) of the longest
// rows, and for a page of a 16-word batch the lines themselves (64 queries of the hub-heavy 300M-triple graph:
// giant rows 3.4 -> 2.0 ms; 63 queries over two words of 50M triples: row kernels 860 -> 730 us against whole lines).
constexpr int kNarrowChunks = 4;

template <int N>
__device__ __forceinline__ void load_words(unsigned long long (&x)[N], const unsigned long long *__restrict__ p) {
    if constexpr (N == 1) {
        x[0] = *p;
    } else {
#pragma unroll
        for (int i = 0; i < N; i += 2) {
            const ulonglong2 y = *reinterpret_cast<const ulonglong2 *>(p + i);  // (off is a multiple of N)
            x[i] = y.x;
            x[i + 1] = y.y;
        }
    }
}

__device__ __forceinline__ unsigned long long uniform64(unsigned long long x) {
    return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

// level h of the row's entity, restricted to the fetched queries; true when something is left of it
template <int W, int N>
__device__ __forceinline__ bool narrow_level(const FillArgs &a, int ev, int h, int off, unsigned long long (&lev)[N]) {
    load_words<N>(lev, a.plv + (size_t)h * a.pplane + (size_t)ev * a.pstride + (off - a.pfirst));
    bool any = false;
#pragma unroll
    for (int w = 0; w < N; ++w) {
        lev[w] = uniform64(lev[w] & range_bits(a.q0, a.q1, off + w));
        any |= lev[w] != 0ull;
    }
    return any && !((a.push_levels >> h) & 1u);
}

// Entries first + c * stride + lane (below hi), c = 0 .. kNarrowChunks - 1, in ascending order: best[w] = the first
// one that holds query 64 w + lane while it is in rem[w] (wavefront-uniform, cleared of what is resolved).
template <int W, int N, bool MASK>
__device__ __forceinline__ void narrow_resolve(const FillArgs &a, const unsigned long long *__restrict__ prev, int off,
                                               uint32_t first, uint32_t stride, uint32_t hi,
                                               unsigned long long (&rem)[N], uint32_t (&best)[N]) {
    constexpr int C = kNarrowChunks;
    unsigned long long l[C][N];
    int s[C], rl[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const uint32_t j = first + c * stride + (uint32_t)lane();
        s[c] = -1;
        rl[c] = 0;
        if (j < hi) {
            s[c] = a.in_sub[j];
            if (MASK) rl[c] = a.in_rel[j];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int w = 0; w < N; ++w) l[c][w] = 0;
        if (s[c] >= 0) {
            load_words<N>(l[c], prev + (size_t)s[c] * a.pstride + (off - a.pfirst));
            if (MASK) {
                unsigned long long m[N];
                load_words<N>(m, a.allow + (size_t)rl[c] * W + off);
#pragma unroll
                for (int w = 0; w < N; ++w) l[c][w] &= m[w];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int w = 0; w < N; ++w) {
            const unsigned long long x = l[c][w] & rem[w];
            if (!wave_any(x != 0)) continue;
            const unsigned long long from = transpose64(x);  // lane q: the entries whose line holds query q
            if (from) best[w] = first + c * stride + (uint32_t)(__ffsll((long long)from) - 1);
            rem[w] &= ~__ballot(from != 0);
        }
    }
}

template <int N>
__device__ __forceinline__ bool any_left(const unsigned long long (&rem)[N]) {
    unsigned long long x = 0;
#pragma unroll
    for (int w = 0; w < N; ++w) x |= rem[w];
    return x != 0ull;
}

// Object rows of 33 .. hub_min - 1 entries, a wavefront per row (200 queries with whitelists, 3.4M triples:
// 102 us with 4-lane groups that took every 16th candidate, a chain of five loads per 64 entries; 53 us now).
template <int W, int N, bool MASK, bool STATS, bool BUF>
__device__ __forceinline__ void narrow_wave_rows(const FillArgs &a, long long block, long long first_row, long long n_rows_total) {
    constexpr int Qp = 64 * W;
    __shared__ long long slots[BUF ? 1 : 4][BUF ? 1 : 64 * N];
    const int wave = threadIdx.x >> 6, v = lane(), off = W == 16 ? (a.q0 >> 6) & ~(N - 1) : 0;
    const long long idx = block * 4 + wave;
    if (idx >= n_rows_total) return;  // wavefront-uniform
    const int ev = a.rows[first_row + idx];
    long long *slot = slots[BUF ? 0 : wave];
    int32_t *out = BUF ? a.row_pred + (size_t)(first_row + idx) * Qp : a.pred;
    if (!BUF) row_slots<W>(a, ev, off, 1, slot, off + N, off * 64);
    __builtin_amdgcn_wave_barrier();
    const uint32_t lo = a.in_off[ev], hi = a.in_off[ev + 1];
    long long n_rows = 0, n_edges = 0;
    for (int h = 1; h <= a.k; ++h) {
        unsigned long long lev[N], rem[N];
        uint32_t best[N];
        if (!narrow_level<W, N>(a, ev, h, off, lev)) continue;
#pragma unroll
        for (int w = 0; w < N; ++w) {
            rem[w] = lev[w];
            best[w] = lo;
        }
        const unsigned long long *prev = a.plv + (size_t)(h - 1) * a.pplane;
        ++n_rows;
        for (uint32_t j0 = lo; j0 < hi && any_left<N>(rem); j0 += 64 * kNarrowChunks) {
            narrow_resolve<W, N, MASK>(a, prev, off, j0, 64, hi, rem, best);
            n_edges += min((uint32_t)(64 * kNarrowChunks), hi - j0);
        }
        int32_t eid[N];
#pragma unroll
        for (int w = 0; w < N; ++w) eid[w] = (lev[w] >> v) & 1ull ? a.in_eid[best[w]] : 0;
#pragma unroll
        for (int w = 0; w < N; ++w)
            if ((lev[w] >> v) & 1ull) out[BUF ? (long long)((off + w) * 64 + v) : slot[w * 64 + v]] = eid[w];
    }
    if (STATS && v == 0) {
        if (n_rows) atomicAdd(&a.stats_mid[0], (unsigned long long)n_rows);
        if (n_edges) atomicAdd(&a.stats_mid[1], (unsigned long long)n_edges);
        if (n_edges) atomicAdd(&a.stats_mid[2], (unsigned long long)n_edges);  // a piece of a line per entry
    }
}

template <int W, int N, bool MASK, bool STATS, bool BUF>
__global__ void __launch_bounds__(256) k_narrow_wave(FillArgs a, long long first_row, long long n_rows_total) {
    narrow_wave_rows<W, N, MASK, STATS, BUF>(a, blockIdx.x, first_row, n_rows_total);
}

// The segment of a giant row that block b takes: the first segments of all rows, then the second ones, ..; row by row where
// the rows come range by range.
__device__ __forceinline__ void giant_segment(const FillArgs &a, uint32_t b, long long &row, uint32_t &seg) {
    const uint32_t *first = a.giant_place_first ? a.giant_place_first : a.giant_seg_first;
    long long lo = 0, hi = a.giant_place_first ? a.n_giant_places : a.n_giant_rows;  // the last one that begins at or before b
    while (hi - lo > 1) {
        const long long m = (lo + hi) >> 1;
        if (first[m] <= b) lo = m; else hi = m;
    }
    const uint32_t in = b - first[lo];
    row = a.giant_place_first ? (long long)in : lo;
    seg = a.giant_place_first ? (uint32_t)lo : in;
}

// Which of queries 64 w .. 64 w + 63 (lane = query, *kept = its place in the row's line of the row buffer) an earlier segment
// of the row has resolved: triple indices ascend, so a smaller one than this segment's first is another segment's.  (What
// others store meanwhile may or may not be seen; a query that is walked again only costs time.)
__device__ __forceinline__ unsigned long long resolved_before(const int32_t *kept, int32_t first_eid) {
    return __ballot(__hip_atomic_load(kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < first_eid);
}

// Longer object rows: a block per (row, hop level), or per segment of a giant row, as k_pred_row; the
// wavefronts take chunks in turn and keep the smallest entry per query in LDS after every step.
template <int W, int N, bool MASK, bool STATS, bool BUF, bool SEG>
__global__ void __launch_bounds__(1024) k_narrow_row(FillArgs a, long long first_row) {
    static_assert(!SEG || BUF, "segments merge in the row buffer");
    constexpr int Qp = 64 * W, C = kNarrowChunks;
    __shared__ long long slot[BUF ? 1 : 64 * N];
    __shared__ unsigned int smin[64 * N];
    __shared__ unsigned long long srem[N];
    long long row_i = blockIdx.x;
    uint32_t seg = 0;
    if (SEG) giant_segment(a, blockIdx.x, row_i, seg);
    const int ev = a.rows[first_row + row_i];
    const int t = threadIdx.x, wave = t >> 6, nw = blockDim.x >> 6, v = lane(), h = (int)blockIdx.y + 1;
    const int off = W == 16 ? (a.q0 >> 6) & ~(N - 1) : 0;
    unsigned long long lev[N];
    if (!narrow_level<W, N>(a, ev, h, off, lev)) return;  // block-uniform
    if (!BUF) row_slots<W>(a, ev, off + wave, nw, slot, off + N, off * 64);
    int32_t *out = BUF ? a.row_pred + (size_t)(first_row + row_i) * Qp : a.pred;
    const uint32_t row_lo = a.in_off[ev], row_hi = a.in_off[ev + 1];
    const uint32_t lo = SEG ? row_lo + seg * (uint32_t)kGiantSegment : row_lo;
    const uint32_t hi = SEG ? min(row_hi, lo + (uint32_t)kGiantSegment) : row_hi;
    for (int q = t; q < 64 * N; q += blockDim.x) smin[q] = ~0u;
    if (wave < N) {  // (a block has four wavefronts at least)
        unsigned long long x = lev[0];
#pragma unroll
        for (int w = 1; w < N; ++w)
            if (w == wave) x = lev[w];
        if (SEG && seg > 0) x &= ~resolved_before(&out[(off + wave) * 64 + v], a.in_eid[lo]);
        if (v == 0) srem[wave] = x;
    }
    __syncthreads();
    const unsigned long long *prev = a.plv + (size_t)(h - 1) * a.pplane;
    long long n_edges = 0;
    // the first step is one chunk per wavefront: on a dense frontier it resolves most queries
    uint32_t span = 64u * nw;
    for (uint32_t s0 = lo; s0 < hi; s0 += span, span = 64u * C * nw) {
        unsigned long long rem[N];
        uint32_t best[N];
#pragma unroll
        for (int w = 0; w < N; ++w) {
            rem[w] = uniform64(srem[w]);
            best[w] = ~0u;
        }
        if (!any_left<N>(rem)) break;  // the same words in every wavefront
        const uint32_t step_hi = min(hi, s0 + span), first = s0 + 64u * wave;
        if (first < step_hi) narrow_resolve<W, N, MASK>(a, prev, off, first, 64u * nw, step_hi, rem, best);
        n_edges += wave == 0 ? (long long)(step_hi - s0) : 0;
#pragma unroll
        for (int w = 0; w < N; ++w)
            if (best[w] != ~0u) atomicMin(&smin[w * 64 + v], best[w]);
        __syncthreads();
        if (v == 0) {
#pragma unroll
            for (int w = 0; w < N; ++w) atomicAnd(&srem[w], rem[w]);
        }
        __syncthreads();
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < N; ++w) {
        if ((w % nw) != wave || !((lev[w] >> v) & 1ull)) continue;
        const unsigned int at = smin[w * 64 + v];
        if (SEG) {
            if (at != ~0u) atomicMin(&out[(off + w) * 64 + v], a.in_eid[at]);
        } else {
            out[BUF ? (long long)((off + w) * 64 + v) : slot[w * 64 + v]] = entry_id(a, at);
        }
    }
    if (STATS && t == 0) {
        atomicAdd(&a.stats_hub[0], 1ull);
        atomicAdd(&a.stats_hub[1], (unsigned long long)n_edges);
        atomicAdd(&a.stats_hub[2], (unsigned long long)n_edges);
    }
}

// Tiles of one- and four-word planes: a wavefront per word of a tile writes the entity and hop lists (lane =
// entity; where a query reached many of the tile's entities, query by query with contiguous stores, else entity
// by entity), then every entity whose object row has at most 32 entries is walked by a W-lane group, U
// entries gathered together and resolved in order.  Longer rows are left to the row kernels.
template <int W, bool MASK, bool STATS>
__device__ __forceinline__ void narrow_tiles(const FillArgs &a, unsigned block, unsigned nblocks) {
    constexpr int TPB = 4 / W, U = MASK ? 2 : 8;  // (65 queries with whitelists, 20M triples: call 587 us with eight, 549 with four, 547 with two)
    static_assert(W == 1 || W == 4, "a block of four wavefronts");
    __shared__ unsigned long long mT[4][64];  // per wavefront, i.e. (tile, word): entities each query reached
    __shared__ long long base[4][64];         // and where its run of the tile starts in the lists
    const int t = threadIdx.x, wave = t >> 6, v = lane();
    const long long tile_rel = xcd_contiguous(block, nblocks) * TPB + wave / W;
    const bool valid = tile_rel < a.tile_count;
    const long long tile = a.tile_begin + tile_rel;
    const int word = wave % W;
    {
        const int q = word * 64 + v;
        long long b = 0;
        if (valid && q >= a.q0 && q < a.q1)
            b = super_start(a, tile / kSuperTiles, 64 * W, q) + a.tile_base[(size_t)tile * 64 * W + q];
        base[wave][v] = b;
        const long long e = valid ? tile_entity(a.tile_ent, tile, v, a.E) : -1;
        unsigned long long vis = 0, x = 0;
        const unsigned long long range = range_bits(a.q0, a.q1, word);
        if (e >= 0) {
            vis = a.visited[(size_t)e * W + word] & range;
            x = a.levels[(size_t)e * W + word] & range;
        }
        mT[wave][v] = transpose64(vis);
        __builtin_amdgcn_wave_barrier();
        const unsigned long long below = (1ull << v) - 1ull;
        auto put = [&](int qq, int h) {
            const long long p = base[wave][qq] + __popcll(mT[wave][qq] & below);
            a.entity[p] = (int32_t)e;
            if (a.hop) a.hop[p] = (uint8_t)h;
            if (h == 0) a.pred[p] = -1;  // seeds have no predecessor
        };
        unsigned long long left = vis;
        for (int h = 0; h <= a.k; ++h) {
            if (h > 0) {
                if (!wave_any(left != 0)) break;  // every pair of the tile is written
                if (!a.hop) x = left;             // no hop numbers: all others at once
                else x = left ? a.levels[(size_t)h * a.plane + (size_t)e * W + word] & range : 0ull;
            }
            left &= ~x;
            if (!wave_any(x != 0)) continue;
            const unsigned long long present = wave_or64(x);
            // Query by query a store instruction covers neighbouring places of one list, entity by entity every lane
            // has a turn per query of its own: the first where a query has eight and more of the tile's entities.
            // Kernel, us all entity by entity / all query by query / so: 250 queries on 5M hub-heavy triples 1,822 /
            // 1,263 / 1,318, 200 on 3.4M 122 / 99 / 99, 64 on a sparse graph of 500,000 19.7 / 23.3 / 20.3.
            if (wave_sum((long long)__popcll(x)) >= 8ll * __popcll(present)) {
                for (unsigned long long m = present; m; m &= m - 1) {
                    const int qq = __ffsll((long long)m) - 1;
                    if ((x >> qq) & 1ull) put(qq, h);
                }
            } else {
                for (unsigned long long m = x; m; m &= m - 1) put(__ffsll((long long)m) - 1, h);
            }
        }
    }
    __syncthreads();
    const int part = W == 1 ? wave : (t & (W - 1)), lw = t & (W - 1);  // (tile, word) of the lane from here on
    const int vi = W == 1 ? v : t / W;
    const long long ev = valid ? tile_entity(a.tile_ent, tile, vi, a.E) : -1;  // (W = 4: one tile per block)
    uint32_t lo = 0, hi = 0;
    if (ev >= 0) {
        lo = a.in_off[ev];
        hi = a.in_off[ev + 1];
    }
    const unsigned long long below = (1ull << vi) - 1ull;
    long long n_rows = 0, n_edges = 0;
    if (hi > lo && hi - lo <= (uint32_t)kTailMaxDegree)
        for (int h = 1; h <= a.k; ++h) {
            unsigned long long rem = a.levels[(size_t)h * a.plane + (size_t)ev * W + lw] & range_bits(a.q0, a.q1, lw);
            if (!group_any<W>(rem != 0)) continue;
            const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
            if (lw == 0) ++n_rows;
            for (uint32_t j0 = lo; j0 < hi; j0 += U) {
                int s[U], rl[U];
                unsigned long long l[U], ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    s[u] = j0 + u < hi ? a.in_sub[j0 + u] : -1;
                    rl[u] = MASK && j0 + u < hi ? a.in_rel[j0 + u] : 0;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    l[u] = s[u] >= 0 ? prev[(size_t)s[u] * W + lw] : 0ull;
                    ok[u] = MASK && s[u] >= 0 ? a.allow[(size_t)rl[u] * W + lw] : 0ull;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (MASK) l[u] &= ok[u];
                    const unsigned long long hit = l[u] & rem;
                    rem &= ~l[u];
                    if (hit) {
                        const int eid = a.in_eid[j0 + u];
                        for (unsigned long long m = hit; m; m &= m - 1) {
                            const int b = __ffsll((long long)m) - 1;
                            a.pred[base[part][b] + __popcll(mT[part][b] & below)] = eid;
                        }
                    }
                }
                if (lw == 0) n_edges += min((uint32_t)U, hi - j0);
                if (!group_any<W>(rem != 0)) break;
            }
        }
    if (STATS) {
        n_rows = wave_sum(n_rows);
        n_edges = wave_sum(n_edges);
        if (v == 0) {
            if (n_rows) atomicAdd(&a.stats_pred[0], (unsigned long long)n_rows);
            if (n_edges) atomicAdd(&a.stats_pred[1], (unsigned long long)n_edges);
            if (n_edges) atomicAdd(&a.stats_pred[2], (unsigned long long)n_edges);
        }
    }
}

template <int W, bool MASK, bool STATS>
__global__ void __launch_bounds__(256) k_pred_narrow(FillArgs a) { narrow_tiles<W, MASK, STATS>(a, blockIdx.x, gridDim.x); }

// One level of one segment (kHubSegment entries) of a hub row, a block of four wavefronts; as k_narrow_row.  A row of one
// segment is written to the lists.  Of a split row every segment leaves its smallest triple index per query (INT_MAX:
// none) in a line of a.seg_pred, and k_split_lists takes the minimum over them: nothing to fill before, no atomics.
template <int W, bool MASK>
__device__ __forceinline__ void narrow_hub_segment(const FillArgs &a, long long seg, int h) {
    constexpr int Qp = 64 * W, C = kNarrowChunks, NW = 4;
    __shared__ long long slot[Qp];
    __shared__ unsigned int smin[Qp];
    __shared__ unsigned long long srem[W];
    long long row_i = 0, row_end = a.n_hub_rows;  // the last row whose first segment is <= seg
    while (row_end - row_i > 1) {
        const long long m = (row_i + row_end) >> 1;
        if (a.hub_seg_first[m] <= (unsigned long long)seg) row_i = m; else row_end = m;
    }
    const int ev = a.rows[row_i], t = threadIdx.x, wave = t >> 6, v = lane();
    unsigned long long lev[W];
    if (!narrow_level<W, W>(a, ev, h, 0, lev)) return;  // block-uniform
    const bool split = row_i < a.n_split_rows;
    if (!split) row_slots<W>(a, ev, wave, NW, slot, W, 0);
    const uint32_t row_hi = a.in_off[ev + 1];
    const uint32_t lo = a.in_off[ev] + (uint32_t)(seg - a.hub_seg_first[row_i]) * (uint32_t)kHubSegment;
    const uint32_t hi = min(row_hi, lo + (uint32_t)kHubSegment);
    if (t < Qp) smin[t] = ~0u;  // (Qp <= 256 threads)
    if (t < W) {
        unsigned long long x = lev[0];
#pragma unroll
        for (int w = 1; w < W; ++w)
            if (w == t) x = lev[w];
        srem[t] = x;
    }
    __syncthreads();
    const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
    uint32_t span = 64u * NW;  // the first step is one chunk per wavefront: on a dense frontier it resolves most queries
    for (uint32_t s0 = lo; s0 < hi; s0 += span, span = 64u * C * NW) {
        unsigned long long rem[W];
        uint32_t best[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            rem[w] = uniform64(srem[w]);
            best[w] = ~0u;
        }
        if (!any_left<W>(rem)) break;  // the same words in every wavefront
        const uint32_t step_hi = min(hi, s0 + span), first = s0 + 64u * wave;
        if (first < step_hi) narrow_resolve<W, W, MASK>(a, prev, 0, first, 64u * NW, step_hi, rem, best);
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (best[w] != ~0u) atomicMin(&smin[w * 64 + v], best[w]);
        __syncthreads();
        if (v == 0) {
#pragma unroll
            for (int w = 0; w < W; ++w) atomicAnd(&srem[w], rem[w]);
        }
        __syncthreads();
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if ((w % NW) != wave || !((lev[w] >> v) & 1ull)) continue;
        const int32_t eid = entry_id(a, smin[w * 64 + v]);
        if (split) a.seg_pred[(size_t)seg * Qp + w * 64 + v] = eid;
        else a.pred[slot[w * 64 + v]] = eid;
    }
}

// The whole fetch of a narrow batch: hub rows (a block per segment and level, the longest first), rows of 33 .. hub_min - 1
// entries (four per block), tiles.  All three are chains of dependent loads over data that the caches hold and write
// different places of the lists, and none fills the GPU: in launches of their own the five kernels of one question on
// 3.4M triples took 60 us, those of 200 questions with whitelists 195.
template <int W, bool MASK>
__global__ void __launch_bounds__(256) k_fetch_narrow(FillArgs a, unsigned hub_blocks, unsigned mid_blocks, long long n_mid) {
    if (blockIdx.x < hub_blocks) narrow_hub_segment<W, MASK>(a, blockIdx.x / (unsigned)a.k, (int)(blockIdx.x % (unsigned)a.k) + 1);
    else if (blockIdx.x < hub_blocks + mid_blocks) narrow_wave_rows<W, W, MASK, false, false>(a, blockIdx.x - hub_blocks, a.n_hub_rows, n_mid);
    else narrow_tiles<W, MASK, false>(a, blockIdx.x - hub_blocks - mid_blocks, gridDim.x - hub_blocks - mid_blocks);
}

// The split rows' predecessors: a block per row.
template <int W>
__global__ void __launch_bounds__(256) k_split_lists(FillArgs a) {
    constexpr int Qp = 64 * W;
    __shared__ long long slot[Qp];
    __shared__ int best[Qp];
    const int ev = a.rows[blockIdx.x], t = threadIdx.x, q = t % Qp, w = q >> 6;
    const unsigned long long x = a.visited[(size_t)ev * W + w] & ~a.levels[(size_t)ev * W + w] & range_bits(a.q0, a.q1, w);
    const bool on = (x >> (q & 63)) & 1ull;  // (seeds have their -1 from the tiles)
    if (t < Qp) best[t] = INT_MAX;
    row_slots<W>(a, ev, t >> 6, 4, slot);
    __syncthreads();
    const uint32_t s0 = a.hub_seg_first[blockIdx.x], s1 = a.hub_seg_first[blockIdx.x + 1];
    int m = INT_MAX;
    if (on)
#pragma unroll 8
        for (uint32_t s = s0 + t / Qp; s < s1; s += 256 / Qp) m = min(m, a.seg_pred[(size_t)s * Qp + q]);
    if (m != INT_MAX) atomicMin(&best[q], m);
    __syncthreads();
    if (t < Qp && on) a.pred[slot[q]] = best[q];
}

// 16-word planes without the bit-sliced pass (k > 6, or no room for its buffer).
// One block per tile of 64 entities.  Phase 1: per query of the fetched range, the
// mask of tile entities it reached (for ranks) and the list position of the
// tile's run; seeds get -1.  Phase 2: every entity whose object row has at most
// 32 entries is walked by one W-lane group, two candidate lines in flight.
// Longer rows are left to k_pred_row.
template <bool MASK, bool STATS>
__global__ void __launch_bounds__(1024) k_pred(FillArgs a) {
    constexpr int W = 16, Qp = 64 * W;
    __shared__ unsigned long long stage[64][W + 1];
    __shared__ unsigned long long mT[Qp];
    __shared__ long long base[Qp];
    const long long tile_rel = xcd_contiguous(blockIdx.x, gridDim.x);
    if (tile_rel >= a.tile_count) return;
    const long long tile = a.tile_begin + tile_rel;
    const int t = threadIdx.x, wave = t >> 6, v = lane(), lw = t & (W - 1);
    {
        int q = t;
        long long b = 0;
        if (q >= a.q0 && q < a.q1)
            b = super_start(a, tile / kSuperTiles, Qp, q) + a.tile_base[(size_t)tile * Qp + q];
        base[q] = b;
    }
    const unsigned long long range_w = range_bits(a.q0, a.q1, wave);
    unsigned long long visw = stage_word<W>(stage, a.visited, a.tile_ent, tile, a.E, wave) & range_w;
    unsigned long long seedw = stage_word<W>(stage, a.levels, a.tile_ent, tile, a.E, wave) & range_w;
    unsigned long long mine = 0;
    if (wave_any(visw != 0)) mine = transpose64(visw);  // lane qq: mask of tile entities query qq reached
    mT[t] = mine;
    __syncthreads();
    auto slot = [&](int q, unsigned long long below) -> long long {
        return base[q] + __popcll(mT[q] & below);
    };
    {   // seeds have no predecessor
        const unsigned long long below_v = (1ull << v) - 1ull;
        for (unsigned long long m = seedw; m; m &= m - 1)
            a.pred[slot(wave * 64 + (__ffsll((long long)m) - 1), below_v)] = -1;
    }
    const int vi = t / W, g0 = v & ~(W - 1);
    const long long ev = tile_entity(a.tile_ent, tile, vi, a.E);
    uint32_t lo = 0, hi = 0;
    if (ev >= 0) {
        lo = a.in_off[ev];
        hi = a.in_off[ev + 1];
    }
    const bool longrow = hi - lo > (uint32_t)kTailMaxDegree;
    const unsigned long long below = (1ull << vi) - 1ull;
    long long n_rows = 0, n_edges = 0, n_lines = 0;
    if (hi > lo && !longrow)
        for (int h = 1; h <= a.k; ++h) {
            unsigned long long rem =
                a.levels[(size_t)h * a.plane + (size_t)ev * W + lw] & range_bits(a.q0, a.q1, lw);
            if (!group_any<W>(rem != 0)) continue;
            const uint32_t *act_prev = a.act + (size_t)(h - 1) * a.actw;
            const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
            if (lw == 0) ++n_rows;
            for (uint32_t j0 = lo; j0 < hi; j0 += W) {
                uint32_t j = j0 + lw;
                int s = 0;
                bool cand = false;
                if (j < hi) {
                    s = a.in_sub[j];
                    cand = (act_prev[s >> 5] >> (s & 31)) & 1u;
                }
                unsigned gm = (unsigned)((__ballot(cand) >> g0) & ((1ull << W) - 1ull));
                if (lw == 0) {
                    n_edges += min((uint32_t)W, hi - j0);
                    n_lines += __popc(gm);
                }
                while (gm) {  // two candidate lines in flight, resolved in edge order
                    int c0 = __ffs((int)gm) - 1;
                    gm &= gm - 1;
                    int c1 = -1;
                    if (gm) {
                        c1 = __ffs((int)gm) - 1;
                        gm &= gm - 1;
                    }
                    int s0 = __shfl(s, g0 + c0), s1 = __shfl(s, g0 + (c1 < 0 ? c0 : c1));
                    unsigned long long l0 = prev[(size_t)s0 * W + lw], l1 = 0;
                    if (c1 >= 0) l1 = prev[(size_t)s1 * W + lw];
                    if (MASK) {
                        l0 &= a.allow[(size_t)a.in_rel[j0 + c0] * W + lw];
                        if (c1 >= 0) l1 &= a.allow[(size_t)a.in_rel[j0 + c1] * W + lw];
                    }
                    unsigned long long hit0 = l0 & rem, hit1 = l1 & rem & ~l0;
                    rem &= ~(l0 | l1);
                    if (hit0) {
                        int eid = a.in_eid[j0 + c0];
                        for (unsigned long long m = hit0; m; m &= m - 1)
                            a.pred[slot(lw * 64 + (__ffsll((long long)m) - 1), below)] = eid;
                    }
                    if (hit1) {
                        int eid = a.in_eid[j0 + c1];
                        for (unsigned long long m = hit1; m; m &= m - 1)
                            a.pred[slot(lw * 64 + (__ffsll((long long)m) - 1), below)] = eid;
                    }
                    if (!group_any<W>(rem != 0)) break;
                }
                if (!group_any<W>(rem != 0)) break;
            }
        }
    if (STATS) {
        n_rows = wave_sum(n_rows);
        n_edges = wave_sum(n_edges);
        n_lines = wave_sum(n_lines);
        if (v == 0) {
            if (n_rows) atomicAdd(&a.stats_pred[0], (unsigned long long)n_rows);
            if (n_edges) atomicAdd(&a.stats_pred[1], (unsigned long long)n_edges);
            if (n_lines) atomicAdd(&a.stats_pred[2], (unsigned long long)n_lines);
        }
    }
}

// Predecessor pass for 16-word planes, bit-sliced, in two kernels.
//
// k_pred_walk: a 16-lane group per entity, lane lw owns word lw of the entity's lines.  The group
// walks the entity's object row (<= 32 entries) in edge-id order with a mask of unresolved
// queries per hop level; a candidate's line resolves the queries in (line & mask), all at once.
// What a (query, entity) pair needs later - its hop number and the position of its predecessor
// in the row - is kept bit-sliced: NB words H[b] hold bit b of (hop + 1) of each of the lane's 64
// queries (so H[0] | H[1] | .. is the visited word) and five words J[b] hold bit b of the row
// position.  A resolving line costs a fixed fifteen instructions for up to 64 pairs, whatever
// the number of set bits.  The planes of every (entity, word) go to a buffer laid out
// [tile][word][entity][plane], which a chunk of tiles fills and the second kernel empties.
//
// k_pred_emit: a block = 16 tiles x one word of the range, a wavefront per tile; lane = entity.  The lane turns its
// planes into one code byte per query, (row position << 3) | (hop + 1), with eight 8 x 8 bit transposes: here and not
// in the walk, which is bound by the instructions it issues (walk of 1,024 queries on 30M triples 753 -> 686 us)
// while this kernel waits for memory.  A wavefront walks the queries of the word that reached the block in a
// scalar loop; per query the lanes pick their code byte, a ballot ranks the reached ones inside the tile's piece of
// the query's run, and the lanes store (entity, hop, predecessor edge) at consecutive list positions: every lane issues
// the same few instructions and a store instruction covers one contiguous piece of a list.  The loop holds
// no load from memory (the edge ids of the reached short rows and the reached long rows' predecessors lie in LDS),
// so nothing in it waits for its own stores.  Rows of more than 32 entries belong to the row
// kernels: such an entity's predecessors come from row_pred, which those kernels fill before
// this one starts (or, without that buffer, the row kernels write them to the lists themselves).
// It waits for memory, short of a copy's rate (4.86 TB/s): a store covers the entities of one tile that one query reached, 55 %
// and 78 % of its lanes in the two calls that follow.  1.32 ms for 516M pairs of 1,024 queries, 5.96 GB by the counters,
// 4.5 TB/s (1.49 ms with a rolled loop and edge ids staged row by row, 1.37 with the loop written out); 2.47 ms for 993M pairs of
// 64 queries on 20M entities, 11.2 GB, 4.5 TB/s (2.47).
constexpr int kSlicedMaxK = 6;     // hop + 1 <= 7 fits three bits

constexpr int kPageEntries = 2;  // entries one lane per entity gathers together (on packed planes 1: 2.4, 2: 2.4, 4: 2.7, 8: 3.3 ms)

// A fetch of a page of a 16-word batch gathers one, two or four words of 128-byte lines, and HBM delivers the
// line.  When the listed entities' lines are past what the infinity cache holds, the page's words of every level
// are packed first, and the gathers run on arrays that it does hold: 20M entities, 64 queries, 160 MB instead of
// 2.5 GB per level - packing 1.3 ms, row walk 4.3 -> 2.4 ms, giant rows 2.0 -> 1.7 ms.  Below that packing costs
// more than it saves where few entities are listed, because it goes over all of them (1.4M listed of 5M, four words: 205
// us against 60 us saved), and with four words also where nearly all are.  Page calls of hub-heavy graphs that list
// 99 % of their entities, us unpacked / packed (one, two, four words):
//     3.0M   1,474 / 1,325   2,007 / 1,909    3,107 / 3,199
//     4.0M   2,002 / 1,779   2,659 / 2,524    4,191 / 4,276
//     4.9M   2,400 / 1,999   3,241 / 2,885    4,953 / 4,838
//     7.9M   3,709 / 3,120   5,115 / 4,757    7,911 / 7,531
//    15.8M   6,876 / 5,814  10,139 / 9,026   14,483 / 13,958
// so the line lies where four words begin to gain.  (A capture packs nothing: see captured().)
constexpr long long kPageLines = 4ll << 20;             // listed entities from which the words are packed: 512 MB of lines
constexpr size_t kPagePlaneBytes = (size_t)4 << 30;     // the packed planes take no more than this

template <int N>
__global__ void __launch_bounds__(256)
k_page_planes(const unsigned long long *__restrict__ levels, long long plane, const uint32_t *__restrict__ act,
              long long actw, long long Epad, int first, unsigned long long *__restrict__ out) {
    const int h = blockIdx.y;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < Epad; e += (long long)gridDim.x * 256) {
        unsigned long long x[N];
#pragma unroll
        for (int w = 0; w < N; ++w) x[w] = 0;
        if ((act[(size_t)h * actw + (e >> 5)] >> (e & 31)) & 1u)  // (the lines of the others are zero)
            load_words<N>(x, levels + (size_t)h * plane + (size_t)e * 16 + first);
        unsigned long long *dst = out + ((size_t)h * Epad + (size_t)e) * N;
        if constexpr (N == 1) {
            dst[0] = x[0];
        } else {
#pragma unroll
            for (int w = 0; w < N; w += 2) *reinterpret_cast<ulonglong2 *>(dst + w) = make_ulonglong2(x[w], x[w + 1]);
        }
    }
}

// From bit planes to one byte per query: plane b = bit b of the code, so byte g of every plane forms an 8 x 8 bit matrix
// (row = plane, column = query 8 g + j) whose transpose holds the codes of those 8 queries.
__device__ __forceinline__ void planes_to_codes(const unsigned long long (&P)[8], uint32_t (&d)[16]) {
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        // byte b of x = byte g of plane b, picked with byte permutes (two planes per permute, then
        // the two pairs): six instructions instead of a shift, a mask and an or per plane and half
        uint32_t src[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) src[b] = g < 4 ? (uint32_t)P[b] : (uint32_t)(P[b] >> 32);
        const uint32_t pick = 0x0c0c0000u | (uint32_t)((4 + (g & 3)) << 8) | (uint32_t)(g & 3);  // [b.byte, a.byte, 0, 0]
        const uint32_t t01 = __builtin_amdgcn_perm(src[1], src[0], pick), t23 = __builtin_amdgcn_perm(src[3], src[2], pick);
        const uint32_t t45 = __builtin_amdgcn_perm(src[5], src[4], pick), t67 = __builtin_amdgcn_perm(src[7], src[6], pick);
        const uint32_t xlo = __builtin_amdgcn_perm(t23, t01, 0x05040100u), xhi = __builtin_amdgcn_perm(t67, t45, 0x05040100u);
        unsigned long long x = ((unsigned long long)xhi << 32) | xlo;
        unsigned long long t;
        t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
        x = x ^ t ^ (t << 7);
        t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
        x = x ^ t ^ (t << 14);
        t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
        x = x ^ t ^ (t << 28);
        d[2 * g] = (uint32_t)x;
        d[2 * g + 1] = (uint32_t)(x >> 32);
    }
}

// Every lane's 64-byte record x to out[8 at ..] (where `on`).  The four lanes of a quad store their records one after the other,
// 16 bytes each, so that a request holds a whole record; every lane its own in four stores were four requests each (row walk of
// 1,024 queries on 30M triples, 0.9 GB of records: 526 us, 419 so).
__device__ __forceinline__ uint32_t quad_get(uint32_t x, int i) {  // lane i of the quad's (i constant)
    return (uint32_t)(i == 0 ? __builtin_amdgcn_mov_dpp((int)x, 0x00, 0xf, 0xf, true) : i == 1 ? __builtin_amdgcn_mov_dpp((int)x, 0x55, 0xf, 0xf, true)
                    : i == 2 ? __builtin_amdgcn_mov_dpp((int)x, 0xAA, 0xf, 0xf, true) : __builtin_amdgcn_mov_dpp((int)x, 0xFF, 0xf, 0xf, true));
}

__device__ __forceinline__ void store_records(unsigned long long *__restrict__ out, size_t at, bool on, const unsigned long long (&rec)[8]) {
    uint32_t x[4][4];  // 16-byte pieces
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            x[i][2 * j] = (uint32_t)rec[2 * i + j];
            x[i][2 * j + 1] = (uint32_t)(rec[2 * i + j] >> 32);
        }
    const bool odd = lane() & 1, high = lane() & 2;
#pragma unroll
    for (int d = 0; d < 4; ++d) {  // piece i of lane q for piece q of lane i
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? x[i][d] : x[i + 1][d]), 0xB1, 0xf, 0xf, true);
            x[i][d] = odd ? got : x[i][d];
            x[i + 1][d] = odd ? x[i + 1][d] : got;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(high ? x[i][d] : x[i + 2][d]), 0x4E, 0xf, 0xf, true);
            x[i][d] = high ? got : x[i][d];
            x[i + 2][d] = high ? x[i + 2][d] : got;
        }
    }
    const uint32_t at_lo = (uint32_t)at, at_hi = (uint32_t)(at >> 32);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const size_t to = ((size_t)quad_get(at_hi, i) << 32) | quad_get(at_lo, i);
        if (quad_get(on, i)) *reinterpret_cast<uint4 *>(out + to * 8 + 2 * (lane() & 3)) = make_uint4(x[i][0], x[i][1], x[i][2], x[i][3]);
    }
}

// G = lanes per entity: 16 (lane = word of the line), 4 for a fetch whose queries sit in four
// aligned words or fewer (lane = word wb + lane % 4), which then walks four times as many entities
// per wavefront, or 1 for a fetch inside one word (lane = entity, word wb).
template <int NB, bool MASK, bool STATS, int G>
__global__ void __launch_bounds__(256)
k_pred_walk(FillArgs a, unsigned long long *__restrict__ codes, unsigned long long *__restrict__ visbuf,
            long long tile0, long long ntile, int w0, int nw, int wb, int sparse) {
    constexpr int W = 16;
    constexpr int EPB = 256 / G;         // entities per block (a divisor of 64: one tile per block)
    constexpr unsigned GMASK = (1u << G) - 1u;
    constexpr int HMAX = (1 << NB) - 2;  // largest hop number the NB bits of (hop + 1) can hold
    const long long grp = xcd_contiguous(blockIdx.x, gridDim.x) * EPB + (threadIdx.x / G);  // entity slot of the chunk
    const long long tile_rel = grp >> 6;
    if (tile_rel >= ntile) return;  // wavefront-uniform: a wavefront's entities belong to one tile
    const int vi = (int)(grp & 63), lw = wb + (threadIdx.x & (G - 1)), v = lane(), g0 = v & ~(G - 1);
    const int gl = threadIdx.x & (G - 1);  // the lane's place in its group
    const long long ev = tile_entity(a.tile_ent, tile0 + tile_rel, vi, a.E);
    const unsigned long long range_w = range_bits(a.q0, a.q1, lw);
    unsigned long long visw = 0, lv0 = 0;
    uint32_t lo = 0, hi = 0;
    // word lw of an entity in a level plane
    auto level_word = [&](int h, long long e) -> unsigned long long {
        if constexpr (G <= 4) return a.plv[(size_t)h * a.pplane + (size_t)e * a.pstride + (lw - a.pfirst)];
        else return a.levels[(size_t)h * a.plane + (size_t)e * W + lw];
    };
    if (ev >= 0) {
        lv0 = level_word(0, ev) & range_w;
        if (a.visited && (G > 4 || a.pstride == W)) visw = a.visited[(size_t)ev * W + lw] & range_w;
        else visw = ~0ull & range_w;  // (the level words below decide)
        lo = a.in_off[ev];
        hi = a.in_off[ev + 1];
    }
    const uint32_t deg = hi - lo;
    const bool shortrow = deg > 0 && deg <= (uint32_t)kTailMaxDegree;
    // G = 16: the first 16 entries of the row, for every hop, with their relations (loads of a hop and of a candidate before:
    // 30M triples 688 -> 669 us, with whitelists 758 -> 674; four candidate lines in flight instead of two: 691 and 778)
    int s_row = 0, r_row = 0;
    if (G > 4 && shortrow && gl < (int)deg) {
        s_row = a.in_sub[lo + gl];
        if (MASK) r_row = a.in_rel[lo + gl];
    }
    unsigned long long H[NB], J[5];
    H[0] = lv0;  // hop 0: hop + 1 = 1
#pragma unroll
    for (int b = 1; b < NB; ++b) H[b] = 0;
#pragma unroll
    for (int b = 0; b < 5; ++b) J[b] = 0;
    long long n_rows = 0, n_edges = 0, n_lines = 0;
    if (group_any<G>((visw & ~lv0) != 0)) {  // some query of the range reached the entity by an edge
        // the level words of the first hops are requested together
        constexpr int PRE = HMAX < 3 ? HMAX : 3;
        unsigned long long pre[PRE];
#pragma unroll
        for (int h = 1; h <= PRE; ++h)
            pre[h - 1] = h <= a.k ? level_word(h, ev) & range_w : 0ull;
#pragma unroll
        for (int h = 1; h <= HMAX; ++h) {
            if (h > a.k) break;
            unsigned long long rem;
            if (h <= PRE) rem = pre[h - 1];
            else rem = level_word(h, ev) & range_w;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (((h + 1) >> b) & 1) H[b] |= rem;
            if (!shortrow || !group_any<G>(rem != 0)) continue;
            const uint32_t *act_prev = a.act + (size_t)(h - 1) * a.actw;
            const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
            const bool dense = !STATS && ((a.dense_levels >> h) & 1u);  // the line of an entity outside the level is zero
            if (STATS && gl == 0) ++n_rows;
            if constexpr (G <= 4) {
                // A page of the batch: eight entries of the row are gathered together (the group's lanes take a word
                // each) and resolved in order.  No frontier bit is asked for first: it costs as much as the piece of a
                // line.  With two and four lanes eight entries (63 queries over two words, 50M triples: 327 us with
                // two at a time, 280 us now).  Under whitelists every entry costs a second gather: two (70 queries of a
                // hub-heavy graph of 20M triples: call 840 us with eight, 796 with four, 781 with two; of 30M triples of
                // concepts 915, 879 and 882).  A lane per entity takes kPageEntries as well, because what it gathers past the
                // entry that resolves the last query is lost and its rate is that of the scattered sectors.
                constexpr int U = G == 1 || MASK ? kPageEntries : 8;
                for (int i0 = 0; i0 < (int)deg; i0 += U) {  // (i0 is the same in all lanes that are still in the loop)
                    int sx[U], rx[U];
                    unsigned long long l[U], ok[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool in = i0 + u < (int)deg;
                        sx[u] = in ? a.in_sub[lo + i0 + u] : -1;
                        rx[u] = MASK && in ? a.in_rel[lo + i0 + u] : 0;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        l[u] = sx[u] >= 0 ? level_word(h - 1, sx[u]) : 0ull;
                        ok[u] = MASK && sx[u] >= 0 ? a.allow[(size_t)rx[u] * W + lw] : 0ull;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (MASK) l[u] &= ok[u];
                        const unsigned long long hit = l[u] & rem;
                        rem &= ~l[u];
                        const int at = i0 + u;
#pragma unroll
                        for (int b = 0; b < 5; ++b)
                            if ((at >> b) & 1) J[b] |= hit;
                    }
                    if (STATS && gl == 0) {
                        n_edges += min(U, (int)deg - i0);
                        n_lines += min(U, (int)deg - i0);
                    }
                    if (!group_any<G>(rem != 0)) break;
                }
                continue;
            }
            // The four groups go through their rows' positions in step, four at a time, so that a position's bits are the same in
            // all lanes: a resolving line costs ten instructions (some forty where every group took its own next candidate).
            for (int half = 0; half < kTailMaxDegree; half += G) {
                int s = s_row, r = r_row;
                bool cand = group_any<G>(rem != 0) && half + gl < (int)deg;
                if (cand) {
                    if (half > 0) {
                        s = a.in_sub[lo + half + gl];
                        if (MASK) r = a.in_rel[lo + half + gl];
                    }
                    cand = dense || ((act_prev[s >> 5] >> (s & 31)) & 1u);
                }
                const unsigned long long all = __ballot(cand);
                if (all == 0) continue;  // (wavefront-uniform among the lanes of the level)
                unsigned mine = (unsigned)(all >> g0) & GMASK;
                const unsigned any = (unsigned)(all | (all >> 16) | (all >> 32) | (all >> 48)) & GMASK;
                if (STATS && gl == 0) {
                    n_edges += max(0, min(G, (int)deg - half));
                    n_lines += __popc(mine);
                }
#pragma unroll
                for (int i0 = 0; i0 < G; i0 += 4) {
                    if (!((any >> i0) & 15u)) continue;
                    unsigned long long l[4], ok[4];
                    int sx[4], rx[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        sx[u] = __shfl(s, g0 + i0 + u);
                        rx[u] = MASK ? __shfl(r, g0 + i0 + u) : 0;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        l[u] = ok[u] = 0;
                        if ((mine >> (i0 + u)) & 1u) {
                            l[u] = prev[(size_t)sx[u] * W + lw];
                            if (MASK) ok[u] = a.allow[(size_t)rx[u] * W + lw];
                        }
                    }
                    unsigned long long found = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (MASK) l[u] &= ok[u];
                        const unsigned long long hit = l[u] & rem;
                        rem &= ~l[u];
                        found |= hit;
                        if (u & 1) J[0] |= hit;
                        if (u & 2) J[1] |= hit;
                    }
                    if (i0 & 4) J[2] |= found;
                    if (i0 & 8) J[3] |= found;
                    if (half) J[4] |= found;
                    if (!group_any<G>(rem != 0)) mine = 0;
                }
            }
        }
    }
    // plane b = bit b of the code: NB bits of (hop + 1) below five bits of the row position, which always starts at
    // bit 3.  k_pred_emit reads the planes as they are, k_emit_sparse one byte per query, and only of words that
    // hold something.
    const bool in_range = lw >= w0 && lw < w0 + nw;
    const size_t at = ((size_t)tile_rel * nw + (in_range ? lw - w0 : 0)) * 64 + vi;
    unsigned long long P[8], reached = 0;  // reached: the queries of the word that reached the entity
#pragma unroll
    for (int b = 0; b < 8; ++b) P[b] = b < NB ? H[b] : b < 3 ? 0ull : J[b - 3];
    if (sparse) {
#pragma unroll
        for (int b = 0; b < NB; ++b) reached |= H[b];
        if (in_range) visbuf[at] = reached;
        if (wave_any(in_range && reached != 0)) {
            uint32_t d[16];
            planes_to_codes(P, d);
#pragma unroll
            for (int b = 0; b < 8; ++b) P[b] = ((unsigned long long)d[2 * b + 1] << 32) | d[2 * b];
        }
    }
    store_records(codes, at, in_range && (!sparse || reached != 0), P);
    if (STATS) {
        n_rows = wave_sum(n_rows);
        n_edges = wave_sum(n_edges);
        n_lines = wave_sum(n_lines);
        if (v == 0) {
            if (n_rows) atomicAdd(&a.stats_pred[0], (unsigned long long)n_rows);
            if (n_edges) atomicAdd(&a.stats_pred[1], (unsigned long long)n_edges);
            if (n_lines) atomicAdd(&a.stats_pred[2], (unsigned long long)n_lines);
        }
    }
}

// A block = 16 consecutive tiles (one wavefront each) x one word of the fetched range.
// 8 wavefronts per SIMD = at most 64 vector registers.
constexpr int kEmitTiles = 16;
constexpr int kEmitPool = 19'456;  // LDS words, two blocks per CU: edge ids of the short rows of the block's 1,024 entities,
                                   // behind them the row_pred values (64 queries each) of those with longer rows
constexpr int kEmitLines = kEmitPool / 64;

// STAGED: the edge ids of the block's short rows are in LDS; LINES: the values of its row_pred entities
// are.  Otherwise the loop reads the edge ids from memory / a pass of its own moves the
// row_pred values with lanes = queries.
template <bool STAGED, bool LINES>
__device__ __forceinline__ void emit_word(const FillArgs &a, const uint32_t (&c)[16], unsigned long long live,
                                          uint32_t pos_lo, uint32_t pos_hi, int ent_id, bool longrow, bool by_query,
                                          const int *my_eids, const int32_t *my_row, const int *my_line) {
    const uint32_t live_lo = __builtin_amdgcn_readfirstlane((uint32_t)live);
    const uint32_t live_hi = __builtin_amdgcn_readfirstlane((uint32_t)(live >> 32));
    // unrolled over the sixteen code registers (four queries each): a query's byte is picked with
    // one bit-field extract
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        uint32_t rest = ((r < 8 ? live_lo : live_hi) >> (4 * (r & 7))) & 15u;
        while (rest) {  // scalar loop over the queries 4 r .. 4 r + 3 that reached the block's tiles
            const int j = __builtin_ctz(rest);
            rest &= rest - 1;
            const int qq = 4 * r + j;
            const uint32_t code = __builtin_amdgcn_ubfe(c[r], (unsigned)(8 * j), 8u);
            const uint32_t hc = code & 7u, jp = code >> 3;
            const bool bit = hc != 0u;
            const unsigned long long m = __ballot(bit);
            if (bit) {
                const unsigned rank =
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                const unsigned long long base =
                    ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)pos_hi, qq) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)pos_lo, qq);
                int32_t *const pe = a.entity + base;
                pe[rank] = ent_id;
                if (a.hop) {
                    uint8_t *const ph8 = a.hop + base;
                    ph8[rank] = (uint8_t)(hc - 1u);
                }
                const bool seed = hc == 1u;
                if (!longrow || seed || (LINES && by_query)) {
                    int val = -1;
                    if (!seed) {
                        if constexpr (LINES) {
                            if constexpr (STAGED) val = by_query ? my_line[qq] : my_eids[jp];
                            else val = by_query ? my_line[qq] : my_row[jp];
                        } else {
                            if constexpr (STAGED) val = my_eids[jp];
                            else val = my_row[jp];
                        }
                    }
                    int32_t *const pp = a.pred + base;
                    pp[rank] = val;
                }
            }
            __builtin_amdgcn_s_barrier();  // the sixteen tiles write their pieces of a query together
        }
    }
}

// The code byte of query qq, and its predecessor where all of them lie in the pool (`at`: the lane's byte offset there; stride:
// 4 for a row_pred line, which has an entry per query, 0 for edge ids, by row position, which is 0 for long rows).  seeds: the
// queries with a seed in this tile, hardly ever any.
struct Emitted {
    uint32_t hc;  // hop + 1
    int val;
};

__device__ __forceinline__ bool bit_of(unsigned long long x, int qq) { return ((qq < 32 ? (uint32_t)x : (uint32_t)(x >> 32)) >> (qq & 31)) & 1u; }

__device__ __forceinline__ Emitted emit_pooled(uint32_t c, int qq, unsigned long long seeds, const int *pool, uint32_t at, uint32_t stride) {
    const uint32_t hc = __builtin_amdgcn_ubfe(c, (unsigned)(8 * (qq & 3)), 3u), jp = __builtin_amdgcn_ubfe(c, (unsigned)(8 * (qq & 3) + 3), 5u);
    int val = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(pool) + (at + (uint32_t)qq * stride + 4u * jp));
    if (bit_of(seeds, qq)) val = hc == 1u ? -1 : val;
    return Emitted{hc, val};
}

__device__ __forceinline__ uint32_t rank_in(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// All predecessors in the pool, hop numbers asked for: what nearly every block does.  The 64 queries are written out (36
// vector and 33 scalar instructions per tile and query with the general form, 30 and 27 so), and the tiles keep together
// by a barrier per eight queries: 516M pairs 1,490 us with the general form, 1,425 with a barrier per query, 1,373 so.
// (The tiles' pieces put together in LDS and stored as whole aligned groups: 1,514.)
__device__ __forceinline__ void emit_word_pooled(const FillArgs &a, const uint32_t (&c)[16], unsigned long long live, unsigned long long seeds,
                                                 uint32_t pos_lo, uint32_t pos_hi, int ent_id, const int *pool, uint32_t at, uint32_t stride) {
    live = uniform64(live);
#pragma unroll
    for (int qq = 0; qq < 64; ++qq) {
        if (bit_of(live, qq)) {
            const Emitted e = emit_pooled(c[qq >> 2], qq, seeds, pool, at, stride);
            const unsigned long long m = __ballot(e.hc != 0u);
            const unsigned long long base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)pos_hi, qq) << 32) |
                                            (uint32_t)__builtin_amdgcn_readlane((int)pos_lo, qq);
            if (e.hc != 0u) {
                const uint32_t rank = rank_in(m);
                int32_t *const pe = a.entity + base;
                uint8_t *const ph = a.hop + base;
                int32_t *const pp = a.pred + base;
                pe[rank] = ent_id;
                ph[rank] = (uint8_t)(e.hc - 1u);
                pp[rank] = e.val;
            }
        }
        if ((qq & 7) == 7) __builtin_amdgcn_s_barrier();
    }
}

// inclusive maximum over the lanes up to each one (values of at least 0)
__device__ __forceinline__ int wave_max_scan(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));  // row_shr 1, 2, 4, 8: within sixteen lanes
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // the last lane of rows 0 and 2 to rows 1 and 3
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));  // lane 31 to the upper half
    return x;
}

__global__ void __launch_bounds__(kEmitTiles * 64) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_pred_emit(FillArgs a, const unsigned long long *__restrict__ planes, long long tile0, long long ntile, int w0, int nw,
            int eid_cap, int line_cap) {
    constexpr int Qp = 1024, TPB = kEmitTiles;
    __shared__ int pool[kEmitPool];
    __shared__ unsigned long long s_live;
    __shared__ int s_need[TPB];
    const long long L = xcd_contiguous(blockIdx.x, gridDim.x);
    const long long nsup = (ntile + TPB - 1) / TPB;
    if (L >= nsup * nw) return;  // block-uniform
    const int wi = (int)(L % nw), w = w0 + wi;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), v = lane(), ql = w * 64 + v;
    const bool valid = (L / nw) * TPB + wave < ntile;  // (behind the last tile: its loads again, nothing written)
    const long long tile_rel = min((L / nw) * TPB + wave, ntile - 1), tile = tile0 + tile_rel;
    if (t == 0) s_live = 0ull;
    // What depends on nothing is requested first: the tile's entities, the planes of (entity, word) (lane = entity; zero
    // where there is no entity), and where query 64 w + v continues in this tile (lane = query)
    const long long ew = tile_entity(a.tile_ent, tile, v, a.E);
    unsigned long long P[8];
    {
        const ulonglong2 *in = reinterpret_cast<const ulonglong2 *>(planes) + (((size_t)tile_rel * nw + wi) * 64 + v) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const ulonglong2 x = in[i];
            P[2 * i] = x.x;
            P[2 * i + 1] = x.y;
        }
    }
    const long long list_q = a.reached_off[ql];
    const uint32_t mega_q = a.mega_base[(size_t)(tile / kSuperTiles / kMegaSupers) * Qp + ql];
    const uint32_t super_q = a.super_base[(size_t)(tile / kSuperTiles) * Qp + ql], tile_q = a.tile_base[(size_t)tile * Qp + ql];
    const size_t eo = ew >= 0 ? (size_t)ew : 0;
    const uint32_t wlo = a.in_off[eo], wdeg = a.in_off[eo + 1] - wlo;
    const unsigned long long vis = valid && ew >= 0 ? P[0] | P[1] | P[2] : 0ull;
    unsigned long long seeds = vis & P[0] & ~(P[1] | P[2]);  // hop + 1 == 1
    seeds = wave_any(seeds != 0) ? uniform64(wave_or64(seeds)) : 0ull;
    // where a lane's predecessors come from: the edge ids of its own short row (by row position),
    // its line of row_pred (by query), or nowhere (the block-per-row kernel writes them).  Seeds
    // get their -1 in the loop.
    const bool longrow = wdeg > (uint32_t)kTailMaxDegree;
    const bool by_query = longrow && a.row_pred && vis != 0;
    int li = 0;
    if (by_query) li = (int)(a.long_index[ew] - a.row_base);
    const int n_stage = longrow || vis == 0 ? 0 : (int)wdeg;
    const unsigned long long below = (1ull << v) - 1ull;
    int off = 0, wtot = 0;  // prefix and sum of n_stage (at most 32) over the wavefront
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const unsigned long long m = __ballot((n_stage >> b) & 1);
        off += __popcll(m & below) << b;
        wtot += __popcll(m) << b;
    }
    const unsigned long long bq_wave = __ballot(by_query);
    if (v == 0) s_need[wave] = wtot | (__popcll(bq_wave) << 16);  // (at most 2,048 and 64)
    const unsigned long long live_wave = wave_or64(vis);
    __syncthreads();
    if (v == 0 && live_wave) atomicOr(&s_live, live_wave);
    const int need = s_need[v & (TPB - 1)];
    int total = 0, lines = 0, line0 = 0;
#pragma unroll
    for (int x = 0; x < TPB; ++x) {
        const int n = __builtin_amdgcn_readlane(need, x);
        if (x < wave) {
            off += n & 0xffff;
            line0 += n >> 16;
        }
        total += n & 0xffff;
        lines += n >> 16;
    }
    const bool staged = total <= eid_cap;  // block-uniform
    int *const eid_tab = pool, *const rp_tab = pool + (staged ? total : 0);
    const bool lined = lines <= line_cap && lines * 64 + (staged ? total : 0) <= kEmitPool;
    if (staged && wtot > 0) {  // wavefront-uniform
        // Lane = entry of the wavefront's rows one behind the other, which lie so in memory as well, but for long rows
        // and entities that were not reached between them.  Every row leaves its lane at its first place, the largest one
        // so far is the row a place belongs to.  (Every lane its own row was a gather of 64 lines per entry of the longest.)
        int *const tab = eid_tab + __builtin_amdgcn_readfirstlane(off);  // (lane 0's prefix: where the wavefront begins)
        const int mine = off - __builtin_amdgcn_readfirstlane(off);
        for (int i = v; i < wtot; i += 64) tab[i] = 0;
        __builtin_amdgcn_wave_barrier();
        if (n_stage > 0) tab[mine] = v + 1;
        __builtin_amdgcn_wave_barrier();
        int before = 0;
        for (int i0 = 0; i0 < wtot; i0 += 256) {
            int e[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int i = i0 + 64 * x + v;
                const int row = max(before, wave_max_scan(i < wtot ? tab[i] : 0));
                before = __builtin_amdgcn_readlane(row, 63);
                e[x] = __shfl((int)wlo - mine, row - 1) + i;
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) e[x] = i0 + 64 * x + v < wtot ? a.in_eid[(uint32_t)e[x]] : 0;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (i0 + 64 * x + v < wtot) tab[i0 + 64 * x + v] = e[x];
        }
    }
    // the row_pred values of this word: 64 queries x the wavefront's entities of that kind, eight
    // lines requested together (lanes = queries)
    if (lined) {
        unsigned long long bq = bq_wave;
        int s_at = line0;
        while (bq) {
            int val[8], at[8], Lx = 0, n = -1;
#pragma unroll
            for (int x = 0; x < 8; ++x) {  // (the last one again where there are fewer)
                if (bq) {
                    Lx = __builtin_ctzll(bq);
                    bq &= bq - 1;
                    ++n;
                }
                at[x] = s_at + n;
                val[x] = a.row_pred[(size_t)__builtin_amdgcn_readlane(li, Lx) * Qp + ql];
            }
#pragma unroll
            for (int x = 0; x < 8; ++x) rp_tab[at[x] * 64 + v] = val[x];
            s_at += n + 1;
        }
    }
    // lane = entity: one code byte per query of the word, (row position << 3) | (hop + 1), zero where
    // the query did not reach the entity
    if (vis == 0) {
#pragma unroll
        for (int b = 0; b < 8; ++b) P[b] = 0;
    }
    uint32_t c[16];
    planes_to_codes(P, c);
    const long long pos = list_q - a.reached_off[a.q0] + mega_q + super_q + tile_q;
    uint32_t pos_lo = (uint32_t)(unsigned long long)pos, pos_hi = (uint32_t)((unsigned long long)pos >> 32);
    __syncthreads();
    const unsigned long long live = s_live;
    if (live == 0ull) return;  // block-uniform
    if (!lined) {
        // Entities whose predecessors wait in row_pred, too many for rp_tab: lanes = queries.
        // Lane i knows where query i's run of this tile starts (pos) and, after a 64 x 64
        // transpose of the visited words, which of the tile's entities query i reached: the
        // rank of entity L in the run is the number of those below L.  Four lines are
        // requested before the first is stored.  Seeds (hop + 1 == 1) are left to the loop.
        unsigned long long bq = bq_wave;
        if (bq) {
            const unsigned long long mT = transpose64(vis);
            unsigned long long seed_w = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    seed_w |= (unsigned long long)(((c[i] >> (8 * j)) & 7u) == 1u) << (4 * i + j);
            const uint32_t seed_lo = (uint32_t)seed_w, seed_hi = (uint32_t)(seed_w >> 32);
            const int32_t *const rp = a.row_pred + ql;
            int32_t *const pp = a.pred + pos;
            while (bq) {
                int Lx[4], val[4];
                bool on[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    Lx[x] = -1;
                    on[x] = false;
                    val[x] = 0;
                    if (bq) {
                        Lx[x] = __builtin_ctzll(bq);
                        bq &= bq - 1;
                        const int liL = __builtin_amdgcn_readlane(li, Lx[x]);
                        const unsigned long long seedL =
                            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)seed_hi, Lx[x]) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)seed_lo, Lx[x]);
                        on[x] = ((mT >> Lx[x]) & 1ull) && !((seedL >> v) & 1ull);
                        if (on[x]) val[x] = rp[(size_t)liL * Qp];
                    }
                }
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (on[x]) pp[__popcll(mT & ((1ull << Lx[x]) - 1ull))] = val[x];
            }
        }
    }
    // Everything requested from memory so far is consumed here, so that the loop holds stores
    // only: a wait on a load inside it would also wait for the loop's own stores.
    asm volatile("" : "+v"(pos_lo), "+v"(pos_hi));
    const int ent_id = (int)ew;
    const int *const my_eids = eid_tab + (staged ? off : 0);
    const int32_t *const my_row = a.in_eid + wlo;
    const int *const my_line = rp_tab + (lined ? line0 + __popcll(bq_wave & below) : 0) * 64;
    if (staged && lined && a.row_pred && a.hop) {  // block-uniform
        // (a lane with neither, whose value is not stored or a seed's, reads the pool's first place: its own may lie behind the end)
        const uint32_t at = by_query ? 4u * (uint32_t)(my_line - pool) : n_stage > 0 ? 4u * (uint32_t)(my_eids - pool) : 0u;
        emit_word_pooled(a, c, live, seeds, pos_lo, pos_hi, ent_id, pool, at, by_query ? 4u : 0u);
    } else if (staged) {
        if (lined) emit_word<true, true>(a, c, live, pos_lo, pos_hi, ent_id, longrow, by_query, my_eids, my_row, my_line);
        else emit_word<true, false>(a, c, live, pos_lo, pos_hi, ent_id, longrow, by_query, my_eids, my_row, my_line);
    } else {
        if (lined) emit_word<false, true>(a, c, live, pos_lo, pos_hi, ent_id, longrow, by_query, my_eids, my_row, my_line);
        else emit_word<false, false>(a, c, live, pos_lo, pos_hi, ent_id, longrow, by_query, my_eids, my_row, my_line);
    }
}

// The lists of a batch whose words are mostly empty (whitelists, early hops): a wavefront per word of a tile, lane = entity,
// nothing shared between the wavefronts.  k_pred_emit goes through all queries of a word for all of a block's 1,024
// entities, whoever reached what, and reads every code byte; here a lane takes the set bits of its own word one after the
// other (where a query reached eight and more of the tile's entities, the wavefront takes the query), four at a time so
// that their codes, and then their triple indices, are requested together.  It is bound by these chains and by the
// scattered pieces of the lists it writes, which is why it loses to k_pred_emit where words are full.
// Fetches of 1,024 queries with whitelists on 30M triples, whole fetch, us k_pred_emit / k_emit_sparse, by the share of (listed
// entity, query) pairs that are reached: 0.4 % 1,211 / 1,051, 0.8 % 1,463 / 1,301, 1.2 % 1,686 / 1,540, 1.4 % 2,064 / 1,974,
// 2.4 % 2,013 / 2,009, 4.2 % 2,264 / 2,458, 4.6 % 2,275 / 2,434, 7.2 % 2,253 / 2,619, 11 % 2,437 / 3,069; two hops 0.5 %
// 1,012 / 877, 1.1 % 1,252 / 1,198, 5.6 % 2,109 / 2,471; pages of 128 queries 2.7 % 757 / 751, 8.4 % 842 / 887: the line lies at
// 2.5 % (at 5 % before k_pred_emit's loop was written out).
constexpr int kSparseShare = 40;   // reached pairs: at most one in this many
constexpr int kHeavyEntities = 8;  // (4 and 16: within 2 %)

__global__ void __launch_bounds__(256)
k_emit_sparse(FillArgs a, const uint8_t *__restrict__ codes, const unsigned long long *__restrict__ visbuf, long long tile0,
              long long ntile, int w0, int nw) {
    constexpr int Qp = 1024, U = 4;
    __shared__ unsigned long long mT[4][64];  // entities of the tile each query reached
    __shared__ long long base[4][64];         // where its run of the tile starts in the lists
    const int wave = threadIdx.x >> 6, v = lane();
    const long long item = xcd_contiguous(blockIdx.x, gridDim.x) * 4 + wave;  // neighbouring tiles of a word together
    if (item >= ntile * nw) return;  // wavefront-uniform
    const long long tile_rel = item % ntile, tile = tile0 + tile_rel;
    const int wi = (int)(item / ntile), w = w0 + wi;
    const size_t at = ((size_t)tile_rel * nw + wi) * 64 + v;
    const int ql = w * 64 + v;
    // requested together: the reached pairs, the tile's entities (lane = entity), where a query's run starts (lane = query)
    // (one behind the other: 1,000 queries with whitelists 534 us, 523 now; over two hops 117 and 106)
    const unsigned long long vis = visbuf[at];
    const int32_t ev = (int32_t)tile_entity(a.tile_ent, tile, v, a.E);
    const long long run = super_start(a, tile / kSuperTiles, Qp, ql) + a.tile_base[(size_t)tile * Qp + ql];
    const size_t eo = ev >= 0 ? (size_t)ev : 0;
    const uint32_t lo = a.in_off[eo], hi = a.in_off[eo + 1];
    if (!wave_any(vis != 0)) return;
    const unsigned long long reached = transpose64(vis);
    base[wave][v] = run;
    mT[wave][v] = reached;
    __builtin_amdgcn_wave_barrier();
    const bool longrow = hi - lo > (uint32_t)kTailMaxDegree;
    // a lane's predecessors: by place in its short row, or by query in its line of row_pred, or written by the row kernels
    const int32_t *from = a.in_eid + lo;
    if (longrow) from = a.row_pred && vis ? a.row_pred + (size_t)(a.long_index[ev] - a.row_base) * Qp + w * 64 : nullptr;
    const unsigned long long below = (1ull << v) - 1ull;
    const uint8_t *my_codes = codes + at * 64;
    auto put = [&](const int (&qq)[U]) {  // (-1: nothing)
        uint32_t code[U];
        int32_t val[U];
#pragma unroll
        for (int u = 0; u < U; ++u) code[u] = qq[u] >= 0 ? my_codes[qq[u]] : 1u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            val[u] = -1;  // seeds
            if ((code[u] & 7u) > 1u && from) val[u] = from[longrow ? qq[u] : (int)(code[u] >> 3)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (qq[u] < 0) continue;
            const long long p = base[wave][qq[u]] + __popcll(mT[wave][qq[u]] & below);
            a.entity[p] = ev;
            if (a.hop) a.hop[p] = (uint8_t)((code[u] & 7u) - 1u);
            if (from || (code[u] & 7u) == 1u) a.pred[p] = val[u];
        }
    };
    // queries that reached many of the tile's entities: a lane per entity; the others: every lane its own
    const unsigned long long heavy = __ballot(__popcll(reached) >= kHeavyEntities);
    for (unsigned long long m = heavy; m;) {
        int qq[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = m ? __ffsll((long long)m) - 1 : -1;
            m &= m - 1;
            qq[u] = q >= 0 && ((vis >> (q & 63)) & 1ull) ? q : -1;
        }
        put(qq);
    }
    for (unsigned long long left = vis & ~heavy; left;) {
        int qq[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            qq[u] = left ? __ffsll((long long)left) - 1 : -1;
            left &= left - 1;
        }
        put(qq);
    }
}

// Object rows of more than 32 entries: one block per row (4 waves; 16 for hub
// rows).  Phase 1 rebuilds the list positions of the row's entity (ranks inside
// its tile).  Phase 2 walks the row in steps of (waves x 4 x 64) entries: inside a
// step the waves take disjoint 64-entry chunks (interleaved, so that a row
// shorter than a step still occupies every wave) and keep, per query, the smallest
// edge id any of them found (LDS atomicMin); after the step the resolved queries
// are removed from the shared mask, so a later step (larger edge ids) never
// touches them.  Each predecessor is then written once.
// SEG (row-buffer mode only): a block per kGiantSegment entries of a giant row instead of one per
// row; the blocks of a row keep the smallest edge id per query in the row's line of the row buffer
// (atomicMin; the line starts at INT_MAX).  A block that walks a whole 140,000-entry row is a chain
// of dependent gathers that outlasts everything else in the launch; the segments of a row run side
// by side, at the price of the early exit between them (it saved a quarter of the entries).
// Under whitelists: where at most kFilterQueries queries are left, entries whose relation none of them may follow are left out
// before their lines are asked for.  us of a fetch of 1,000 queries by that number (0: never); the relations' bits are what a
// block has LDS for beside its queues (half a KB):
//    30M triples        k = 2   0:   710    4:   712    12:   714    24:   730    48:   757    128:   784
//                       k = 3   0: 2,027    4: 1,943    12: 1,944    24: 1,959    48: 1,982    128: 2,029
//    hub-heavy 20M      k = 3   0: 3,302    4: 3,260    12: 3,231    24: 3,226    48: 3,232    128: 3,244
//    3.4M               k = 3   0:   391    4:   373    12:   363    24:   361    48:   365    128:   371
constexpr int kFilterQueries = 12, kFilterRelations = 4096;

template <bool MASK, bool STATS, bool BUF, bool SEG = false>
__global__ void __launch_bounds__(1024) k_pred_row(FillArgs a, long long first_row) {
    static_assert(!SEG || BUF, "segments merge in the row buffer");
    constexpr int W = 16, Qp = 64 * W;
    constexpr int C = 4;  // 64-entry chunks per wavefront and step, loaded together
    __shared__ long long slot[BUF ? 1 : Qp];
    __shared__ unsigned int smin[W * kClaimStride];  // smallest entry per query (index into in_sub)
    __shared__ PredQueue queue[16];
    __shared__ unsigned long long srem[W], slevel[W];
    __shared__ unsigned long long usable[MASK ? kFilterRelations / 64 : 1];  // relations that a query that is left may follow
    long long row_i = blockIdx.x;
    uint32_t seg = 0;
    if (SEG) giant_segment(a, blockIdx.x, row_i, seg);
    const int ev = a.rows[first_row + row_i];
    const int t = threadIdx.x, wave = t >> 6, nw = blockDim.x >> 6, v = lane(), lw = v & (W - 1);
    // gridDim.y > 1: one block per (row, hop level), so the levels of a long row run side by side
    const int h_first = gridDim.y > 1 ? (int)blockIdx.y + 1 : 1, h_last = gridDim.y > 1 ? h_first : a.k;
    if (gridDim.y > 1) {  // nothing of this level in the row's entity: leave before the list positions
        const unsigned long long x = a.levels[(size_t)h_first * a.plane + (size_t)ev * W + lw] & range_bits(a.q0, a.q1, lw);
        if (!wave_any(x != 0) || ((a.push_levels >> h_first) & 1u)) return;  // the same words in every wavefront
    }
    if (!BUF) row_slots<W>(a, ev, wave, nw, slot);
    int32_t *out = BUF ? a.row_pred + (size_t)(first_row + row_i) * Qp : a.pred;
    const uint32_t row_lo = a.in_off[ev], row_hi = a.in_off[ev + 1];
    const uint32_t lo = SEG ? row_lo + seg * (uint32_t)kGiantSegment : row_lo;
    const uint32_t hi = SEG ? min(row_hi, lo + (uint32_t)kGiantSegment) : row_hi;
    long long n_rows = 0, n_edges = 0, n_lines = 0;
    for (int h = h_first; h <= h_last; ++h) {
        __syncthreads();
        if (t < W) {
            const unsigned long long x = a.levels[(size_t)h * a.plane + (size_t)ev * W + t] & range_bits(a.q0, a.q1, t);
            srem[t] = x;
            slevel[t] = x;
        }
        for (int q = t; q < Qp; q += blockDim.x) smin[(q >> 6) * kClaimStride + (q & 63)] = ~0u;
        __syncthreads();
        if (!wave_any(slevel[lw] != 0) || ((a.push_levels >> h) & 1u)) continue;  // block-uniform
        if (SEG && seg > 0) {  // (sixteen wavefronts: one per word)
            const unsigned long long done = resolved_before(&out[t], a.in_eid[lo]);
            if (v == 0) srem[wave] &= ~done;
            __syncthreads();
        }
        const uint32_t *act_prev = a.act + (size_t)(h - 1) * a.actw;
        const unsigned long long *prev = a.levels + (size_t)(h - 1) * a.plane;
        const bool dense = !STATS && ((a.dense_levels >> h) & 1u);  // the line of an entity outside the level is zero
        if (wave == 0) ++n_rows;
        // The first step is short (one chunk per wavefront): on a dense frontier the first
        // candidates of a row resolve most queries, and what is resolved after that step is not
        // claimed again by sixteen wavefronts in parallel.
        uint32_t span = 64u * nw;
        for (uint32_t s0 = lo; s0 < hi; s0 += span, span = 64u * C * nw) {
            const uint32_t step_hi = min(hi, s0 + span);
            unsigned long long rem = srem[lw];
            if (!wave_any(rem != 0)) break;  // same decision in every wave
            const unsigned long long before = rem;
            bool by_relation = false;  // block-uniform
            if constexpr (MASK) {
                int left = v < W ? __popcll(rem) : 0;
#pragma unroll
                for (int m = W / 2; m >= 1; m >>= 1) left += __shfl_xor(left, m);
                by_relation = a.R <= kFilterRelations && __builtin_amdgcn_readfirstlane(left) <= kFilterQueries;
                if (by_relation) {
                    for (int r0 = 64 * wave; r0 < a.R; r0 += 64 * nw) {  // lane = relation
                        const int r = min(r0 + v, a.R - 1);
                        unsigned long long any = 0;
#pragma unroll
                        for (int w = 0; w < W; w += 2) {
                            const ulonglong2 x = *reinterpret_cast<const ulonglong2 *>(a.allow + (size_t)r * W + w);
                            any |= (x.x & srem[w]) | (x.y & srem[w + 1]);
                        }
                        const unsigned long long bits = __ballot(any != 0);
                        if (v == 0) usable[r0 / 64] = bits;
                    }
                    __syncthreads();
                }
            }
            // chunk c of this wavefront is chunk c * nw + wave of the step: a row shorter than a
            // step still spreads over all wavefronts
            const uint32_t w0 = s0 + 64u * wave;
            int sj[C], rj[C];
            bool cj[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {  // all loads of the step first
                const uint32_t j = w0 + 64u * nw * c + v;
                cj[c] = j < step_hi;
                const uint32_t at = cj[c] ? j : s0;  // (no branch, which the next chunk's loads would wait behind)
                sj[c] = a.in_sub[at];
                rj[c] = MASK ? a.in_rel[at] : 0;
            }
            if (MASK && by_relation) {
#pragma unroll
                for (int c = 0; c < C; ++c) cj[c] = cj[c] && ((usable[rj[c] >> 6] >> (rj[c] & 63)) & 1u);
            }
            if (!dense) {
                uint32_t bits[C];
#pragma unroll
                for (int c = 0; c < C; ++c) bits[c] = act_prev[sj[c] >> 5] >> (sj[c] & 31);
#pragma unroll
                for (int c = 0; c < C; ++c) cj[c] = cj[c] && (bits[c] & 1u);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                uint32_t j0 = w0 + 64u * nw * c;
                if (j0 < step_hi && wave_any(rem != 0)) {
                    n_lines += pred_resolve_unordered<MASK>(sj[c], rj[c], cj[c], a, prev, queue[wave], rem,
                                                               [&](unsigned long long hit, int at) {
                        claim(&smin[lw * kClaimStride], hit, j0 + (uint32_t)at);
                    });
                    n_edges += min((uint32_t)64, step_hi - j0);
                }
            }
            unsigned long long resolved = before & ~rem;  // by this group of lanes
            __syncthreads();
            if (resolved) atomicAnd(&srem[lw], ~resolved);
            __syncthreads();
        }
        __syncthreads();
        for (int q1 = t; q1 < Qp; q1 += 4 * blockDim.x) {  // four triple indices are requested before the first is stored
            int32_t eid[4];
            bool on[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int q = q1 + x * (int)blockDim.x;
                on[x] = q < Qp && ((slevel[q >> 6] >> (q & 63)) & 1ull);
                eid[x] = INT_MAX;
                if (on[x]) eid[x] = entry_id(a, smin[(q >> 6) * kClaimStride + (q & 63)]);
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int q = q1 + x * (int)blockDim.x;
                if (!on[x]) continue;
                if (!SEG) out[BUF ? (long long)q : slot[q]] = eid[x];
                else if (eid[x] != INT_MAX) atomicMin(&out[q], eid[x]);
            }
        }
    }
    if (STATS && v == 0) {
        if (n_rows) atomicAdd(&a.stats_hub[0], (unsigned long long)n_rows);
        if (n_edges) atomicAdd(&a.stats_hub[1], (unsigned long long)n_edges);
        if (n_lines) atomicAdd(&a.stats_hub[2], (unsigned long long)n_lines);
    }
}

// Without the bit-sliced pass (W < 16, or k > 6) the row kernels write the lists themselves, and the
// segments of a giant row cannot merge there: they merge in a buffer of the giant rows' lines (row_pred
// of this launch), which this kernel moves to the list positions, a block per row.  (One block per
// giant row instead: 350 us of a 1.06 ms call of 200 queries with whitelists on 3.4M triples; 80 us now, the call 0.80 ms.)
template <int W>
__global__ void __launch_bounds__(256) k_giant_lists(FillArgs a) {
    constexpr int Qp = 64 * W;
    __shared__ long long slot[Qp];
    const int ev = a.rows[blockIdx.x];
    row_slots<W>(a, ev, threadIdx.x >> 6, 4, slot);
    __syncthreads();
    const int32_t *line = a.row_pred + (size_t)blockIdx.x * Qp;
    for (int q = threadIdx.x; q < Qp; q += 256) {
        const int w = q >> 6;
        const unsigned long long x = a.visited[(size_t)ev * W + w] & ~a.levels[(size_t)ev * W + w] & range_bits(a.q0, a.q1, w);
        if ((x >> (q & 63)) & 1ull) a.pred[slot[q]] = line[q];  // (seeds have their -1 from the tile kernel)
    }
}

// ---------------------------------------------------------------- traversed
// traversed[q][h] += out-degree of every entity whose level-h bit of q is set
template <int W>
__global__ void k_traversed(int32_t E, int Q, int k, long long plane, long long ntiles,
                            const unsigned long long *__restrict__ levels,
                            const uint32_t *__restrict__ out_off, unsigned long long *trav) {
    __shared__ unsigned long long stage[64][W + 1];
    __shared__ uint32_t sdeg[64];
    const int t = threadIdx.x, w = t >> 6, b = t & 63;
    const long long st = blockIdx.x;
    for (int h = 0; h < k; ++h) {
        unsigned long long acc = 0;
        for (int tt = 0; tt < kMegaSupers; ++tt) {
            long long tile = st * kMegaSupers + tt;
            if (tile >= ntiles) break;
            __syncthreads();
            stage[t / W][t % W] = levels[(size_t)h * plane + (size_t)tile * 64 * W + t];
            if (t < 64) {
                long long e = tile * 64 + t;
                sdeg[t] = e < E ? out_off[e + 1] - out_off[e] : 0u;
            }
            __syncthreads();
            for (int v = 0; v < 64; ++v)
                if ((stage[v][w] >> b) & 1ull) acc += sdeg[v];
        }
        if (acc && t < Q) atomicAdd(&trav[(size_t)t * k + h], acc);
    }
}

// The list of a result's active entities and their positions in it, built once per result.  The
// tiles of every count / list / predecessor kernel of a resident graph (or of a sharded one whose
// predecessor pass runs in one piece) are cut from this list.  Other sharded graphs keep tiles of
// consecutive ids: their predecessor pass works on ranges of ids, the ranges the object-sorted triples
// are streamed in.
static logoskg_status ensure_active_list(logoskg_result *r, hipStream_t st) {
    logoskg_graph *g = r->g;
    if (r->tile_ent || (g->num_shards > 1 && !joined_rows(g))) return LOGOSKG_OK;
    const long long actw = r->Epad / 32, nchunks = (actw + kActChunkWords - 1) / kActChunkWords;
    LKG_TRY(g->pool.alloc((void **)&r->tile_ent, ((size_t)r->Epad + 64) * sizeof(int32_t), st));
    LKG_TRY(g->pool.alloc((void **)&r->cpos, (size_t)r->Epad * sizeof(int32_t), st));
    LKG_TRY(g->pool.alloc((void **)&r->act_chunk, ((size_t)nchunks + 2) * sizeof(uint32_t) + 8, st));
    r->d_nact = reinterpret_cast<unsigned long long *>(r->act_chunk + (nchunks + 1) / 2 * 2);
    r->n_active = -1;
    ProfScope ps(g->prof, KK_SCAN, st);
    if (active_in_one_launch(r->Epad, r->k + 1)) {
        k_active_list<<<dim3((unsigned)((actw + kActiveListThreads - 1) / kActiveListThreads)), dim3(kActiveListThreads), 0, st>>>(r->act, actw, r->k + 1, r->d_nact, r->tile_ent, r->cpos);
        LKG_HIP(hipGetLastError());
        return LOGOSKG_OK;
    }
    const unsigned nb = (unsigned)((nchunks + 3) / 4);
    k_active_count<<<dim3(nb), dim3(256), 0, st>>>(r->act, actw, r->k + 1, nchunks, r->act_chunk);
    long long sum_chunks = kActSumChunks;
    if (const char *most = getenv("LOGOSKG_ACTIVE_SUM_CHUNKS")) sum_chunks = std::max(0, atoi(most));  // (tests reach the scan's form so)
    if (nchunks <= sum_chunks) {
        k_active_fill<true><<<dim3(nb), dim3(256), 0, st>>>(r->act, actw, r->k + 1, nchunks, r->act_chunk, r->d_nact, r->tile_ent, r->cpos);
    } else {
        k_active_scan<<<dim3(1), dim3(1024), 0, st>>>(nchunks, r->act_chunk, r->d_nact, r->tile_ent);
        k_active_fill<false><<<dim3(nb), dim3(256), 0, st>>>(r->act, actw, r->k + 1, nchunks, r->act_chunk, r->d_nact, r->tile_ent, r->cpos);
    }
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

// Per-query counts of the set bits of one plane (visited, or a level; 16-word planes: what `seen` names) as three nested exclusive
// prefixes plus the offsets of the query-major lists; the tables are allocated on first use.
static logoskg_status count_plane(logoskg_result *r, const unsigned long long *plane_bits, const Seen &seen, uint16_t **tile_base,
                                  uint32_t **super_base, uint32_t **mega_base, long long **d_off,
                                  std::vector<int64_t> *off, hipStream_t st) {
    logoskg_graph *g = r->g;
    const int W = r->W, Qp = 64 * W;
    const long long ntiles = r->Epad / kTileEntities;
    const long long nsuper = (ntiles + kSuperTiles - 1) / kSuperTiles;
    const long long nmega = (nsuper + kMegaSupers - 1) / kMegaSupers;
    r->last_stream = st;
    if (!*tile_base) LKG_TRY(g->pool.alloc((void **)tile_base, (size_t)ntiles * Qp * 2, st));
    if (!*super_base) LKG_TRY(g->pool.alloc((void **)super_base, (size_t)nsuper * Qp * 4, st));
    if (!*mega_base) LKG_TRY(g->pool.alloc((void **)mega_base, (size_t)nmega * Qp * 4, st));
    if (!*d_off) LKG_TRY(g->pool.alloc((void **)d_off, (size_t)(Qp + 1) * 8, st));
    LKG_TRY(ensure_active_list(r, st));
    {
        ProfScope ps(g->prof, KK_COUNT, st);
        const dim3 grid((unsigned)nsuper), block(1024);
        const ScanArgs scan = {*super_base, *mega_base, g->count_tickets, nsuper, r->Q, *d_off, g->h_off,
                               r->tile_ent ? r->d_nact : nullptr, g->h_ctr + C_TOTAL};
        if (W == 1) k_count_narrow<1><<<grid, block, 0, st>>>(plane_bits, ntiles, g->E, r->tile_ent, r->d_nact, *tile_base, scan);
        else if (W == 4) k_count_narrow<4><<<grid, block, 0, st>>>(plane_bits, ntiles, g->E, r->tile_ent, r->d_nact, *tile_base, scan);
        else k_count<<<grid, block, 0, st>>>(seen, ntiles, g->E, r->tile_ent, r->d_nact, *tile_base, *super_base);
    }
    if (W == 16) {
        ProfScope ps(g->prof, KK_SCAN, st);
        k_scan_level<<<dim3((unsigned)nmega, (unsigned)(Qp / 256)), dim3(256), 0, st>>>(nsuper, kMegaSupers, Qp, *super_base, *mega_base);
        k_scan_top<<<dim3(1), dim3(Qp), 0, st>>>(nmega, r->Q, Qp, *mega_base, *d_off, r->tile_ent ? r->d_nact : nullptr,
                                                 g->h_off, g->h_ctr + C_TOTAL);
    }
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipStreamSynchronize(st));
    off->assign(g->h_off, g->h_off + r->Q + 1);
    if (r->tile_ent && r->n_active < 0) r->n_active = (long long)g->h_ctr[C_TOTAL];  // (one word behind the counters' mirror)
    if (g->prof.on) g->prof.acc[KK_COUNT].units[3] += (r->tile_ent ? (r->n_active + 63) / 64 * 64 : r->Epad) * W;
    return LOGOSKG_OK;
}

void set_row_segments(FillArgs *a, const RowClasses &rows) {
    a->n_giant_rows = rows.n_giant;
    a->giant_seg_first = rows.giant_seg_first;
    a->n_giant_segs = rows.n_giant_segs;
    a->giant_place_first = rows.giant_place_first;
    a->n_giant_places = rows.n_giant_places;
    a->hub_seg_first = rows.hub_seg_first;
    a->n_hub_rows = rows.n_hub;
    a->n_hub_segs = rows.n_hub_segs;
    a->n_split_rows = rows.n_split;
    a->n_split_segs = rows.n_split_segs;
}

logoskg_status count_reached(logoskg_result *r, hipStream_t st) {
    LKG_TRY(count_plane(r, r->visited, r->W == 16 ? seen_levels(r, r->n_levels) : Seen{}, &r->tile_base, &r->super_base,
                        &r->mega_base, &r->d_reached_off, &r->reached_off, st));
    r->has_counts = true;
    return LOGOSKG_OK;
}

__global__ void k_long_index(const int32_t *__restrict__ rows, long long n, int32_t *index) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) index[rows[i]] = (int32_t)i;
}

// First predecessor fetch with 16-word planes: the entity -> long-row position map and the
// buffer the row kernels write to (one 1024-query line per long row of a launch).  A graph whose
// buffer would pass 8 GiB keeps the direct path.
logoskg_status prepare_row_pred(logoskg_graph *g, hipStream_t st) {
    if (g->row_pred_tried) return LOGOSKG_OK;
    g->row_pred_tried = true;
    // planes, or code bytes and visited words, between the two kernels of the bit-sliced predecessor pass: room
    // for every tile of the graph and 16 words, but not more than 1.25 GiB
    g->plane_buf_bytes = std::min<size_t>((size_t)5 << 28, (size_t)(g->Epad / 64 + kEmitTiles) * 16 * 64 * (64 + 8));
    if (graph_alloc(g, (void **)&g->plane_buf, g->plane_buf_bytes) != LOGOSKG_OK) g->plane_buf_bytes = 0;
    LKG_HIP(hipEventCreateWithFlags(&g->ev_rows, hipEventDisableTiming));

    const RowClasses *joined = joined_rows(g);  // (of a sharded graph)
    const long long rows = g->num_shards > 1 && !joined ? max_chunk_rows(g) : (long long)g->in_rows.n_long;
    if (rows <= 0 || (size_t)rows * 4096 > kRowPredBytes) return LOGOSKG_OK;
    LKG_TRY(graph_alloc(g, (void **)&g->long_index, (size_t)g->E * sizeof(int32_t)));
    if (graph_alloc(g, (void **)&g->row_pred, (size_t)rows * 4096) != LOGOSKG_OK) return LOGOSKG_OK;
    g->row_pred_rows = rows;
    LKG_HIP(hipMemsetAsync(g->long_index, 0xFF, (size_t)g->E * sizeof(int32_t), st));  // -1: not a long row
    k_long_index<<<dim3((unsigned)((g->in_rows.n_long + 255) / 256)), dim3(256), 0, st>>>(
        joined ? joined->longrows : g->in_rows.longrows, g->in_rows.n_long, g->long_index);
    if (g->pairs.off) {  // (no more rows than in_rows has; without room for it a fetch goes by all triples)
        const size_t bytes = (size_t)g->E * sizeof(int32_t);
        if (hipMalloc((void **)&g->pairs.long_index, bytes) == hipSuccess) {
            g->pairs.bytes += bytes;
            g->static_bytes += bytes;
            LKG_HIP(hipMemsetAsync(g->pairs.long_index, 0xFF, (size_t)g->E * sizeof(int32_t), st));
            const long long n = (long long)g->pairs.rows.n_long;
            if (n > 0) k_long_index<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(g->pairs.rows.longrows, n, g->pairs.long_index);
        } else {
            (void)hipGetLastError();
            g->pairs.long_index = nullptr;
        }
    }
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

// Entity lists of 16-word planes without hop numbers (level lists among them): a block = 16 tiles x one word of the range, a
// wavefront per tile, lane = entity, as k_pred_emit writes its lists.  A wavefront per word of the whole line leaves fourteen
// of sixteen idle where a page holds two words (a level page of 96 of 1,024 queries on 30M triples: 115 us, 67 so).  Bound by
// the number of stores, which are pieces of a tile; for more words than four (word_lists) the runs that k_lists puts together
// in LDS are worth more, unless the pieces are nearly whole or the tiles few.  us, k_lists / this kernel, by words of the page
// (tiles; share of their pairs that is listed):
//    30M triples        (13,958; .43)    2: 131 /  88    4: 164 / 147    5: 191 / 179    6: 213 / 213    8: 263 / 297    16:   479 /   582
//    under whitelists   (13,227; .02)    2:  57 /  39    4:  58 /  51    5:  59 /  58    6:  62 /  67    8:  61 /  80    16:    87 /   152
//    hub-heavy 20M      (30,447; .38)    2: 242 / 170    4: 323 / 310    5: 388 / 383    6: 455 / 461    8: 524 / 641    16: 1,025 / 1,282
//    three hops of it   (30,550; .83)    2: 327 / 243    4: 517 / 430    5: 637 / 528    6: 785 / 630    8: 1,033 / 884  16: 2,203 / 1,811
//    under whitelists   (30,360; .08)    2: 168 / 107    4: 188 / 187    5: 208 / 223    6: 237 / 266    8: 248 / 352    16:   406 /   675
//    hub-heavy 4M        (6,111; .78)    2:  86 /  45    4: 118 / 102    5: 141 / 118    6: 164 / 136    8: 213 / 176    16:   407 /   358
//    3.4M triples        (1,598; .42)    2:  38 /  23    4:  39 /  27    5:  42 /  28    6:  44 /  33    8:  48 /  38    16:    58 /    50
//    under whitelists    (1,562; .03)    2:  22 /  19    4:  23 /  21    5:  23 /  21    6:  23 /  24    8:  24 /  26    16:    30 /    34
//    hub-heavy 0.8M      (1,403; .05)    2:  31 /  21    4:  32 /  25    5:  34 /  25    6:  35 /  29    8:  36 /  30    16:    47 /    42
constexpr int kWordTiles = 16, kWordListWords = 4, kWordListPercent = 70, kWordListFewTiles = 2048, kWordListShare = 24;

static bool word_lists(const FillArgs &a, int words) {
    const long long pairs = a.ntiles * 64 * 64 * words;
    return words <= kWordListWords || a.entries * 100 >= pairs * kWordListPercent ||
           (a.ntiles <= kWordListFewTiles && a.entries * kWordListShare >= pairs);
}

__global__ void __launch_bounds__(kWordTiles * 64) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_word_lists(FillArgs a, int w0, int nw) {
    constexpr int Qp = 1024;
    __shared__ unsigned long long s_live;
    const long long L = xcd_contiguous(blockIdx.x, gridDim.x), nsup = (a.ntiles + kWordTiles - 1) / kWordTiles;
    if (L >= nsup * nw) return;  // block-uniform
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), v = lane(), w = w0 + (int)(L % nw), ql = w * 64 + v;
    const long long at = (L / nw) * kWordTiles + wave, tile = min(at, a.ntiles - 1);
    if (threadIdx.x == 0) s_live = 0ull;
    // what depends on nothing is requested together: the entities, and where query 64 w + v goes on (lane = query)
    const int32_t ew = (int32_t)tile_entity(a.tile_ent, tile, v, a.E);
    const long long pos = super_start(a, tile / kSuperTiles, Qp, ql) + a.tile_base[(size_t)tile * Qp + ql];
    const uint32_t pos_lo = (uint32_t)(unsigned long long)pos, pos_hi = (uint32_t)((unsigned long long)pos >> 32);
    const unsigned long long vis = at < a.ntiles && ew >= 0 ? a.visited[(size_t)ew * 16 + w] & range_bits(a.q0, a.q1, w) : 0ull;
    const unsigned long long mine = wave_or64(vis);
    __syncthreads();
    if (v == 0 && mine) atomicOr(&s_live, mine);
    __syncthreads();
    const unsigned long long live = uniform64(s_live);
    if (live == 0ull) return;  // block-uniform
    const uint32_t lo = (uint32_t)vis, hi = (uint32_t)(vis >> 32);
#pragma unroll
    for (int qq = 0; qq < 64; ++qq) {
        if (bit_of(live, qq)) {
            const bool bit = ((qq < 32 ? lo : hi) >> (qq & 31)) & 1u;
            const unsigned long long m = __ballot(bit);
            const unsigned long long base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)pos_hi, qq) << 32) |
                                            (uint32_t)__builtin_amdgcn_readlane((int)pos_lo, qq);
            if (bit) {
                int32_t *const pe = a.entity + base;
                pe[rank_in(m)] = ew;
            }
        }
        if ((qq & 7) == 7) __builtin_amdgcn_s_barrier();  // the tiles write their pieces of a query about together
    }
}

template <int W, int TILES>
static void launch_lists_t(Profiler &prof, const FillArgs &a, hipStream_t st) {
    const long long nblocks = (a.ntiles + TILES - 1) / TILES;
    ProfScope ps(prof, KK_LISTS, st);
    int nb = 1;
    while ((1 << nb) <= a.k) ++nb;
    dim3 grid((unsigned)nblocks), block(64 * W);
    if (!a.hop) k_lists<W, 0, TILES><<<grid, block, 0, st>>>(a);
    else if (nb <= 2) k_lists<W, 2, TILES><<<grid, block, 0, st>>>(a);
    else if (nb <= 4) k_lists<W, 4, TILES><<<grid, block, 0, st>>>(a);
    else k_lists<W, 8, TILES><<<grid, block, 0, st>>>(a);
}

// Tiles per block.  A wavefront takes the queries of its word one after the other through all tiles of the block, so a
// block of many tiles is a long chain, and until the GPU's wavefront slots are full nothing speaks for more than one
// tile: one while all tiles' wavefronts fit the slots, four while the blocks' do.  Behind that the longer runs of a
// large block are worth more: a super tile on four-word planes, half of one on 16-word planes; one-word planes stay at
// four.  us without / with hop numbers (words, tiles; by tiles per block):
//    1 word,     718 tiles      1:  34 /  38     4:  55 /  64     8:  84 / 100    16: 142 / 176
//    1 word,  15,203 tiles      1:  78 / 128     4:  71 / 109     8:  95 / 137    16: 151 / 226
//    4 words,  1,689 tiles      1:  52 /  62     4:  60 /  75     8:  89 / 110    16: 153 / 198
//    4 words,  4,591 tiles      1: 115 / 167     4:  79 / 145     8: 103 / 159    16: 168 / 275
//    4 words, 15,262 tiles      1: 429 / 645     4: 308 / 437     8: 294 / 424    16: 284 / 508
//   16 words,    719 tiles      1:  41 /  49     4:  59 /  74     8:  89 / 120
//   16 words,  1,670 tiles      1:  58 /  73     4:  55 /  71     8:  74 /  97
//   16 words, 13,676 tiles      1: 252 / 360     4: 138 / 280     8: 138 / 305
constexpr long long kListsWaves = 8192;

template <int W>
static void launch_lists_w(Profiler &prof, const FillArgs &a, hipStream_t st) {
    constexpr int most = W == 16 ? kSuperTiles / 2 : W == 4 ? kSuperTiles : 4;
    if constexpr (W == 16) {
        const int w0 = a.q0 / 64, nw = (a.q1 - 1) / 64 - w0 + 1;
        if (!a.hop && word_lists(a, nw)) {
            if (a.ntiles == 0) return;
            ProfScope ps(prof, KK_LISTS, st);
            const long long blocks = (a.ntiles + kWordTiles - 1) / kWordTiles * nw;
            k_word_lists<<<dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(kWordTiles * 64), 0, st>>>(a, w0, nw);
            return;
        }
    }
    if (a.ntiles * W <= kListsWaves) launch_lists_t<W, 1>(prof, a, st);
    else if (a.ntiles * W <= 4 * kListsWaves) launch_lists_t<W, 4>(prof, a, st);
    else launch_lists_t<W, most>(prof, a, st);
}

// True when the 16-word tile kernel can serve this launch (it then can also write the entity and
// hop lists, see FillArgs::fuse_lists).
// A level with a small frontier (at most a quarter of the triples leave it: the first level, whose
// frontier is the seeds) reaches a long object row for few queries: walking the row from
// its first entry until each of them has met a frontier subject reads most of the row.  Such a
// level is resolved from the subject side instead: the out-rows of the frontier entities are
// walked as in a push hop, and an edge (u -> o, id t) with o a long row offers t, for every query in
// level[h-1](u) & level[h](o) (& the relation's whitelist), to o's line of the row buffer with an
// atomicMin.  k_pred_push_init first sets the level's entries of the long rows to INT_MAX.
__global__ void __launch_bounds__(256) k_pred_push_init(FillArgs a, int h, long long n_rows) {
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n_rows) return;  // wavefront-uniform
    const int ev = a.rows[i];
    if (!((a.act[(size_t)h * a.actw + (ev >> 5)] >> (ev & 31)) & 1u)) return;
    const int w0 = a.q0 >> 6, w1 = (a.q1 - 1) >> 6;
    for (int w = w0; w <= w1; ++w) {
        const unsigned long long x = a.levels[(size_t)h * a.plane + (size_t)ev * 16 + w] & range_bits(a.q0, a.q1, w);
        if ((x >> lane()) & 1ull) a.row_pred[(size_t)i * 1024 + w * 64 + lane()] = INT_MAX;
    }
}

// One wavefront per short frontier row (SEG = false) or per 64-entry segment of a longer one; lane = out-edge.
template <bool MASK, bool SEG>
__global__ void __launch_bounds__(256)
k_pred_push(FillArgs a, int h, const int32_t *__restrict__ tail_rows, const RowSegment *__restrict__ segs,
            const unsigned long long *__restrict__ ctr, const uint32_t *__restrict__ out_off,
            const int32_t *__restrict__ out_obj, const uint16_t *__restrict__ out_rel,
            const int32_t *__restrict__ out_eid) {
    const long long item = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= (long long)ctr[SEG ? C_NSEG : C_NTAIL]) return;  // wavefront-uniform
    int u;
    uint32_t lo, hi;
    if (SEG) {
        const RowSegment sg = segs[item];
        u = sg.row;
        lo = sg.begin;
        hi = min(lo + (uint32_t)kPushSegment, out_off[u + 1]);
    } else {
        u = tail_rows[item];
        lo = out_off[u];
        hi = out_off[u + 1];
    }
    const int w0 = a.q0 >> 6, w1 = (a.q1 - 1) >> 6, v = lane();
    unsigned long long mine = 0;  // lane w: word w of the subject's frontier line
    if (v >= w0 && v <= w1)
        mine = a.levels[(size_t)(h - 1) * a.plane + (size_t)u * 16 + v] & range_bits(a.q0, a.q1, v);
    if (!wave_any(mine != 0)) return;  // none of the fetched queries has this subject in its frontier
    const uint32_t j = lo + (uint32_t)v;  // a segment holds at most 64 entries, a short row 32
    int o = 0, li = -1, rl = 0, eid = 0;
    if (j < hi) {
        o = out_obj[j];
        li = a.long_index[o];  // -1: a short object row, which the row walk of the tiles resolves
        if (li >= 0) {
            eid = out_eid[j];
            if (MASK) rl = out_rel[j];
        }
    }
    for (int w = w0; w <= w1; ++w) {
        const unsigned long long lu = shfl64(mine, w);
        if (lu == 0ull || li < 0) continue;
        unsigned long long m = lu & a.levels[(size_t)h * a.plane + (size_t)o * 16 + w];
        if (MASK && m) m &= a.allow[(size_t)rl * 16 + w];
        for (; m; m &= m - 1)
            atomicMin(&a.row_pred[(size_t)li * 1024 + w * 64 + (__ffsll((long long)m) - 1)], eid);
    }
}

bool pred_uses_staged_kernel(const FillArgs &a, int W) {
    return W == 16 && a.k <= kSlicedMaxK && a.plane_buf != nullptr;
}

__global__ void k_fill_int(int32_t *p, long long n, int32_t value) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

template <int W>
constexpr long long Qp_of() { return 64 * W; }

// A block of the pool may not be taken or given back inside a sequence that a stream capture records: the replays
// would use it after the pool has handed it on.  Kernels that are better with one have a form without.
bool captured(hipStream_t st) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// The row kernels: N words of the lines (narrow form), or N = 0: whole 16-word lines.
template <int W, int N, bool MASK, bool STATS>
static void launch_rows(Profiler &prof, const FillArgs &a, long long n_hub_rows, long long n_other_rows,
                        hipStream_t st_tiles, hipStream_t st_hub) {
    if (a.k == 0) return;  // seeds only: no level 1, no predecessors
    // issued first: the tile kernel waits for it, and launched after the hub kernel it ran half as fast
    if (n_other_rows > 0) {  // with row_pred: must precede the tile kernel on its stream
        hipStream_t st = a.row_pred ? st_tiles : st_hub;
        ProfScope ps(prof, KK_PRED_MID, st);
        const dim3 grid((unsigned)((n_other_rows + 3) / 4)), block(256);
        if constexpr (N > 0) {
            if (a.row_pred) k_narrow_wave<W, N, MASK, STATS, true><<<grid, block, 0, st>>>(a, n_hub_rows, n_other_rows);
            else k_narrow_wave<W, N, MASK, STATS, false><<<grid, block, 0, st>>>(a, n_hub_rows, n_other_rows);
        } else {
            if (a.row_pred) k_pred_wave<MASK, STATS, true><<<grid, block, 0, st>>>(a, n_hub_rows, n_other_rows);
            else k_pred_wave<MASK, STATS, false><<<grid, block, 0, st>>>(a, n_hub_rows, n_other_rows);
        }
    }
    if (n_hub_rows <= 0) return;
    ProfScope ps(prof, KK_PRED_HUB, st_hub);
    const long long giants = std::min(a.n_giant_rows, n_hub_rows), hubs = n_hub_rows - giants;
    // one block per hop level of a row: the levels are independent, and the longest row sets the
    // duration of the launch
    const unsigned levels = (unsigned)a.k;
    auto rows = [&](const FillArgs &x, long long first, long long n, unsigned threads) {
        const dim3 grid((unsigned)n, levels), block(threads);
        if constexpr (N > 0) {
            if (x.row_pred) k_narrow_row<W, N, MASK, STATS, true, false><<<grid, block, 0, st_hub>>>(x, first);
            else k_narrow_row<W, N, MASK, STATS, false, false><<<grid, block, 0, st_hub>>>(x, first);
        } else {
            if (x.row_pred) k_pred_row<MASK, STATS, true, false><<<grid, block, 0, st_hub>>>(x, first);
            else k_pred_row<MASK, STATS, false, false><<<grid, block, 0, st_hub>>>(x, first);
        }
    };
    if (giants > 0) {
        // Segments merge in row_pred; without it (the row kernels write the lists themselves) in a buffer of
        // the giants' own lines.  No room for that, or a capture: a block per giant row.
        FillArgs b = a;
        void *buf = nullptr;
        logoskg_graph *g = static_cast<logoskg_graph *>(a.host_graph);
        const bool segments = a.giant_seg_first && giants == a.n_giant_rows;
        if (segments && !a.row_pred && !captured(st_hub) &&
            g->pool.alloc(&buf, (size_t)giants * Qp_of<W>() * sizeof(int32_t), st_hub) == LOGOSKG_OK)
            b.row_pred = static_cast<int32_t *>(buf);
        if (segments && b.row_pred) {
            k_fill_int<<<dim3((unsigned)((giants * Qp_of<W>() + 255) / 256)), dim3(256), 0, st_hub>>>(
                b.row_pred, giants * Qp_of<W>(), INT_MAX);
            const dim3 grid((unsigned)a.n_giant_segs, levels), block(1024);
            if constexpr (N > 0) k_narrow_row<W, N, MASK, STATS, true, true><<<grid, block, 0, st_hub>>>(b, 0);
            else k_pred_row<MASK, STATS, true, true><<<grid, block, 0, st_hub>>>(b, 0);
        } else {
            rows(a, 0, giants, 1024);
        }
        if (buf) {
            k_giant_lists<W><<<dim3((unsigned)giants), dim3(256), 0, st_hub>>>(b);
            const bool zeroed[1] = {false};
            g->pool.release_after(&buf, zeroed, 1, st_hub);
        }
    }
    // Four wavefronts per row fill the GPU where there are rows enough (a row of a thousand entries leaves
    // most of a large block waiting at its barriers); fewer rows than that get sixteen.
    if (hubs > 0) rows(a, giants, hubs, hubs * levels < 2048 ? 1024u : 256u);
}

// A narrow batch's fetch in two launches: true when it was issued.  Split rows merge in a buffer of the pool; without one
// (no room, or a capture) the kernels run one by one.
template <int W, bool MASK>
static bool launch_fetch_narrow(Profiler &prof, FillArgs a, long long n_hub_rows, long long n_other_rows, hipStream_t st) {
    logoskg_graph *g = static_cast<logoskg_graph *>(a.host_graph);
    if (!a.hub_seg_first || n_hub_rows != a.n_hub_rows) return false;
    const bool rows = a.k > 0;  // (seeds only: no level 1, no predecessors)
    const long long hub = rows ? a.n_hub_segs * a.k : 0;
    const long long mid = ((rows ? (n_other_rows + 3) / 4 : 0) + hub + 7) / 8 * 8 - hub;  // (the tiles' XCDs)
    const long long tiles = ((a.tile_count * W + 3) / 4 + 7) / 8 * 8;
    if ((hub + mid + tiles) * 256 > (long long)UINT32_MAX) return false;  // (a launch holds fewer threads; deep searches)
    void *buf = nullptr;
    if (rows && a.n_split_rows > 0) {
        if (captured(st) || g->pool.alloc(&buf, (size_t)a.n_split_segs * Qp_of<W>() * sizeof(int32_t), st) != LOGOSKG_OK) return false;
        a.seg_pred = static_cast<int32_t *>(buf);
    }
    {
        ProfScope ps(prof, KK_PRED, st);
        k_fetch_narrow<W, MASK><<<dim3((unsigned)(hub + mid + tiles)), dim3(256), 0, st>>>(a, (unsigned)hub, (unsigned)mid,
                                                                                        rows ? n_other_rows : 0);
    }
    if (buf) {
        ProfScope ps(prof, KK_PRED_HUB, st);
        k_split_lists<W><<<dim3((unsigned)a.n_split_rows), dim3(256), 0, st>>>(a);
        const bool zeroed[1] = {false};
        g->pool.release_after(&buf, zeroed, 1, st);
    }
    return true;
}

template <int W, bool MASK, bool STATS>
static void launch_pred_wms(Profiler &prof, const FillArgs &a0, long long n_hub_rows, long long n_other_rows,
                            hipStream_t st_tiles, hipStream_t st_hub) {
    FillArgs a = a0;
    if constexpr (W <= 4 && !STATS)
        if (st_tiles == st_hub && launch_fetch_narrow<W, MASK>(prof, a, n_hub_rows, n_other_rows, st_tiles)) return;
    const bool mt = pred_uses_staged_kernel(a, W);
    if (!mt) a.row_pred = nullptr;
    if (!mt || W != 16 || STATS) a.push_levels = 0;
    void *packed = nullptr;  // a page's words of the level planes
    if constexpr (W <= 4) {
        launch_rows<W, W, MASK, STATS>(prof, a, n_hub_rows, n_other_rows, st_tiles, st_hub);
    } else {
        // a page of the batch inside one, two or four aligned words of the lines: the narrow form
        bool done = false;
        if constexpr (!STATS) {
            const int w0 = a.q0 >> 6, w1 = (a.q1 - 1) >> 6;
            const int words = w0 == w1 ? 1 : w0 >> 1 == w1 >> 1 ? 2 : w0 >> 2 == w1 >> 2 ? 4 : 0;
            // (one stream: the row and tile kernels read the packed planes)
            if (words && mt && a.row_pred && a.tile_ent && a.n_listed >= kPageLines && st_hub == st_tiles && !captured(st_hub)) {
                logoskg_graph *g = static_cast<logoskg_graph *>(a.host_graph);
                const long long Epad = a.plane / 16;
                const size_t bytes = (size_t)(a.k + 1) * Epad * words * 8;
                if (bytes <= kPagePlaneBytes && g->pool.alloc(&packed, bytes, st_hub) == LOGOSKG_OK) {
                    unsigned long long *dst = static_cast<unsigned long long *>(packed);
                    const int first = w0 & ~(words - 1);
                    ProfScope ps(prof, KK_PRED_WALK, st_hub);
                    const dim3 grid((unsigned)std::min<long long>(16384, (Epad + 255) / 256), (unsigned)a.k + 1), block(256);
                    if (words == 1) k_page_planes<1><<<grid, block, 0, st_hub>>>(a.levels, a.plane, a.act, a.actw, Epad, first, dst);
                    else if (words == 2) k_page_planes<2><<<grid, block, 0, st_hub>>>(a.levels, a.plane, a.act, a.actw, Epad, first, dst);
                    else k_page_planes<4><<<grid, block, 0, st_hub>>>(a.levels, a.plane, a.act, a.actw, Epad, first, dst);
                    a.plv = dst;
                    a.pplane = Epad * words;
                    a.pstride = words;
                    a.pfirst = first;
                }
            }
            done = true;
            if (w0 == w1) launch_rows<W, 1, MASK, STATS>(prof, a, n_hub_rows, n_other_rows, st_tiles, st_hub);
            else if (w0 >> 1 == w1 >> 1) launch_rows<W, 2, MASK, STATS>(prof, a, n_hub_rows, n_other_rows, st_tiles, st_hub);
            else if (w0 >> 2 == w1 >> 2) launch_rows<W, 4, MASK, STATS>(prof, a, n_hub_rows, n_other_rows, st_tiles, st_hub);
            else done = false;
        }
        if (!done) launch_rows<W, 0, MASK, STATS>(prof, a, n_hub_rows, n_other_rows, st_tiles, st_hub);
    }
    if constexpr (W == 16 && !STATS) {
        if (a.push_levels) {  // the pushed levels of the long rows, from the subject side (behind the row kernels:
                              // the giant rows' lines are filled before those run)
            logoskg_graph *g = static_cast<logoskg_graph *>(a.host_graph);
            logoskg_result *r = static_cast<logoskg_result *>(a.host_result);
            const long long n_long = n_hub_rows + n_other_rows;
            for (int h = 1; h <= a.k && n_long > 0; ++h) {
                if (!((a.push_levels >> h) & 1u)) continue;
                // (timed with the row kernels whose work it takes over; profiler scopes do not nest)
                if (census_lists(g, r, h - 1, nullptr, st_hub, KK_PRED_HUB) != LOGOSKG_OK) break;  // (the caller reads the last error)
                ProfScope ps(prof, KK_PRED_HUB, st_hub);
                k_pred_push_init<<<dim3((unsigned)((n_long + 3) / 4)), dim3(256), 0, st_hub>>>(a, h, n_long);
                // the lists' lengths are on the device; the hop's own statistics bound them
                const long long rows = r->stats[(size_t)h - 1].active_rows;
                const long long max_seg = rows + r->stats[(size_t)h - 1].frontier_edges / kPushSegment;
                if (rows > 0) {
                    k_pred_push<MASK, false><<<dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st_hub>>>(
                        a, h, g->fr_tail, g->fr_seg, g->d_ctr, g->out_off, g->out_obj, g->out_rel, g->out_eid);
                    k_pred_push<MASK, true><<<dim3((unsigned)((max_seg + 3) / 4)), dim3(256), 0, st_hub>>>(
                        a, h, g->fr_tail, g->fr_seg, g->d_ctr, g->out_off, g->out_obj, g->out_rel, g->out_eid);
                }
            }
        }
    }
    // the list writer reads the row buffer: it starts behind the block-per-row kernel
    const bool rows_first = n_hub_rows > 0 && a.row_pred && mt && st_hub != st_tiles && a.ev_rows;
    if (rows_first) (void)hipEventRecord((hipEvent_t)a.ev_rows, st_hub);
    if (a.tile_count > 0 && mt) {
        // in chunks of tiles whose planes or code bytes (64 bytes per entity and word) and, for the sparse writer, visited
        // words fit the buffer
        const int w0 = a.q0 / 64, nw = (a.q1 - 1) / 64 - w0 + 1;
        const size_t per_tile = (size_t)nw * 64 * (64 + (a.sparse ? 8 : 0));
        long long chunk = (long long)(a.plane_buf_bytes / per_tile);
        chunk = std::max<long long>(kEmitTiles, chunk / kEmitTiles * kEmitTiles);
        for (long long c0 = 0; c0 < a.tile_count; c0 += chunk) {
            const long long n = std::min(chunk, a.tile_count - c0), t0 = a.tile_begin + c0;
            unsigned long long *visbuf = a.plane_buf + (size_t)n * nw * 64 * 8;  // behind the codes
            const long long nsup = (n + kEmitTiles - 1) / kEmitTiles;
            dim3 gw((unsigned)((n * 4 + 7) / 8 * 8));
            dim3 ge((unsigned)((nsup * nw + 7) / 8 * 8));
            {
                ProfScope ps(prof, KK_PRED_WALK, st_tiles);
                // a range inside four aligned words takes four lanes per entity (16 entities per wavefront)
                const int wb = w0 & ~3;
                if (nw == 1) {  // one word: a lane per entity (64 entities per wavefront)
                    dim3 g1((unsigned)(((n + 3) / 4 + 7) / 8 * 8));  // 256 entities per block
                    if (a.k <= 2) k_pred_walk<2, MASK, STATS, 1><<<g1, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, w0, a.sparse);
                    else k_pred_walk<3, MASK, STATS, 1><<<g1, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, w0, a.sparse);
                } else if (w0 >> 1 == (w0 + nw - 1) >> 1) {  // two aligned words
                    dim3 g2((unsigned)(((n + 1) / 2 + 7) / 8 * 8));  // 128 entities per block
                    if (a.k <= 2) k_pred_walk<2, MASK, STATS, 2><<<g2, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, w0 & ~1, a.sparse);
                    else k_pred_walk<3, MASK, STATS, 2><<<g2, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, w0 & ~1, a.sparse);
                } else if (w0 + nw <= wb + 4) {
                    dim3 g4((unsigned)((n + 7) / 8 * 8));  // 64 entities per block
                    if (a.k <= 2) k_pred_walk<2, MASK, STATS, 4><<<g4, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, wb, a.sparse);
                    else k_pred_walk<3, MASK, STATS, 4><<<g4, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, wb, a.sparse);
                } else {
                    if (a.k <= 2) k_pred_walk<2, MASK, STATS, 16><<<gw, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, 0, a.sparse);
                    else k_pred_walk<3, MASK, STATS, 16><<<gw, dim3(256), 0, st_tiles>>>(a, a.plane_buf, visbuf, t0, n, w0, nw, 0, a.sparse);
                }
            }
            if (rows_first && c0 == 0) (void)hipStreamWaitEvent(st_tiles, (hipEvent_t)a.ev_rows, 0);
            ProfScope ps(prof, KK_PRED, st_tiles);
            if (a.sparse)
                k_emit_sparse<<<dim3((unsigned)(((n * nw + 3) / 4 + 7) / 8 * 8)), dim3(256), 0, st_tiles>>>(
                    a, reinterpret_cast<const uint8_t *>(a.plane_buf), visbuf, t0, n, w0, nw);
            else k_pred_emit<<<ge, dim3(kEmitTiles * 64), 0, st_tiles>>>(a, a.plane_buf, t0, n, w0, nw, a.emit_eid_cap, a.emit_line_cap);
            if (prof.on) {  // entities x words whose planes pass from the first kernel to the second
                prof.acc[KK_PRED_WALK].units[3] += n * 64 * nw;
                prof.acc[KK_PRED].units[0] += n * 64 * nw;
            }
        }
    } else if (a.tile_count > 0) {
        ProfScope ps(prof, KK_PRED, st_tiles);
        if constexpr (W <= 4) {
            const long long blocks = (a.tile_count * W + 3) / 4;
            k_pred_narrow<W, MASK, STATS><<<dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, st_tiles>>>(a);
        } else {
            k_pred<MASK, STATS><<<dim3((unsigned)((a.tile_count + 7) / 8 * 8)), dim3(64 * W), 0, st_tiles>>>(a);
        }
    }
    if (packed) {
        const bool zeroed[1] = {false};
        static_cast<logoskg_graph *>(a.host_graph)->pool.release_after(&packed, zeroed, 1, st_tiles);
    }
}

// predecessor kernels over the tiles [a.tile_begin, +a.tile_count) and the long rows a.rows[0 ..
// n_hub_rows + n_other_rows): the hub rows first (16 waves per row), then the others (one wave
// each).  The counting mode runs instantiations of its own, so that kernel statistics of the
// ordinary ones are not mixed with it.
template <int W>
static void launch_pred_w(Profiler &prof, const FillArgs &a, long long n_hub_rows, long long n_other_rows,
                          bool mask, hipStream_t st_tiles, hipStream_t st) {
    const bool stats = a.stats_pred != nullptr;
    if (mask) {
        if (stats) launch_pred_wms<W, true, true>(prof, a, n_hub_rows, n_other_rows, st_tiles, st);
        else launch_pred_wms<W, true, false>(prof, a, n_hub_rows, n_other_rows, st_tiles, st);
    } else {
        if (stats) launch_pred_wms<W, false, true>(prof, a, n_hub_rows, n_other_rows, st_tiles, st);
        else launch_pred_wms<W, false, false>(prof, a, n_hub_rows, n_other_rows, st_tiles, st);
    }
}

void launch_lists(Profiler &prof, const FillArgs &a, int W, hipStream_t st) {
    switch (W) {
        case 1: launch_lists_w<1>(prof, a, st); break;
        case 4: launch_lists_w<4>(prof, a, st); break;
        default: launch_lists_w<16>(prof, a, st); break;
    }
}

// The block-per-row kernel of the hub rows goes to st_hub and may overlap the rest; the kernel of
// the other long rows goes to st_tiles ahead of the tile kernel when its results pass through
// a.row_pred, to st_hub otherwise.
void launch_pred(Profiler &prof, const FillArgs &a, int W, long long n_hub_rows, long long n_other_rows, bool mask,
                 hipStream_t st_tiles, hipStream_t st_hub) {
    switch (W) {
        case 1: launch_pred_w<1>(prof, a, n_hub_rows, n_other_rows, mask, st_tiles, st_hub); break;
        case 4: launch_pred_w<4>(prof, a, n_hub_rows, n_other_rows, mask, st_tiles, st_hub); break;
        default: launch_pred_w<16>(prof, a, n_hub_rows, n_other_rows, mask, st_tiles, st_hub); break;
    }
}

}  // namespace lkg

using namespace lkg;

extern "C" logoskg_status logoskg_result_offsets(const logoskg_result *r, int64_t *reached_off) {
    if (!r || !reached_off) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    if (!r->has_counts) { set_error("result was computed with LOGOSKG_NO_COUNTS"); return LOGOSKG_EINVAL; }
    memcpy(reached_off, r->reached_off.data(), (size_t)(r->Q + 1) * sizeof(int64_t));
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_fetch(logoskg_result *r, int32_t q0, int32_t q1, int64_t capacity,
                                               int32_t *entity, uint8_t *hop, int32_t *pred, void *stream) {
    if (!r) { set_error("NULL result"); return LOGOSKG_EINVAL; }
    if (!r->has_counts) { set_error("result was computed with LOGOSKG_NO_COUNTS"); return LOGOSKG_EINVAL; }
    if (r->walk_exact) {
        set_error("hop and predecessor are not defined for a LOGOSKG_WALK_EXACT result: use logoskg_result_level_fetch");
        return LOGOSKG_EINVAL;
    }
    if (q0 < 0 || q1 > r->Q || q0 > q1) { set_error("bad query range [%d, %d)", q0, q1); return LOGOSKG_EINVAL; }
    int64_t need = r->reached_off[(size_t)q1] - r->reached_off[(size_t)q0];
    if (capacity < need) {
        set_error("capacity %lld < %lld entries", (long long)capacity, (long long)need);
        return LOGOSKG_ERANGE;
    }
    if (need == 0) return LOGOSKG_OK;
    if (!entity) { set_error("entity buffer is NULL"); return LOGOSKG_EINVAL; }
    logoskg_graph *g = r->g;
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    r->last_stream = st;
    if (r->small_n >= 0) {
        if (!g->prof.counters) return small_fetch(r, q0, q1, entity, hop, pred, st);
        if (!r->tile_base) LKG_TRY(count_reached(r, st));  // measured kernels: the general ones and their tables (same offsets)
    }
    const int W = r->W;
    FillArgs a = {};
    a.E = g->E; a.R = g->R; a.Q = r->Q; a.k = r->k; a.q0 = q0; a.q1 = q1; a.hub_min = g->hub_min;
    a.tile_ent = r->tile_ent; a.cpos = r->cpos; a.n_listed = r->n_active;
    a.ntiles = r->tile_ent ? (r->n_active + 63) / 64 : r->Epad / kTileEntities;
    a.tile_begin = 0; a.tile_count = a.ntiles;
    a.plane = r->Epad * W; a.actw = r->Epad / 32;
    a.visited = r->visited; a.levels = r->levels; a.allow = r->allow;
    a.plv = a.levels; a.pplane = a.plane; a.pstride = W; a.pfirst = 0;
    a.act = r->act; a.tile_base = r->tile_base; a.super_base = r->super_base; a.mega_base = r->mega_base;
    a.reached_off = r->d_reached_off;
    if (pred && W == 16) LKG_TRY(prepare_row_pred(g, st));
    // without whitelists the rows of distinct pairs (where the row buffer is used they need their own index)
    const bool pairs = !r->has_mask && g->pairs.off && g->num_shards <= 1 && !(pred && W == 16 && g->row_pred && !g->pairs.long_index);
    // what is launched from here on may read the pairs: allocations on the way go without them, not the pairs
    struct InUse {
        bool &flag;
        ~InUse() { flag = false; }
    } in_use{g->pairs.in_use};
    in_use.flag = true;
    if (g->pairs.off && !r->has_mask && captured(st)) g->pairs.recorded = true;
    const RowClasses &in_rows = pairs ? g->pairs.rows : g->in_rows;
    a.in_off = pairs ? g->pairs.off : g->in_off;
    a.in_sub = pairs ? g->pairs.sub : g->in_sub;
    a.in_eid = pairs ? g->pairs.eid : g->in_eid;
    a.in_rel = g->in_rel;
    a.rows = in_rows.longrows;
    a.row_base = 0; a.long_index = nullptr; a.row_pred = nullptr; a.fuse_lists = 0;
    a.plane_buf = nullptr; a.plane_buf_bytes = 0; a.ev_rows = nullptr;
    // levels whose frontier (the level below) holds most of the triples: the same rule as the pull hops
    for (int h = 1; h <= r->k && h < 32; ++h)
        if ((long long)r->stats[(size_t)h - 1].frontier_edges * 100 >= g->T * (long long)kDensePullPercent)
            a.dense_levels |= 1u << h;
    if (g->num_shards <= 1) set_row_segments(&a, in_rows);  // (a sharded graph: per object range, or of its joined rows)
    a.host_graph = g;
    a.host_result = r;
    if (pred && W == 16) {
        a.long_index = pairs ? g->pairs.long_index : g->long_index;
        a.row_pred = g->row_pred;
        a.plane_buf = g->plane_buf;
        a.plane_buf_bytes = g->plane_buf_bytes;
        a.ev_rows = g->ev_rows;
        // (LOGOSKG_EMIT_CAPS="e,l" shrinks what k_pred_emit puts in LDS so that tests reach its other paths)
        a.emit_eid_cap = kEmitPool;
        a.emit_line_cap = kEmitLines;
        if (const char *caps = getenv("LOGOSKG_EMIT_CAPS")) {
            int e = kEmitPool, l = kEmitLines;
            if (sscanf(caps, "%d,%d", &e, &l) == 2) {
                a.emit_eid_cap = std::max(0, std::min(e, kEmitPool));
                a.emit_line_cap = std::max(0, std::min(l, kEmitLines));
            }
        }
    }
    a.entity = entity; a.hop = hop; a.pred = pred; a.entries = need;
    {   // mostly empty words: the lists by k_emit_sparse
        const long long words = (q1 - 1) / 64 - q0 / 64 + 1;
        a.sparse = need * kSparseShare <= a.ntiles * 64 * 64 * words;
    }
    const bool counting = g->prof.counters;
    // 16-word planes: the kernels that ask visited (all but the pair of walk and writer on a list of active entities)
    if (W == 16) {
        if (pred && a.row_pred && a.tile_ent && pred_uses_staged_kernel(a, W)) {
            a.visited = nullptr;
        } else {
            g->visited_asked = true;
            LKG_TRY(share_visited(r, st));
        }
    }
    // levels whose frontier holds at most a quarter of the triples: their long rows are resolved from the
    // subject side (resident graphs, row buffer in use, minimum-hop search); needs the triple index of
    // every entry of SUB
    if (pred && W == 16 && g->num_shards <= 1 && !counting && !r->walk_exact && a.row_pred && a.long_index &&
        pred_uses_staged_kernel(a, W)) {
        uint32_t levels = 0;
        for (int h = 1; h <= r->k && h < 32; ++h)
            if (r->stats[(size_t)h - 1].active_rows > 0 &&
                (long long)r->stats[(size_t)h - 1].frontier_edges * kPredPushShare <= g->T)
                levels |= 1u << h;
        if (levels && ensure_out_eid(g, st) == LOGOSKG_OK) {
            a.push_levels = levels;
        }
    }
    a.stats_pred = counting ? g->d_ctr + C_STATS + 4 * KK_PRED : nullptr;
    a.stats_hub = counting ? g->d_ctr + C_STATS + 4 * KK_PRED_HUB : nullptr;
    a.stats_mid = counting ? g->d_ctr + C_STATS + 4 * KK_PRED_MID : nullptr;
    if (counting) LKG_HIP(hipMemsetAsync(g->d_ctr + C_STATS, 0, 4 * KK_NUM * sizeof(unsigned long long), st));
    // The kernels of a fetch run in turn on the caller's stream.  The list kernel, the per-tile
    // predecessor kernel and the per-row predecessor kernels are independent, and with
    // LOGOSKG_OVERLAP_FETCH=1 a resident graph puts them on the helper streams and joins them on the
    // caller's; measured on every benchmark configuration that gains nothing (they are bound by
    // instruction issue and gather latency and share the same units) and costs small batches the
    // fork and join, so it is not the default.
    const char *overlap_env = getenv("LOGOSKG_OVERLAP_FETCH");
    const bool serial = !(overlap_env && overlap_env[0] == '1');
    // With predecessors the tile kernel writes all three lists, except on 16-word planes without the
    // bit-sliced pass, where the list kernel runs beside the predecessor kernels.
    a.fuse_lists = pred && (W <= 4 || pred_uses_staged_kernel(a, W));
    const long long n_hub = in_rows.n_hub, n_mid = in_rows.n_long - in_rows.n_hub;
    // (nothing to fork for when the fused tile pass has no hub rows beside it)
    if (pred && g->num_shards <= 1 && !serial && (n_hub > 0 || !a.fuse_lists)) {
        LKG_HIP(hipEventRecord(g->ev_fork, st));
        for (int i = 0; i < 2; ++i) LKG_HIP(hipStreamWaitEvent(g->side[i], g->ev_fork, 0));
        if (a.fuse_lists) {
            launch_pred(g->prof, a, W, n_hub, n_mid, r->has_mask, st, g->side[0]);
        } else {
            launch_pred(g->prof, a, W, n_hub, n_mid, r->has_mask, g->side[0], g->side[1]);
            launch_lists(g->prof, a, W, st);
        }
        for (int i = 0; i < 2; ++i) {
            LKG_HIP(hipEventRecord(g->ev_join[i], g->side[i]));
            LKG_HIP(hipStreamWaitEvent(st, g->ev_join[i], 0));
        }
    } else {
        if (!a.fuse_lists) launch_lists(g->prof, a, W, st);
        if (pred) {
            if (g->num_shards > 1) LKG_TRY(sharded_pred(g, &a, W, r->has_mask, st));
            else launch_pred(g->prof, a, W, n_hub, n_mid, r->has_mask, st, st);
        }
    }
    LKG_HIP(hipGetLastError());
    if (g->prof.on) {
        if (!a.fuse_lists) g->prof.acc[KK_LISTS].units[3] += need;
        if (pred) g->prof.acc[KK_PRED].units[3] += need;
    }
    if (counting) {  // measurement mode only: wait for the counters
        LKG_HIP(hipMemcpyAsync(g->h_ctr, g->d_ctr, C_TOTAL * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        LKG_HIP(hipStreamSynchronize(st));
        for (int kind : {KK_PRED, KK_PRED_HUB, KK_PRED_MID})  // (the two-kernel tile pass counts in its first kernel)
            for (int u = 0; u < 3; ++u)
                g->prof.acc[kind == KK_PRED && pred_uses_staged_kernel(a, W) ? KK_PRED_WALK : kind].units[u] +=
                    (long long)g->h_ctr[C_STATS + 4 * kind + u];
    }
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_level_offsets(logoskg_result *r, int32_t h, int64_t *level_off,
                                                       void *stream) {
    if (!r || !level_off) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    if (h < 0 || h > r->k) { set_error("level %d outside [0, %d]", h, r->k); return LOGOSKG_EINVAL; }
    LKG_HIP(hipSetDevice(r->g->device));
    r->level_counted = -1;
    const unsigned long long *level = r->levels + (size_t)h * r->Epad * r->W;
    LKG_TRY(count_plane(r, level, Seen{level}, &r->lvl_tile_base, &r->lvl_super_base,
                        &r->lvl_mega_base, &r->d_level_off, &r->level_off, (hipStream_t)stream));
    r->level_counted = h;
    memcpy(level_off, r->level_off.data(), (size_t)(r->Q + 1) * sizeof(int64_t));
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_level_fetch(logoskg_result *r, int32_t h, int32_t q0, int32_t q1,
                                                     int64_t capacity, int32_t *entity, void *stream) {
    if (!r) { set_error("NULL result"); return LOGOSKG_EINVAL; }
    if (h < 0 || h > r->k || r->level_counted != h) {
        set_error("level %d was not counted: call logoskg_result_level_offsets for it first", h);
        return LOGOSKG_EINVAL;
    }
    if (q0 < 0 || q1 > r->Q || q0 > q1) { set_error("bad query range [%d, %d)", q0, q1); return LOGOSKG_EINVAL; }
    const int64_t need = r->level_off[(size_t)q1] - r->level_off[(size_t)q0];
    if (capacity < need) {
        set_error("capacity %lld < %lld entries", (long long)capacity, (long long)need);
        return LOGOSKG_ERANGE;
    }
    if (need == 0) return LOGOSKG_OK;
    if (!entity) { set_error("entity buffer is NULL"); return LOGOSKG_EINVAL; }
    logoskg_graph *g = r->g;
    LKG_HIP(hipSetDevice(g->device));
    r->last_stream = (hipStream_t)stream;
    const int W = r->W;
    FillArgs a = {};
    // the level plane plays the part of the visited plane; no hop numbers are asked for
    a.E = g->E; a.R = g->R; a.Q = r->Q; a.k = 0; a.q0 = q0; a.q1 = q1; a.hub_min = g->hub_min;
    a.tile_ent = r->tile_ent; a.cpos = r->cpos; a.n_listed = r->n_active;
    a.ntiles = r->tile_ent ? (r->n_active + 63) / 64 : r->Epad / kTileEntities;
    a.tile_begin = 0; a.tile_count = a.ntiles;
    a.plane = r->Epad * W; a.actw = r->Epad / 32;
    a.visited = r->levels + (size_t)h * r->Epad * W; a.levels = a.visited; a.allow = r->allow;
    a.act = r->act; a.tile_base = r->lvl_tile_base; a.super_base = r->lvl_super_base; a.mega_base = r->lvl_mega_base;
    a.reached_off = r->d_level_off;
    a.entity = entity; a.entries = need;
    launch_lists(g->prof, a, W, (hipStream_t)stream);
    LKG_HIP(hipGetLastError());
    if (g->prof.on) g->prof.acc[KK_LISTS].units[3] += need;
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_traversed(logoskg_result *r, int64_t *traversed, void *stream) {
    if (!r || (r->k > 0 && !traversed)) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    if (r->k == 0) return LOGOSKG_OK;
    logoskg_graph *g = r->g;
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    r->last_stream = st;
    const int W = r->W;
    const long long ntiles = r->Epad / kTileEntities;
    const long long nblocks = (ntiles + kMegaSupers - 1) / kMegaSupers;
    LKG_HIP(hipMemsetAsync(traversed, 0, (size_t)r->Q * r->k * 8, st));
    dim3 grid((unsigned)nblocks), block(64 * W);
    ProfScope ps(g->prof, KK_TRAVERSED, st);
    unsigned long long *tr = (unsigned long long *)traversed;
    const unsigned long long *lv = r->levels;
    switch (W) {
        case 1: k_traversed<1><<<grid, block, 0, st>>>(g->E, r->Q, r->k, r->Epad * W, ntiles, lv, g->out_off, tr); break;
        case 4: k_traversed<4><<<grid, block, 0, st>>>(g->E, r->Q, r->k, r->Epad * W, ntiles, lv, g->out_off, tr); break;
        default: k_traversed<16><<<grid, block, 0, st>>>(g->E, r->Q, r->k, r->Epad * W, ntiles, lv, g->out_off, tr); break;
    }
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}
