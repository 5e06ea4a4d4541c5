// logoskg_khop: batched k-hop expansion on one gfx950 GPU.
//
// State (paper Sec. 3.3): the query vectors q^(h) of up to 1024 queries are
// packed entity-major, W uint64 words per entity (bit j%64 of word j/64 =
// query j).  level[h] holds the bits that become set for the first time at hop
// h, visited = OR of all levels so far (on 16-word planes made when something asks for the plane: see Seen), act[h] has one
// bit per entity whose level[h] line is non-zero.
//
// One hop (Eq. 4, q.SUB.OBJ with the relation whitelist applied to the active
// triples of Eq. 5) is evaluated in one of two directions:
//   push: for every subject row in the frontier, OR its line into the lines of
//         its objects (atomicOr), skipping bits already visited;
//   pull: for every object row that still misses a query whose frontier is
//         alive, OR the lines of its subjects that are in the frontier, and
//         stop as soon as nothing is missing; no atomics on short rows, and
//         visited is updated in the same kernel (planes of one and four words)
//         or the levels themselves are asked what was reached before (16 words,
//         searches of few hops: keeps_visited).
//         Without whitelists the rows are those of the distinct (subject,
//         object) pairs where these are built.
// Both give the same level[h].  Rows of up to 32 entries are handled by a
// W-lane group each; longer rows are cut into fixed-size segments, one
// wavefront per segment, so a 100,000-entry hub spreads over many CUs.
//
// With LOGOSKG_WALK_EXACT the visited filter is dropped (Eq. 4 iterated as
// written): level[h] = image of level[h-1], an entity may be in several levels;
// visited is still their union.
#include <algorithm>

#include "common.h"

namespace lkg {

// counters of a level (kLevelCounters words behind the live words): the append cursors of its push lists, the
// census' sums, the error word of the seeds (level 0), the blocks that have added theirs, and what the next hop is to
// do if it was launched ahead of the host's decision: kHopNotPulled, or the form of the pull
enum { kHopNotPulled = 0, kHopPulled = 1, kHopPulledDense = 2 };
enum { L_CUR_TAIL = 0, L_CUR_SEG, L_ERR, L_TICKET, L_PULL };
static_assert(L_PULL < kLevelCounters && (int)L_CUR_TAIL == (int)C_NTAIL && (int)L_CUR_SEG == (int)C_NSEG,
              "the push kernels read the cursors as C_NTAIL and C_NSEG");

// ---------------------------------------------------------------- seeds, mask table
__global__ void k_seed(int Q, long long num_seeds, const long long *__restrict__ seed_off,
                       const int32_t *__restrict__ seeds, int32_t E, int W,
                       unsigned long long *level0, unsigned long long *visited, uint32_t *act0,
                       unsigned long long *ctr, long long *kept_off, int32_t *kept_seeds) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= Q) return;
    long long a = seed_off[q], b = seed_off[q + 1];
    kept_off[q] = a;  // the result keeps a copy: the caller's arrays are borrowed for the call only
    if (q == Q - 1) kept_off[Q] = b;
    if (a < 0 || b < a || b > num_seeds || (q == 0 && a != 0) || (q == Q - 1 && b != num_seeds)) {
        atomicOr(&ctr[L_ERR], 1ull);
        return;
    }
    unsigned long long bit = 1ull << (q & 63);
    for (long long i = a; i < b; ++i) {
        int32_t e = seeds[i];
        kept_seeds[i] = e;
        if ((uint32_t)e >= (uint32_t)E) {
            atomicOr(&ctr[L_ERR], 2ull);
            continue;
        }
        size_t idx = (size_t)e * W + (q >> 6);
        atomicOr(&level0[idx], bit);
        atomicOr(&visited[idx], bit);
        atomicOr(&act0[e >> 5], 1u << (e & 31));
    }
}

// allow[r][w]: bit b set when query 64w+b may follow relation r (the vector REL.m
// of every query, transposed so that one triple's relation selects a whole line).
// A wavefront per 64 queries and 64 relations: lane = query, one word of its mask, and a 64 x 64 bit transpose
// gives lane = relation.  (A thread per (relation, word) that collected its 64 bits one load after the other took
// 16 us for 200 queries and 500 relations and 21 us for 1,024; 4 us now.)
__global__ void __launch_bounds__(256)
k_allow(int Q, int R, int W, int rel_words, const unsigned long long *__restrict__ rel_mask, unsigned long long *allow) {
    const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= rel_words * W) return;  // wavefront-uniform
    const int w = item % W, rw = item / W, q = w * 64 + lane(), r = rw * 64 + lane();
    const unsigned long long x = transpose64(q < Q ? rel_mask[(size_t)q * rel_words + rw] : 0ull);
    if (r < R) allow[(size_t)r * W + w] = x;
}

// A hop is dense from kDensePullPercent of the triples leaving its frontier; from how many of them it pulls: push_most().
__host__ __device__ inline bool dense_rule(long long edges, long long T) { return edges * 100 >= T * kDensePullPercent; }

// ---------------------------------------------------------------- frontier census
// The census of a level's active bitmap gives the host what it needs to pick the direction: rows, triples and
// work-list sizes of the frontier.  The lists themselves (short subject rows; segments of the longer ones) are
// appended by a second kernel when the hop pushes.
//
// Both take eight entities per thread: their bits are one byte of the bitmap, and only where one is set are the
// nine offsets read (two 16-byte loads and one more).  A block sums in LDS; the last block adds the blocks' sums up
// and writes the totals to pinned host memory, so that no copy runs between the census and the host's wait.  The
// tickets and cursors lie behind the live words and come zeroed with them: no fill either.  With an entity per thread and step, five atomics per
// block of 1,024 and a fill before and a copy behind, a census took 17 .. 33 us and its fill and copy 13 us;
// 12 us now for 3M entities, 9 us for 407,000 with the live words of narrow planes (a chain of a few reads and the tickets).
constexpr int kCensusEntities = 8;  // per thread

// the degrees of the active ones among entities e0 .. e0 + 7 (0 elsewhere), and their bits
__device__ __forceinline__ unsigned census_degrees(const uint32_t *__restrict__ act, int32_t E,
                                                   const uint32_t *__restrict__ out_off, long long e0,
                                                   uint32_t (&d)[kCensusEntities]) {
#pragma unroll
    for (int i = 0; i < kCensusEntities; ++i) d[i] = 0;
    if (e0 >= E) return 0;
    const unsigned bits = (act[e0 >> 5] >> (e0 & 31)) & 0xffu;
    if (bits == 0) return 0;
    uint32_t o[kCensusEntities + 1];
    if (e0 + kCensusEntities <= E) {  // out_off has E + 1 entries, e0 is a multiple of 8
        const uint4 a = *reinterpret_cast<const uint4 *>(out_off + e0), b = *reinterpret_cast<const uint4 *>(out_off + e0 + 4);
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
        o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
        o[8] = out_off[e0 + 8];
    } else {
#pragma unroll
        for (int i = 0; i <= kCensusEntities; ++i) o[i] = out_off[min(e0 + i, (long long)E)];
    }
#pragma unroll
    for (int i = 0; i < kCensusEntities; ++i)
        if ((bits >> i) & 1u) d[i] = o[i + 1] - o[i];
    return bits;
}

__device__ __forceinline__ unsigned segments_of(uint32_t d) {
    return d > (uint32_t)kTailMaxDegree ? (d + kPushSegment - 1) / kPushSegment : 0u;
}

// The OR over the 64 lanes of a wavefront of x[0 .. W - 1], word by word: lane l returns word own_word<W>(l).  Four
// words are split between the quarters of the wavefront first (seven exchanges instead of 24).
template <int W>
__device__ __forceinline__ int own_word() { return W == 1 ? 0 : lane() >> 4; }

template <int W>
__device__ __forceinline__ unsigned long long wave_or_words(const unsigned long long (&x)[W]) {
    static_assert(W == 1 || W == 4, "narrow planes");
    unsigned long long r = x[0];
    if constexpr (W == 4) {
        const bool hi = lane() & 32, odd = lane() & 16;
        const unsigned long long a = (hi ? x[2] : x[0]) | shfl_xor64(hi ? x[0] : x[2], 32);
        const unsigned long long b = (hi ? x[3] : x[1]) | shfl_xor64(hi ? x[1] : x[3], 32);
        r = (odd ? b : a) | shfl_xor64(odd ? a : b, 16);
    }
#pragma unroll
    for (int m = W == 1 ? 32 : 8; m >= 1; m >>= 1) r |= shfl_xor64(r, m);
    return r;
}

template <int W>
__device__ __forceinline__ void load_line(unsigned long long (&x)[W], const unsigned long long *__restrict__ p) {
    if constexpr (W == 1) {
        x[0] = *p;
    } else {
#pragma unroll
        for (int i = 0; i < W; i += 2) {
            const ulonglong2 y = *reinterpret_cast<const ulonglong2 *>(p + i);
            x[i] = y.x;
            x[i + 1] = y.y;
        }
    }
}

// Planes of one and four words (LW > 0): the same pass collects the level's live words (see k_live) from the lines of the
// active rows.  A launch of its own for them was 6 us per pulled hop; without them a row could not stop early where
// some queries of the batch have nothing left to expand.  Behind a pulled hop (PULLED) the pass reads the level's lines
// in order, lane = entity, and makes the bitmap from them: set by the pull kernels, a bit was an atomic per row, and they
// were half of a hop's time on 407,000 entities.
template <int LW, bool PULLED>
__global__ void __launch_bounds__(LW ? 512 : 1024)
k_census(uint32_t *act, int32_t E, const uint32_t *__restrict__ out_off, unsigned long long *ctr,
         unsigned long long *sums, unsigned long long *host, const unsigned long long *__restrict__ lines,
         unsigned long long *live, const unsigned long long *go, long long T, long long push_most, int Q) {
    if constexpr (PULLED)
        if (go && *go == kHopNotPulled) return;  // launched ahead for a hop that is not taken this way
    static_assert(!PULLED || LW > 0, "16-word lines are not read for their bits");
    constexpr int NT = LW ? 512 : 1024, NS = 3 + LW;  // threads, words per block
    constexpr int G = 4;                              // PULLED: entities per lane
    __shared__ unsigned long long part[NT / 64][NS];
    unsigned long long lists = 0, rows = 0, edges = 0;  // short rows | segments << 32, rows | active entities << 32
    unsigned long long lv[LW > 0 ? LW : 1] = {};
    const int wave = threadIdx.x >> 6;
    auto add = [&](uint32_t d) {
        lists += (unsigned long long)(d > 0 && d <= (uint32_t)kTailMaxDegree) | ((unsigned long long)segments_of(d) << 32);
        rows += d > 0;
        edges += d;
    };
    if constexpr (PULLED) {
        const long long stride = (long long)gridDim.x * NT * G;
        for (long long base = ((long long)blockIdx.x * NT + 64 * wave) * G; base < E; base += stride) {  // wavefront-uniform
            unsigned long long x[G][LW];
            uint32_t a[G], b[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const long long e = base + 64 * g + lane();
                a[g] = b[g] = 0;
#pragma unroll
                for (int w = 0; w < LW; ++w) x[g][w] = 0;
                if (e < E) {
                    load_line<LW>(x[g], lines + (size_t)e * LW);
                    a[g] = out_off[e];
                    b[g] = out_off[e + 1];
                }
            }
            unsigned long long mine = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                unsigned long long any = x[g][0];
#pragma unroll
                for (int w = 1; w < LW; ++w) any |= x[g][w];
                const unsigned long long m = __ballot(any != 0);
                if (lane() == g) mine = m;
                rows += (unsigned long long)(any != 0) << 32;
                if (any != 0 && b[g] > a[g]) {
                    add(b[g] - a[g]);
#pragma unroll
                    for (int w = 0; w < LW; ++w) lv[w] |= x[g][w];
                }
            }
            // (the bitmap covers E rounded up to a multiple of 64 entities)
            if (lane() < G && base + 64 * lane() < E) *reinterpret_cast<unsigned long long *>(act + base / 32 + 2 * lane()) = mine;
        }
    } else {
        const long long stride = (long long)gridDim.x * NT * kCensusEntities;
        for (long long e0 = ((long long)blockIdx.x * NT + threadIdx.x) * kCensusEntities; e0 < E; e0 += stride) {
            uint32_t d[kCensusEntities];
            const unsigned bits = census_degrees(act, E, out_off, e0, d);
            if (!bits) continue;
#pragma unroll
            for (int i = 0; i < kCensusEntities; ++i) add(d[i]);
            rows += (unsigned long long)__popc(bits) << 32;
            if constexpr (LW > 0) {
#pragma unroll
                for (int i = 0; i < kCensusEntities; ++i)
                    if (d[i] > 0)
#pragma unroll
                        for (int w = 0; w < LW; ++w) lv[w] |= lines[(size_t)(e0 + i) * LW + w];
            }
        }
    }
    // the block's sums (and live words) in part[0 ..][] and, by thread, of thread i in the last block
    auto put_part = [&]() {
        lists = (unsigned long long)wave_sum((long long)lists);
        rows = (unsigned long long)wave_sum((long long)rows);
        edges = (unsigned long long)wave_sum((long long)edges);
        if constexpr (LW > 0) {
            const unsigned long long x = wave_or_words<LW>(lv);
            if ((lane() & (64 / LW - 1)) == 0) part[wave][3 + own_word<LW>()] = x;
        }
        if (lane() == 0) {
            part[wave][0] = lists;
            part[wave][1] = rows;
            part[wave][2] = edges;
        }
    };
    auto total = [&](int i) {
        unsigned long long x = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) x = i < 3 ? x + part[w][i] : x | part[w][i];
        return x;
    };
    put_part();
    __syncthreads();
    // The block's sums go to a line of their own; whoever takes the last ticket adds them all up.  (Three atomics
    // per block on the level's counters were 6 ns each, one after the other: 16 us with 367 blocks.)
    __shared__ int last;
    if (threadIdx.x < NS)
        __hip_atomic_store(&sums[(size_t)blockIdx.x * NS + threadIdx.x], total((int)threadIdx.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sums (of this wavefront's lanes) are in before the ticket is taken
    if (threadIdx.x == 0) last = atomicAdd(&ctr[L_TICKET], 1ull) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;  // block-uniform
    lists = rows = edges = 0;
#pragma unroll
    for (int w = 0; w < LW; ++w) lv[w] = 0;
    if (threadIdx.x < gridDim.x) {  // at most kCensusBlocks = 512 blocks
        unsigned long long *x = sums + (size_t)threadIdx.x * NS;
        lists = __hip_atomic_load(x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        rows = __hip_atomic_load(x + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        edges = __hip_atomic_load(x + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int w = 0; w < LW; ++w) lv[w] = __hip_atomic_load(x + 3 + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    put_part();
    __syncthreads();
    if constexpr (LW > 0)
        if (threadIdx.x >= 3 && threadIdx.x < NS) live[threadIdx.x - 3] = total((int)threadIdx.x);
    // 16-word planes: every query counts as live where the next hop gathers all lines (hardly any query has nothing
    // left then, and one wrongly taken as live only keeps a row from stopping early: its bit is in no frontier line);
    // otherwise k_live finds them
    if constexpr (LW == 0)
        if (threadIdx.x < 16 && dense_rule((long long)total(2), T)) live[threadIdx.x] = query_bits(Q, (int)threadIdx.x);
    if (threadIdx.x != 0) return;
    lists = total(0);
    rows = total(1);
    host[C_NTAIL] = lists & 0xffffffffull;
    host[C_NSEG] = lists >> 32;
    host[C_NROWS] = rows & 0xffffffffull;
    host[C_NACTIVE] = rows >> 32;
    host[C_FEDGES] = edges = total(2);
    host[C_ERR] = __hip_atomic_load(&ctr[L_ERR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (LW > 0) ctr[L_PULL] = (long long)edges <= push_most ? kHopNotPulled : dense_rule((long long)edges, T) ? kHopPulledDense : kHopPulled;
    __threadfence_system();
    __hip_atomic_store(&host[kCensusDone], 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The push lists of a level; ctr[L_CUR_TAIL] and ctr[L_CUR_SEG] are the append cursors (zero before) and then the
// lengths that the push kernels read.
__global__ void __launch_bounds__(1024)
k_census_lists(const uint32_t *__restrict__ act, int32_t E, const uint32_t *__restrict__ out_off, int32_t *list_tail,
               RowSegment *list_seg, unsigned long long *ctr) {
    // a block reserves the places of its entries with one atomic per list
    __shared__ int wave_n[2][16];
    __shared__ unsigned long long first[2];
    const int wave = threadIdx.x >> 6;
    const long long stride = (long long)gridDim.x * 1024 * kCensusEntities;
    for (long long base = (long long)blockIdx.x * 1024 * kCensusEntities; base < E; base += stride) {  // block-uniform
        const long long e0 = base + (long long)threadIdx.x * kCensusEntities;
        uint32_t d[kCensusEntities];
        census_degrees(act, E, out_off, e0, d);
        int nt = 0, ns = 0;
#pragma unroll
        for (int i = 0; i < kCensusEntities; ++i) {
            nt += d[i] > 0 && d[i] <= (uint32_t)kTailMaxDegree;
            ns += (int)segments_of(d[i]);
        }
        int all_t, all_s;
        const int pt = wave_excl_scan(nt, all_t), ps = wave_excl_scan(ns, all_s);
        if (lane() == 0) {
            wave_n[0][wave] = all_t;
            wave_n[1][wave] = all_s;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            int n = 0;
            for (int w = 0; w < 16; ++w) n += wave_n[threadIdx.x][w];
            first[threadIdx.x] = n ? atomicAdd(&ctr[threadIdx.x ? L_CUR_SEG : L_CUR_TAIL], (unsigned long long)n) : 0ull;
        }
        __syncthreads();
        unsigned long long bt = first[0] + pt, bs = first[1] + ps;
        for (int w = 0; w < wave; ++w) {
            bt += wave_n[0][w];
            bs += wave_n[1][w];
        }
#pragma unroll
        for (int i = 0; i < kCensusEntities; ++i) {
            const int32_t e = (int32_t)(e0 + i);
            if (d[i] > 0 && d[i] <= (uint32_t)kTailMaxDegree) list_tail[bt++] = e;
            const unsigned n = segments_of(d[i]);
            if (wave_any(n != 0)) write_segments(list_seg, bs, n, e, n ? out_off[e] : 0u);
            bs += n;
        }
        __syncthreads();  // (the counts are rewritten by the next turn)
    }
}

template <int W>
__device__ __forceinline__ unsigned long long or_across_groups(unsigned long long acc) {
#pragma unroll
    for (int m = W; m < 64; m <<= 1) acc |= shfl_xor64(acc, m);
    return acc;
}

// live[w] = OR of the frontier lines of every subject row that has a triple:
// the queries for which this hop can still reach something.  A pull row stops
// as soon as it has all of them.  (Narrow planes: by the census.)
template <int W>
__device__ __forceinline__ int take_candidates(unsigned long long &rest);

template <int W>
__global__ void __launch_bounds__(256)
k_live(const uint32_t *__restrict__ act, int32_t E, const uint32_t *__restrict__ out_off,
       const unsigned long long *__restrict__ prev, unsigned long long *live) {
    __shared__ unsigned long long sl[16];
    if (threadIdx.x < 16) sl[threadIdx.x] = 0;
    __syncthreads();
    // a wavefront tests 64 consecutive entities (coalesced), then its groups fetch the lines of
    // the frontier rows among them, two at a time
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    const int lw = threadIdx.x & (W - 1);
    unsigned long long acc = 0;
    for (long long base = ((long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < E;
         base += nwaves * 64) {
        const long long e = base + lane();
        bool on = false;
        if (e < E) on = ((act[e >> 5] >> (e & 31)) & 1u) && out_off[e + 1] > out_off[e];
        unsigned long long m = __ballot(on);
        while (m) {
            const int p0 = take_candidates<W>(m), p1 = take_candidates<W>(m);
            unsigned long long l0 = 0, l1 = 0;
            if (p0 >= 0) l0 = prev[(size_t)(base + p0) * W + lw];
            if (p1 >= 0) l1 = prev[(size_t)(base + p1) * W + lw];
            acc |= l0 | l1;
        }
    }
    acc = or_across_groups<W>(acc);
    if (lane() < W && acc) atomicOr(&sl[lane()], acc);
    __syncthreads();
    if (threadIdx.x < W) {
        unsigned long long x = sl[threadIdx.x];
        if (x & ~live[threadIdx.x]) atomicOr(&live[threadIdx.x], x);
    }
}

// ---------------------------------------------------------------- push
__device__ __forceinline__ void mark_active(uint32_t *act, int e) {
    uint32_t bit = 1u << (e & 31);
    if (!(act[e >> 5] & bit)) atomicOr(&act[e >> 5], bit);
}

// `known` = the bits that need not be set again: the visited plane (minimum-hop search: an entity
// keeps its first level) or, for walk-exact levels, the level under construction itself.  NULL in the first hop, where
// visited holds nothing but the seeds: k_update_visited takes out the few pairs that are seeds, and an edge costs
// an atomic and no read of a line in front of it.
//
// Lines of at most kFewWords non-zero words (the seeds' nearly always) go lane = edge: every lane sets the words of its
// own edge's object, 64 edges of a segment or G of a short row in flight.  With lane = word, four edges of a segment and
// one of a short row were in flight, most lanes idle, and the kernels were chains of as many turns (first hop, us,
// segments / short rows: 1,024 queries on 30M triples 23 / 30 -> 8 / 6, 200 with whitelists on 3.4M 6 / 17 -> 4 / 6, 25M
// edges of hub subjects on 20M entities 1,396 -> 1,095, where the atomics on 2.5 GB of lines remain).
constexpr int kFewWords = 4;

// one edge per lane: the words `words` (bits; the caller's lanes agree on how many) of a line into object o's
template <int W, bool MASK, typename Line>
__device__ __forceinline__ void push_edge(bool on, int o, int r, unsigned words, Line word_of, const unsigned long long *__restrict__ allow,
                                          const unsigned long long *known, unsigned long long *cur, uint32_t *act_cur) {
    bool any = false;
    while (words) {
        const int w = __ffs((int)words) - 1;
        words &= words - 1;
        unsigned long long m = word_of(w);
        if (!on) continue;
        if (MASK) m &= allow[(size_t)r * W + w];
        if (m && known) m &= ~known[(size_t)o * W + w];
        if (m) {
            atomicOr(&cur[(size_t)o * W + w], m);
            any = true;
        }
    }
    if (any) mark_active(act_cur, o);
}

// A group of G lanes per short frontier row.
template <int W>
constexpr int push_tail_lanes() { return W == 16 ? 16 : 8; }

template <int W, bool MASK>
__global__ void __launch_bounds__(256)
k_push_tail(const int32_t *__restrict__ rows, long long first, const unsigned long long *__restrict__ ctr,
            const uint32_t *__restrict__ off, const uint32_t *__restrict__ row_begin,
            const int32_t *__restrict__ obj,
            const uint16_t *__restrict__ rel, const unsigned long long *__restrict__ allow,
            const unsigned long long *__restrict__ prev, const unsigned long long *known,
            unsigned long long *cur, uint32_t *act_cur) {
    constexpr int G = push_tail_lanes<W>();
    const long long gidx = first + ((long long)blockIdx.x * blockDim.x + threadIdx.x) / G;
    const int gl = threadIdx.x & (G - 1), g0 = lane() & ~(G - 1);
    if (gidx >= (long long)ctr[C_NTAIL]) return;  // the lanes of a group together
    const int s = rows[gidx];
    const uint32_t lo = row_begin[s], hi = lo + (off[s + 1] - off[s]);
    const unsigned long long line = gl < W ? prev[(size_t)s * W + gl] : 0ull;
    const unsigned words = (unsigned)((__ballot(line != 0) >> g0) & ((1u << G) - 1u));
    if (W <= kFewWords || __popc(words) <= kFewWords) {
        for (uint32_t j0 = lo; j0 < hi; j0 += G) {  // the lanes of a group together: they hold each other's words
            const uint32_t j = j0 + gl;
            const bool on = j < hi;
            const int o = on ? obj[j] : 0, r = MASK && on ? rel[j] : 0;
            push_edge<W, MASK>(on, o, r, words, [&](int w) { return __shfl(line, g0 + w); }, allow, known, cur, act_cur);
        }
        return;
    }
    for (uint32_t j = lo; j < hi; ++j) {  // 16 words: lane = word, an edge after the other
        const int o = obj[j];
        unsigned long long m = line;
        if (MASK) m &= allow[(size_t)rel[j] * W + gl];
        if (m && known) m &= ~known[(size_t)o * W + gl];
        if (m) atomicOr(&cur[(size_t)o * W + gl], m);
        const bool any = group_any<G>(m != 0);
        if (any && gl == 0) mark_active(act_cur, o);
    }
}

// One wavefront per segment (64 consecutive edges) of a long frontier row, a lane per edge; where many words of the line
// hold something the 64/W groups take the edges in turn, lane = word.
template <int W, bool MASK>
__global__ void __launch_bounds__(256)
k_push_seg(const RowSegment *__restrict__ segs, const unsigned long long *__restrict__ ctr,
           const uint32_t *__restrict__ off, const uint32_t *__restrict__ row_begin,
           const int32_t *__restrict__ obj,
           const uint16_t *__restrict__ rel, const unsigned long long *__restrict__ allow,
           const unsigned long long *__restrict__ prev, const unsigned long long *known,
           unsigned long long *cur, uint32_t *act_cur) {
    const long long item = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (item >= (long long)ctr[C_NSEG]) return;
    const RowSegment sg = segs[item];
    const int lw = lane() & (W - 1), g = lane() / W;
    const unsigned long long line = prev[(size_t)sg.row * W + lw];
    const uint32_t row_end = row_begin[sg.row] + (off[sg.row + 1] - off[sg.row]);
    const uint32_t hi = min(sg.begin + (uint32_t)kPushSegment, row_end);
    static_assert(kPushSegment == 64, "an edge per lane");
    const uint32_t j = sg.begin + lane();
    const bool on = j < hi;
    const int o = on ? obj[j] : 0, r = MASK && on ? rel[j] : 0;
    const unsigned words = (unsigned)__ballot(line != 0) & ((1u << W) - 1u);
    if (W <= kFewWords || __popc(words) <= kFewWords) {  // wavefront-uniform
        push_edge<W, MASK>(on, o, r, words, [&](int w) {
            return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(line >> 32), w) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)line, w);
        }, allow, known, cur, act_cur);
        return;
    }
    const int n = (int)(hi - sg.begin);
    for (int i = 0; i < n; i += 64 / W) {
        const int idx = i + g;
        const int oc = __shfl(o, idx & 63), rc = MASK ? __shfl(r, idx & 63) : 0;
        if (idx < n) {
            unsigned long long m = line;
            if (MASK) m &= allow[(size_t)rc * W + lw];
            if (m && known) m &= ~known[(size_t)oc * W + lw];
            if (m) atomicOr(&cur[(size_t)oc * W + lw], m);
            const bool any = group_any<W>(m != 0);
            if (any && lw == 0) mark_active(act_cur, oc);
        }
    }
}

// The first hop of searches that do not keep visited: pairs that are seeds leave its level, and so do active bits of lines that held nothing
// else.  Only an entity that is active in both levels can hold one, of which there are as many as seeds: a thread per 64
// entities reads their two bitmap words.  (With visited kept as on narrow planes, 11M lines of 20M entities were read twice
// and written: 514 us, 5 us now, and as many lines less to clear.)
__global__ void __launch_bounds__(256)
k_drop_seeds(long long words, const uint32_t *__restrict__ act0, uint32_t *act1, const unsigned long long *__restrict__ level0,
             unsigned long long *level1) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= words) return;
    unsigned long long *const bits = reinterpret_cast<unsigned long long *>(act1) + i;
    const unsigned long long was = *bits;
    unsigned long long gone = 0;
    for (unsigned long long m = was & reinterpret_cast<const unsigned long long *>(act0)[i]; m; m &= m - 1) {
        const int b = __ffsll((long long)m) - 1;
        const ulonglong2 *seeds = reinterpret_cast<const ulonglong2 *>(level0 + ((size_t)i * 64 + b) * 16);
        ulonglong2 *line = reinterpret_cast<ulonglong2 *>(level1 + ((size_t)i * 64 + b) * 16);
        unsigned long long any = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const ulonglong2 x = line[w], y = seeds[w];
            const ulonglong2 z = make_ulonglong2(x.x & ~y.x, x.y & ~y.y);
            if (z.x != x.x || z.y != x.y) line[w] = z;
            any |= z.x | z.y;
        }
        if (any == 0) gone |= 1ull << b;
    }
    if (gone) *bits = was & ~gone;
}

// visited |= level[h] on the lines the push kernels touched.
// One wavefront per 64 entities: it reads their two words of the active bitmap once and touches
// only the lines of the active ones (after a push from a small frontier almost none), W lanes per
// line, so a dense level is still updated with contiguous accesses.
// FIRST: the hop has set bits without asking visited; those that were there (the seeds) leave the level, and
// so do lines and active bits that held nothing else.
template <int W, bool FIRST>
__global__ void __launch_bounds__(256)
k_update_visited(long long Epad, uint32_t *act_cur, unsigned long long *cur, unsigned long long *visited) {
    const long long base = ((long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
    if (base >= Epad) return;  // Epad is a multiple of 64
    const unsigned long long m =
        ((unsigned long long)act_cur[base / 32 + 1] << 32) | (unsigned long long)act_cur[base / 32];
    if (m == 0) return;
    constexpr int GPW = 64 / W;
    const int g = lane() / W, lw = lane() & (W - 1);
    unsigned long long gone = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int e = i * GPW + g;
        const bool on = (m >> e) & 1ull;
        const size_t x = ((size_t)base + e) * W + lw;
        unsigned long long c = 0;
        if (on) {
            const unsigned long long was = visited[x], set = cur[x];
            c = FIRST ? set & ~was : set;
            if (FIRST && c != set) cur[x] = c;
            if (c) visited[x] = was | c;
        }
        const bool any = group_any<W>(c != 0);
        if (FIRST && on && !any) gone |= 1ull << e;
    }
    if constexpr (FIRST) {
        if (!wave_any(gone != 0)) return;
#pragma unroll
        for (int x = 32; x >= 1; x >>= 1) gone |= shfl_xor64(gone, x);
        if (lane() < 2) act_cur[base / 32 + lane()] = (uint32_t)((m & ~gone) >> (32 * lane()));
    }
}

// ---------------------------------------------------------------- pull
// From this share of the triples leaving the frontier the pull kernels gather every edge's line
// without asking for its frontier bit first.  A bit test is a scattered 4-byte load, i.e. a 64-byte
// sector through the L1 per edge, and these kernels are bound by what the L2s deliver; skipping the
// test costs the lines of the edges outside the frontier (zero lines: a level line is non-zero only
// where its active bit is set), which is less traffic as soon as half the edges are inside.
// Removes up to 64/W candidates from the (wave-uniform) mask and returns the
// lane position of the one that belongs to the caller's group, or -1.
template <int W>
__device__ __forceinline__ int take_candidates(unsigned long long &rest) {
    constexpr int GPW = 64 / W;
    int g = lane() / W, mine = -1;
#pragma unroll
    for (int t = 0; t < GPW; ++t) {
        if (rest) {
            int p = __ffsll((long long)rest) - 1;
            rest &= rest - 1;
            if (t == g) mine = p;
        }
    }
    return mine;
}

// 64 consecutive in-edges of one object row, in three stages so that a caller can
// keep the loads of later chunks in flight: subject (and relation) ids, the
// frontier bit of every subject, then the gather of the frontier lines of the
// candidates (pull_gather).
struct PullEdges {
    int s, r;
};

template <bool MASK>
__device__ __forceinline__ PullEdges pull_load_edges(uint32_t j0, uint32_t hi, const int32_t *__restrict__ in_sub,
                                                     const uint16_t *__restrict__ in_rel) {
    PullEdges e{-1, 0};
    uint32_t j = j0 + lane();
    if (j < hi) {
        e.s = in_sub[j];
        if (MASK) e.r = in_rel[j];
    }
    return e;
}

__device__ __forceinline__ bool pull_test(const PullEdges &e, const uint32_t *__restrict__ act_prev) {
    return e.s >= 0 && ((act_prev[e.s >> 5] >> (e.s & 31)) & 1u);
}

// Gather stage.  The candidates' subject ids are compacted into a per-wavefront
// LDS queue (position = number of candidates in lower lanes); group g of round r
// then reads entry r * (groups per round) + g, so picking a candidate costs one
// LDS read instead of a search in the ballot mask and a cross-lane move.  A lane
// loads two plane words (16 bytes): W/2 lanes cover a line and one load
// instruction of a wavefront fetches 128/W lines, which halves the number of
// vector memory instructions against one word per lane.  Up to four rounds of
// loads are in flight; only the last, partly filled batch is predicated.
// a0 / a1 collect words 2*(lane % (W/2)) and 2*(lane % (W/2)) + 1 (W = 1: a0 only).
template <int W, bool MASK>
__device__ __forceinline__ int pull_gather(const PullEdges &e, bool cand, const unsigned long long *__restrict__ prev,
                                           const unsigned long long *__restrict__ allow, unsigned long long &a0,
                                           unsigned long long &a1, int *queue_s, uint16_t *queue_r) {
    const unsigned long long cm = __ballot(cand);
    const int ncand = __popcll(cm);
    if constexpr (W == 1) {
        if (cand) {
            unsigned long long ln = prev[e.s];
            if (MASK) ln &= allow[e.r];
            a0 |= ln;
        }
    } else {
        constexpr int LW = W / 2, GPW = 64 / LW;            // lanes per line, lines per load instruction
        constexpr int NR = GPW >= 32 ? 64 / GPW : 4, B = NR * GPW;  // rounds and candidates per batch
        const ulonglong2 *prev2 = reinterpret_cast<const ulonglong2 *>(prev);
        const ulonglong2 *allow2 = reinterpret_cast<const ulonglong2 *>(allow);
        if (ncand == 0) return 0;
        if (cand) {
            const int pos = __popcll(cm & ((1ull << lane()) - 1ull));
            queue_s[pos] = e.s;
            if (MASK) queue_r[pos] = (uint16_t)e.r;
        }
        __builtin_amdgcn_wave_barrier();
        const int lw = lane() & (LW - 1), g = lane() / LW;
        int base = 0;
        for (; base + B <= ncand; base += B) {  // full batches
            ulonglong2 l[NR];
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                const int i = base + x * GPW + g;
                l[x] = prev2[(size_t)queue_s[i] * LW + lw];
                if (MASK) {
                    const ulonglong2 m = allow2[(size_t)queue_r[i] * LW + lw];
                    l[x].x &= m.x;
                    l[x].y &= m.y;
                }
            }
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                a0 |= l[x].x;
                a1 |= l[x].y;
            }
        }
        if (base < ncand) {
            ulonglong2 l[NR], ok[NR];  // (put together behind all loads: in the branch, each round waited for its own)
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                const int i = base + x * GPW + g;
                l[x] = ok[x] = make_ulonglong2(0, 0);
                if (i < ncand) {
                    l[x] = prev2[(size_t)queue_s[i] * LW + lw];
                    if (MASK) ok[x] = allow2[(size_t)queue_r[i] * LW + lw];
                }
            }
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                if (MASK) {
                    l[x].x &= ok[x].x;
                    l[x].y &= ok[x].y;
                }
                a0 |= l[x].x;
                a1 |= l[x].y;
            }
        }
        __builtin_amdgcn_wave_barrier();  // the queue is rewritten by the next chunk
    }
    return ncand;
}

// Folds the accumulators of pull_gather into one word per lane (word lane % W),
// the union over the whole wavefront.
template <int W>
__device__ __forceinline__ unsigned long long fold_gathered(unsigned long long a0, unsigned long long a1) {
    if constexpr (W == 1) {
        return or_across_groups<1>(a0);
    } else {
        a0 = or_across_groups<W / 2>(a0);
        a1 = or_across_groups<W / 2>(a1);
        const int lw = lane() & (W - 1);
        const unsigned long long x = shfl64(a0, lw >> 1), y = shfl64(a1, lw >> 1);
        return (lw & 1) ? y : x;
    }
}

__device__ __forceinline__ void add_stats(unsigned long long *stats, long long rows, long long edges,
                                          long long lines) {
    // called by every lane of a wavefront with per-lane partial counts
    rows = wave_sum(rows);
    edges = wave_sum(edges);
    lines = wave_sum(lines);
    if (lane() == 0) {
        if (rows) atomicAdd(&stats[0], (unsigned long long)rows);
        if (edges) atomicAdd(&stats[1], (unsigned long long)edges);
        if (lines) atomicAdd(&stats[2], (unsigned long long)lines);
    }
}

template <int W>
__device__ __forceinline__ unsigned group_ballot(bool p) {
    if constexpr (W == 1) return p ? 1u : 0u;
    else {
        unsigned long long b = __ballot(p);
        return (unsigned)((b >> (lane() & ~(W - 1))) & ((1ull << W) - 1ull));
    }
}

// Short object rows (<= 32 entries): a W-lane group works on kTailRows rows at
// once.  A row is a chain of dependent loads (row record -> what has reached the row and its
// subject ids -> frontier bits -> frontier lines), and with all wavefront
// slots of a CU taken the kernel is bound by that latency, so the work list carries
// the row bounds (no look-up in the offsets) and every group keeps
// the chains of two rows in flight: each stage is issued for both rows before
// either result is used.  Per stage the group's lanes load W entries of a row,
// then gather the frontier lines of its candidates, two per row at a time.
// (three or four rows per group measured the same: the kernel then runs at the
// rate at which the memory system serves its scattered lines.)
constexpr int kTailRows = 2;
constexpr int kTailLines = 2;  // candidate lines of each row requested together

// Word lw of what has reached the entities v[0 .. N - 1].  The bits of the base and of two levels, then the lines that they
// ask for, are requested for all of them together.
template <int N>
__device__ __forceinline__ void seen_words(const Seen &s, const int (&v)[N], const bool (&have)[N], int lw, unsigned long long (&x)[N]) {
    constexpr int W = 16, L = 2;
    bool base[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
        x[r] = 0ull;
        base[r] = have[r] && s.base && active_in_base(s, v[r]);
    }
    int l0 = s.first;
    do {
        bool on[N][L];
#pragma unroll
        for (int i = 0; i < L; ++i)
#pragma unroll
            for (int r = 0; r < N; ++r)
                on[r][i] = have[r] && l0 + i < s.last && ((s.sure && l0 + i == s.last - 1) || active_in(s, l0 + i, v[r]));
#pragma unroll
        for (int r = 0; r < N; ++r) {
            if (base[r]) x[r] |= s.base[(size_t)v[r] * W + lw];
            base[r] = false;
        }
#pragma unroll
        for (int i = 0; i < L; ++i)
#pragma unroll
            for (int r = 0; r < N; ++r)
                if (on[r][i]) x[r] |= s.levels[(size_t)(l0 + i) * s.plane + (size_t)v[r] * W + lw];
        l0 += L;
    } while (l0 < s.last);
}

template <int W, bool MASK, bool STATS, bool DENSE>
__global__ void __launch_bounds__(256)
k_pull_tail(const ShortRow *__restrict__ rows, long long n, const int32_t *__restrict__ in_sub, const uint16_t *__restrict__ in_rel,
            const unsigned long long *__restrict__ allow, const uint32_t *__restrict__ act_prev,
            const unsigned long long *__restrict__ prev, const unsigned long long *__restrict__ live,
            unsigned long long *visited, Seen seen, unsigned long long *cur, uint32_t *act_cur,
            unsigned long long *stats, int walk_exact) {
    constexpr int NR = kTailRows;
    const long long group = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / W;
    const int lw = threadIdx.x & (W - 1), g0 = lane() & ~(W - 1);
    uint32_t lo[NR], hi[NR], j0[NR];
    int v[NR];
    bool have[NR];
    unsigned long long vis[NR], need[NR], acc[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {  // the row's id and bounds come in one record
        have[r] = group * NR + r < n;
        v[r] = 0;
        lo[r] = hi[r] = 0;
        if (have[r]) {
            const ShortRow row = rows[group * NR + r];
            v[r] = row.row;
            lo[r] = row.begin;
            hi[r] = row.end;
        }
    }
    int s_next[NR], rel_next[NR];  // subject (and relation) ids of the next W entries, loaded one stage ahead
#pragma unroll
    for (int r = 0; r < NR; ++r) {  // what has reached the row and the first entries are requested together
        vis[r] = need[r] = acc[r] = 0;
        s_next[r] = -1;
        rel_next[r] = 0;
        if (have[r]) {
            if (W < 16) vis[r] = visited[(size_t)v[r] * W + lw];
            if (lo[r] + lw < hi[r]) {
                s_next[r] = in_sub[lo[r] + lw];
                if (MASK) rel_next[r] = in_rel[lo[r] + lw];
            }
        }
    }
    const unsigned long long live_w = live[lw];
    if constexpr (W == 16) seen_words<NR>(seen, v, have, lw, vis);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        need[r] = (walk_exact ? ~0ull : ~vis[r]) & live_w;
        if (!have[r]) need[r] = 0;
        if (!group_any<W>(need[r] != 0)) hi[r] = lo[r];
        j0[r] = lo[r];
    }
    uint32_t row_end[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) row_end[r] = hi[r];
    long long n_edges = 0, n_lines = 0;
    auto any_open = [&]() {
        bool o = false;
#pragma unroll
        for (int r = 0; r < NR; ++r) o |= j0[r] < hi[r];
        return o;
    };
    while (any_open()) {
        int s[NR], rl[NR];
        bool cand[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const bool open = j0[r] < hi[r];
            s[r] = open ? s_next[r] : -1;
            rl[r] = rel_next[r];
            s_next[r] = -1;
            const uint32_t j = j0[r] + W + lw;
            if (open && j < hi[r]) {
                s_next[r] = in_sub[j];
                if (MASK) rel_next[r] = in_rel[j];
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
            cand[r] = s[r] >= 0 && (DENSE || ((act_prev[s[r] >> 5] >> (s[r] & 31)) & 1u));
        unsigned gm[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            gm[r] = group_ballot<W>(cand[r]);
            if (j0[r] < hi[r]) n_edges += min((uint32_t)W, hi[r] - j0[r]);
            n_lines += __popc(gm[r]);
        }
        auto any_candidate = [&]() {
            unsigned o = 0;
#pragma unroll
            for (int r = 0; r < NR; ++r) o |= gm[r];
            return o != 0;
        };
        constexpr int NL = kTailLines;
        while (any_candidate()) {  // two candidate lines of each row in flight
            int c[NR][NL];
            unsigned long long l[NR][NL], ok[NR][NL];
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int x = 0; x < NL; ++x) {
                    c[r][x] = -1;
                    if (gm[r]) {
                        c[r][x] = __ffs((int)gm[r]) - 1;
                        gm[r] &= gm[r] - 1;
                    }
                }
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int x = 0; x < NL; ++x) {
                    const int src = g0 + (c[r][x] < 0 ? 0 : c[r][x]);
                    const int sx = __shfl(s[r], src);
                    l[r][x] = ok[r][x] = 0;  // (put together behind all loads)
                    if (c[r][x] >= 0) l[r][x] = prev[(size_t)sx * W + lw];
                    if (MASK) {
                        const int rx = __shfl(rl[r], src);
                        if (c[r][x] >= 0) ok[r][x] = allow[(size_t)rx * W + lw];
                    }
                }
            if (MASK) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
#pragma unroll
                    for (int x = 0; x < NL; ++x) l[r][x] &= ok[r][x];
            }
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int x = 0; x < NL; ++x) acc[r] |= l[r][x];
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (j0[r] < hi[r]) {
                j0[r] += W;
                if (!group_any<W>((need[r] & ~acc[r]) != 0)) hi[r] = j0[r];  // nothing left to find in this row
            }
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const unsigned long long nw = acc[r] & need[r];
        if (row_end[r] > lo[r] && group_any<W>(nw != 0)) {
            cur[(size_t)v[r] * W + lw] = nw;
            if (W < 16) visited[(size_t)v[r] * W + lw] = vis[r] | nw;
            else if (seen.keep) visited[(size_t)v[r] * W + lw] |= nw;  // (read again: no register holds it through the row)
            if (lw == 0) atomicOr(&act_cur[v[r] >> 5], 1u << (v[r] & 31));
        }
    }
    if (STATS) {
        const bool lead = (lw == 0);
        long long n_rows = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) n_rows += (row_end[r] > lo[r]) ? 1 : 0;
        add_stats(stats, lead ? n_rows : 0, lead ? n_edges : 0, lead ? n_lines : 0);
    }
}

// One wavefront per segment (<= 1024 entries) of a longer object row.  A row
// with one segment is finished here; segments of a multi-segment row merge
// through atomicOr on level[h] and look at what the others have found so far
// to stop early; k_pull_finish then marks those rows active (and folds them into visited on planes that keep it).
template <int W, bool MASK, bool STATS, bool DENSE>
__global__ void __launch_bounds__(256)
k_pull_seg(const PullSegment *__restrict__ segs, long long n,
           const int32_t *__restrict__ in_sub, const uint16_t *__restrict__ in_rel,
           const unsigned long long *__restrict__ allow, const uint32_t *__restrict__ act_prev,
           const unsigned long long *__restrict__ prev, const unsigned long long *__restrict__ live,
           unsigned long long *visited, Seen seen, unsigned long long *cur, uint32_t *act_cur,
           unsigned long long *stats, int walk_exact) {
    __shared__ int queue_s[4][64];
    __shared__ uint16_t queue_r[4][64];
    long long item = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const bool have = item < n;  // wave-uniform
    const int lw = lane() & (W - 1);
    int v = 0;
    uint32_t lo = 0, hi = 0;
    bool multi = false;
    unsigned long long vis = 0, need = 0, acc = 0;
    if (have) {
        const PullSegment sg = segs[item];  // carries its bounds: no look-up in the offsets before the first loads
        v = sg.row;
        lo = sg.begin;
        hi = sg.end;
        multi = sg.multi != 0;
        if constexpr (W < 16) {
            vis = visited[(size_t)v * W + lw];
        } else {
            const int vs[1] = {v};
            const bool all[1] = {true};
            unsigned long long x[1];
            seen_words<1>(seen, vs, all, lw, x);
            vis = x[0];
        }
        need = (walk_exact ? ~0ull : ~vis) & live[lw];
        if (multi) need &= ~__atomic_load_n(&cur[(size_t)v * W + lw], __ATOMIC_RELAXED);
    }
    const bool work = wave_any(need != 0);
    long long n_edges = 0, n_lines = 0;
    unsigned long long a0 = 0, a1 = 0;
    if (work) {
        // software pipeline: ids of chunk i+2 and frontier bits of chunk i+1 are requested
        // before the lines of chunk i are gathered
        PullEdges e0 = pull_load_edges<MASK>(lo, hi, in_sub, in_rel);
        PullEdges e1 = pull_load_edges<MASK>(lo + 64, hi, in_sub, in_rel);
        // DENSE: nearly every subject is in the frontier, so the one-bit test (a 64-byte sector per
        // edge) is skipped and every edge's line is gathered: the line of an entity outside the frontier is zero
        bool c0 = DENSE ? e0.s >= 0 : pull_test(e0, act_prev);
        int it = 0;
        for (uint32_t j0 = lo; j0 < hi; j0 += 64, ++it) {
            PullEdges e2 = pull_load_edges<MASK>(j0 + 128, hi, in_sub, in_rel);
            const bool c1 = DENSE ? e1.s >= 0 : pull_test(e1, act_prev);
            n_lines += pull_gather<W, MASK>(e0, c0, prev, allow, a0, a1, queue_s[threadIdx.x >> 6], queue_r[threadIdx.x >> 6]);
            n_edges += min((uint32_t)64, hi - j0);
            e0 = e1;
            c0 = c1;
            e1 = e2;
            // Early exit: behind the first two chunks, which of a row in pull_sub's order hold what most queries have
            // reached, then rarely: every fourth.
            if ((it & 3) == 3 || (!MASK && it < 2)) {
                acc = fold_gathered<W>(a0, a1);
                if (multi) acc |= __atomic_load_n(&cur[(size_t)v * W + lw], __ATOMIC_RELAXED);
                if (!wave_any((need & ~acc) != 0)) break;
            }
        }
        acc |= fold_gathered<W>(a0, a1);
        unsigned long long nb = acc & need;
        if (wave_any(nb != 0)) {
            if (!multi) {
                if (lane() < W) {
                    cur[(size_t)v * W + lane()] = nb;
                    if (W < 16) visited[(size_t)v * W + lane()] = vis | nb;
                    else if (seen.keep) visited[(size_t)v * W + lane()] |= nb;
                }
                if (lane() == 0) atomicOr(&act_cur[v >> 5], 1u << (v & 31));
            } else if (lane() < W && nb) {
                atomicOr(&cur[(size_t)v * W + lane()], nb);
            }
        }
    }
    if (STATS) {
        bool lead = lane() == 0;
        add_stats(stats, (lead && work) ? 1 : 0, lead ? n_edges : 0, lead ? n_lines : 0);
    }
}

// Rows that were expanded by several segments: mark active, and where the plane is kept visited |= level[h].
template <int W>
__global__ void __launch_bounds__(256)
k_pull_finish(const int32_t *__restrict__ rows, long long n, unsigned long long *visited,
              const unsigned long long *__restrict__ cur, uint32_t *act_cur, bool keep) {
    long long gidx = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / W;
    const int lw = threadIdx.x & (W - 1);
    unsigned long long c = 0;
    int v = 0;
    if (gidx < n) {
        v = rows[gidx];
        c = cur[(size_t)v * W + lw];
    }
    if (group_any<W>(c != 0)) {
        if (keep) visited[(size_t)v * W + lw] |= c;
        if (lw == 0) atomicOr(&act_cur[v >> 5], 1u << (v & 31));
    }
}

// ---- narrow planes (one and four words): lane = entry.  A lane loads the whole line of a subject (8 or 32 bytes), so the
// entries of a row need no hand-over between lanes; a wavefront takes a segment of a long row, eight lanes a short one,
// and the words are put together at the end.  Long and short rows share one launch, a row of several segments is merged
// through atomics on the level and on visited, and the census behind the hop makes the bitmap: no other kernel follows.
// What bounds it is the chain of loads of a row (record, visited and ids, lines) with everything in the caches, so
// each lane keeps several entries in flight.  One-word lines are gathered without asking for the frontier bit first,
// whatever the frontier's size: the bit costs as much as the line, which is zero outside the level.
// (Two hops on 3.4M triples, us, three kernels as for 16-word planes against this one: one question 60 -> 22, 8 walk-exact
// ones 90 -> 34, 200 questions with whitelists 125 -> 60.)
// acc |= the lines of entries j, j + step, .. (U of them, those below hi)
template <int W, int U, bool MASK>
__device__ __forceinline__ void pull_entries(bool dense, uint32_t j, uint32_t step, uint32_t hi,
                                             const int32_t *__restrict__ in_sub, const uint16_t *__restrict__ in_rel, const unsigned long long *__restrict__ allow,
                                             const uint32_t *__restrict__ act_prev,
                                             const unsigned long long *__restrict__ prev, unsigned long long (&acc)[W]) {
    int s[U], r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t at = j + (uint32_t)u * step;
        s[u] = -1;
        r[u] = 0;
        if (at < hi) {
            s[u] = in_sub[at];
            if (MASK) r[u] = in_rel[at];
        }
    }
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) on[u] = s[u] >= 0;
    if (W > 1 && !dense) {  // (wavefront-uniform)
#pragma unroll
        for (int u = 0; u < U; ++u) on[u] = on[u] && ((act_prev[s[u] >> 5] >> (s[u] & 31)) & 1u);
    }
    unsigned long long l[U][W];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int w = 0; w < W; ++w) l[u][w] = 0;
        if (on[u]) {
            load_line<W>(l[u], prev + (size_t)s[u] * W);
            if (MASK) {
                unsigned long long m[W];
                load_line<W>(m, allow + (size_t)r[u] * W);
#pragma unroll
                for (int w = 0; w < W; ++w) l[u][w] &= m[w];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w] |= l[u][w];
}

// word lane % W of the OR over a group of G lanes
template <int W, int G>
__device__ __forceinline__ unsigned long long group_or_words(const unsigned long long (&x)[W]) {
    unsigned long long r = x[0];
    if constexpr (W == 4) {
        const bool hi = lane() & 2, odd = lane() & 1;
        const unsigned long long a = (hi ? x[2] : x[0]) | shfl_xor64(hi ? x[0] : x[2], 2);
        const unsigned long long b = (hi ? x[3] : x[1]) | shfl_xor64(hi ? x[1] : x[3], 2);
        r = (odd ? b : a) | shfl_xor64(odd ? a : b, 1);
    }
#pragma unroll
    for (int m = W; m < G; m <<= 1) r |= shfl_xor64(r, m);
    return r;
}

// Entries per lane and step, and the lanes of a short row.  Hops of one question / of 8 walk-exact ones / of 200 questions
// with whitelists on 3.4M triples, us for two hops: eight lanes and two entries 22 / 34 / 60, four lanes and four
// entries 23 / 36 / 63, one lane and eight entries (W lanes on four words) 35 / 62 / 69: a lane per row is too few wavefronts.
constexpr int kSegEntries = 4, kTailEntries = 2, kNarrowTailLanes = 8;

// go: NULL, or what the census in front has decided (a hop launched before the host knows; see narrow_hops)
template <int W, bool MASK>
__global__ void __launch_bounds__(256)
k_pull_narrow(const PullSegment *__restrict__ segs, long long n_seg, unsigned seg_blocks, const ShortRow *__restrict__ rows,
              long long n_rows, const int32_t *__restrict__ in_sub, const uint16_t *__restrict__ in_rel,
              const unsigned long long *__restrict__ allow, const uint32_t *__restrict__ act_prev,
              const unsigned long long *__restrict__ prev, const unsigned long long *__restrict__ live,
              unsigned long long *visited, unsigned long long *cur, int walk_exact, bool dense,
              const unsigned long long *go) {
    if (go) {
        const unsigned long long form = *go;
        if (form == kHopNotPulled) return;
        dense = form == kHopPulledDense;
    }
    if (blockIdx.x < seg_blocks) {  // block-uniform: the segments first, they take longest
        const long long item = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
        if (item >= n_seg) return;  // wavefront-uniform
        const PullSegment sg = segs[item];
        const bool multi = sg.multi != 0;
        const size_t mine = (size_t)sg.row * W + own_word<W>();
        const unsigned long long vis = visited[mine], need = (walk_exact ? ~0ull : ~vis) & live[own_word<W>()];
        if (!wave_any(need != 0)) return;
        unsigned long long acc[W] = {}, nw = 0;
        for (uint32_t j0 = sg.begin; j0 < sg.end; j0 += 64 * kSegEntries) {
            pull_entries<W, kSegEntries, MASK>(dense, j0 + lane(), 64, sg.end, in_sub, in_rel, allow, act_prev, prev, acc);
            nw = wave_or_words<W>(acc) & need;
            if (!wave_any((need & ~nw) != 0)) break;
        }
        // The segments of a row end about together, and their atomics wait for each other: only what is still missing.
        // (One that read visited when others had added theirs leaves those bits out: they are in the level already.)
        if (multi && wave_any(nw != 0)) nw &= ~__hip_atomic_load(&cur[mine], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((lane() & (64 / W - 1)) != 0 || !wave_any(nw != 0)) return;
        if (!multi) {
            cur[mine] = nw;
            visited[mine] = vis | nw;
        } else if (nw) {
            atomicOr(&cur[mine], nw);
            atomicOr(&visited[mine], nw);
        }
        return;
    }
    constexpr int G = kNarrowTailLanes, U = kTailEntries;
    const long long group = ((long long)(blockIdx.x - seg_blocks) * 256 + threadIdx.x) / G;
    if (group >= n_rows) return;  // the lanes of a group together
    const int lg = threadIdx.x & (G - 1);
    const ShortRow row = rows[group];
    const size_t mine = (size_t)row.row * W + (lg & (W - 1));
    const unsigned long long vis = visited[mine], need = (walk_exact ? ~0ull : ~vis) & live[lg & (W - 1)];
    if (!group_any<G>(need != 0)) return;
    unsigned long long acc[W] = {}, found = 0;
    for (uint32_t j0 = row.begin; j0 < row.end; j0 += U * G) {
        pull_entries<W, U, MASK>(dense, j0 + lg, G, row.end, in_sub, in_rel, allow, act_prev, prev, acc);
        found = group_or_words<W, G>(acc);
        if (!group_any<G>((need & ~found) != 0)) break;
    }
    const unsigned long long nw = found & need;
    if (lg >= W || !group_any<W>(nw != 0)) return;
    cur[mine] = nw;
    visited[mine] = vis | nw;
}

// ---------------------------------------------------------------- planes back to zero
// A finished result's planes are zero except in the lines of entities that have their bit in some
// level's active bitmap: when the result is released those lines (of the level and of visited) and
// the bitmaps are cleared, so that the next call that gets the block starts from zeros without a
// fill of all k + 2 planes.  One wavefront per 64 entities, 16 bytes per lane (0.9M lines of three levels and as many of
// visited: 78 us, 100 with 8 bytes).
// (vis_levels: visited holds something only where one of the first so many levels does)
template <int W>
__global__ void __launch_bounds__(256)
k_sparse_clear(long long Epad, int levels, int vis_levels, uint32_t *act, long long actw, unsigned long long *visited,
               unsigned long long *level_planes, long long plane, unsigned long long *live) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < levels * (16 + kLevelCounters); i += blockDim.x) live[i] = 0ull;  // (and the counters behind them)
    const long long base = ((long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
    if (base >= Epad) return;  // Epad is a multiple of 64
    constexpr int L = W > 1 ? W / 2 : 1, GPW = 64 / L;  // lanes per line (16 bytes each), lines per store
    const int g = lane() / L, l = lane() & (L - 1);
    unsigned long long any = 0;
    for (int h = 0; h <= levels; ++h) {  // the levels, then visited with the union of their bits
        unsigned long long m = any;
        unsigned long long *dst = visited;
        if (h < levels) {
            uint32_t *a = act + (size_t)h * actw + base / 32;
            m = ((unsigned long long)a[1] << 32) | (unsigned long long)a[0];
            any |= h < vis_levels ? m : 0ull;
            dst = level_planes + (size_t)h * plane;
            if (m && lane() < 2) a[lane()] = 0u;
        }
        if (m == 0) continue;
#pragma unroll
        for (int i = 0; i < 64 / GPW; ++i) {
            const int e = i * GPW + g;
            if (!((m >> e) & 1ull)) continue;
            unsigned long long *x = dst + ((size_t)base + e) * W;
            if constexpr (W == 1) *x = 0ull;
            else reinterpret_cast<ulonglong2 *>(x)[l] = make_ulonglong2(0ull, 0ull);
        }
    }
}

// visited = the OR of the first n levels, on the lines of entities that are active in one of them.  Every line is written
// whole and from the levels alone: one that runs again beside a reader of the plane changes nothing.
__global__ void __launch_bounds__(256)
k_fold_visited(long long Epad, int n, const uint32_t *__restrict__ act, long long actw, const unsigned long long *__restrict__ levels,
               long long plane, unsigned long long *visited) {
    const long long base = ((long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
    if (base >= Epad) return;  // Epad is a multiple of 64
    const int g = lane() >> 3, l = lane() & 7;  // eight lanes of 16 bytes per line
    unsigned long long any = 0;
    for (int h = 0; h < n; ++h) any |= *reinterpret_cast<const unsigned long long *>(act + (size_t)h * actw + base / 32);
    if (any == 0) return;
    ulonglong2 x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = make_ulonglong2(0ull, 0ull);
    for (int h = 0; h < n; ++h) {
        const unsigned long long m = *reinterpret_cast<const unsigned long long *>(act + (size_t)h * actw + base / 32);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (!((m >> (8 * i + g)) & 1ull)) continue;
            const ulonglong2 y = reinterpret_cast<const ulonglong2 *>(levels + (size_t)h * plane + ((size_t)base + 8 * i + g) * 16)[l];
            x[i].x |= y.x;
            x[i].y |= y.y;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((any >> (8 * i + g)) & 1ull) reinterpret_cast<ulonglong2 *>(visited + ((size_t)base + 8 * i + g) * 16)[l] = x[i];
}

// ---------------------------------------------------------------- host side
static inline unsigned blocks_for(long long threads, int block) {
    return (unsigned)((threads + block - 1) / block);
}

// Most triples that may leave the frontier of hop h where it pushes (direction by rule).  A twelfth of all where a pulled hop is three
// kernels over whole lines.  On planes of one and four words it is one kernel over the graph, against two launches more and
// what the frontier's triples cost for a push.  us of a search of one hop, 200 questions on concept graphs, pushed / pulled, by
// triples in the frontier:
//    triples     without whitelists                                                     with them
//      0.3M      66:  87 /  72    1,001:  94 /  77    10,013: 110 /  90    30,000: 145 / 108      66:  91 /  75    30,000: 127 / 118
//      0.8M      31:  84 /  72    1,021:  96 /  76    10,014: 113 /  89   100,069: 272 / 180      31:  85 /  75   100,069: 199 / 188
//      1.6M      59:  85 /  77    1,003:  98 /  80    10,005: 114 /  94   100,000: 265 / 190      59:  88 /  81   100,000: 203 / 198
//      3.4M      56:  88 /  85    1,000:  98 /  88    10,011: 113 / 100   100,019: 272 / 204      56:  90 / 100   100,019: 209 / 215
//      3.4M hub   4:  85 /  93    1,029: 103 /  98    10,027: 110 / 110   100,001: 257 / 222       4:  89 / 110   100,001: 232 / 235
//        6M       2:  92 /  99    1,000: 105 / 102    10,000: 113 / 113   100,008: 248 / 209       2:  99 / 116   100,008: 206 / 215
//       10M       4: 104 / 118    1,019: 111 / 120    30,005: 149 / 153   100,008: 250 / 230       4: 105 / 141   100,008: 218 / 243
// Without whitelists the line is the square of the graph's triples over 2^30, at or behind the crossings (30M: 700,000 ..
// 900,000).  With them only four-word planes pull earlier: up to kMaskedPullTriples every frontier gains, from there to twice as
// many a hop that is not the last, whose successor is then launched ahead of the host's turn (three hops on 3.4M, 7,107 triples
// in the first frontier: 338 us pushed, 333 pulled), unless its frontier is next to nothing.  Below kFewTriples
// one-word searches hardly leave k_small_search; four-word ones would gain as at 0.3M.
constexpr long long kFewTriples = 1 << 18, kMaskedPullTriples = 1 << 21, kMaskedPullEdges = 1024;

static long long push_most(const logoskg_graph *g, const logoskg_result *r, int h) {
    const long long T = g->T, twelfth = T / 12;
    if (r->W == 16 || g->num_shards > 1 || T < kFewTriples) return twelfth;
    if (r->has_mask && (r->W == 1 || T > 2 * kMaskedPullTriples)) return twelfth;
    if (r->has_mask) return T <= kMaskedPullTriples ? 0 : h < r->k ? kMaskedPullEdges : twelfth;
    return std::min(twelfth, T * T >> 30);  // (T < 2^31)
}

static unsigned long long *level_counters(const logoskg_result *r, int h) {
    return r->live + (size_t)16 * (r->k + 1) + (size_t)kLevelCounters * h;
}

// A search on 16-word planes whose hops keep visited, as those on narrow planes do: one of many hops (hop h of the others asks up
// to h levels, and so does the count), one on planes that stay in the L2s (visited 32 MB, 4 MB for walk-exact ones, which ask
// for nothing), and one on a graph whose last result was asked for the plane, which would be made from the levels each time.
// us of a search of 1,024 queries, without / with it:
//    30M triples, 3M entities       k = 2:   471 /   533    3:   812 /   859    4: 1,210 / 1,189    5: 1,453 / 1,317    8: 1,696 / 1,444
//    hub-heavy 20M, 2M entities     k = 2:   913 / 1,067    3: 1,425 / 1,512    4: 2,011 / 1,958    5: 2,663 / 2,392    8: 3,499 / 2,860
//    under whitelists               k = 2: 1,033 / 1,196    3: 1,706 / 1,842    4: 2,435 / 2,464    5: 3,137 / 2,965    8: 4,721 / 3,730
//    with lists, 1M entities        k = 2:   777 /   800    3: 1,206 / 1,225    4: 1,436 / 1,427    407,000:  3: 680 / 682    4: 764 / 766
//    200,000 entities               k = 2:   387 /   391    3:   500 /   494    4:   571 /   561    20,000:   3: 208 / 188    4: 270 / 244
//    walk-exact, 3M                 k = 3:   752 /   860    6: 1,672 / 1,836    100,000: 3: 190 / 211    20,000: 3: 164 / 162    6: 262 / 249
constexpr int kSeenMaxK = 4;
constexpr long long kSeenMinEntities = 1 << 18, kSeenMinWalkEntities = 1 << 15;

static bool keeps_visited(const logoskg_graph *g, const logoskg_result *r) {
    if (r->W != 16) return false;
    if (g->visited_asked) return true;
    return r->walk_exact ? r->Epad < kSeenMinWalkEntities : r->k > kSeenMaxK || r->Epad < kSeenMinEntities;
}

Seen seen_levels(const logoskg_result *r, int upto) {
    const int have = std::min(r->vis_levels.load(), upto);
    const int gate = r->keep_visited || have > kSeenGate ? 0 : have;
    return Seen{have ? r->visited : nullptr, r->levels, r->act, r->Epad * (long long)r->W, r->Epad / 32, gate, have, upto, false, r->keep_visited};
}

static logoskg_status launch_fold(logoskg_result *r, int upto, hipStream_t st) {
    ProfScope ps(r->g->prof, KK_UPDATE, st);
    if (r->vis_dirty.load() < upto) r->vis_dirty.store(upto);
    k_fold_visited<<<dim3(blocks_for(r->Epad / 64, 4)), dim3(256), 0, st>>>(r->Epad, upto, r->act, r->Epad / 32, r->levels,
                                                                          r->Epad * 16, r->visited);
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

logoskg_status fold_visited(logoskg_result *r, int upto, hipStream_t st) {
    if (r->W != 16 || r->vis_levels.load() >= upto) return LOGOSKG_OK;
    LKG_TRY(launch_fold(r, upto, st));
    r->vis_levels.store(upto);
    return LOGOSKG_OK;
}

bool visited_by_search(const logoskg_result *r) { return r->W != 16 || r->vis_levels.load() >= r->n_levels; }

// vis_levels stays where the search left it: what tells later calls that the plane is whole is the event, for which their
// streams wait.  A launch that a capture records has not run and cannot wait for what ran outside: every such call folds.
logoskg_status share_visited(logoskg_result *r, hipStream_t st) {
    if (visited_by_search(r)) return LOGOSKG_OK;
    if (captured(st)) return launch_fold(r, r->n_levels, st);
    std::lock_guard<std::mutex> lock(r->vis_mutex);
    if (r->vis_made) {
        LKG_HIP(hipStreamWaitEvent(st, r->vis_made, 0));
        return LOGOSKG_OK;
    }
    LKG_TRY(launch_fold(r, r->n_levels, st));
    hipEvent_t made = nullptr;  // (without one the next call folds again, the same values)
    if (hipEventCreateWithFlags(&made, hipEventDisableTiming) == hipSuccess && hipEventRecord(made, st) == hipSuccess) r->vis_made = made;
    else {
        (void)hipGetLastError();
        if (made) (void)hipEventDestroy(made);
    }
    return LOGOSKG_OK;
}

// The same for the host, on a helper stream: the search has ended.  Callers may be recording a sequence meanwhile, to which
// nothing of this belongs and which a wait would end in the runtime's usual mode; a recorded fetch may have drawn the
// helper streams into it.
static logoskg_status finish_visited(logoskg_result *r) {
    LKG_HIP(hipSetDevice(r->g->device));
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    LKG_HIP(hipThreadExchangeStreamCaptureMode(&mode));
    hipStream_t st = r->g->side[0];
    if (captured(st)) st = helper_stream(r->g->device, 3);
    logoskg_status s = LOGOSKG_EDEVICE;
    if (!st) set_error("could not create a helper stream");
    else s = share_visited(r, st);
    const hipError_t e = s == LOGOSKG_OK ? hipStreamSynchronize(st) : hipSuccess;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    LKG_TRY(s);
    LKG_HIP(e);
    return LOGOSKG_OK;
}

template <int W, bool MASK>
static void launch_push(logoskg_graph *g, logoskg_result *r, int h, const unsigned long long *hc,
                        const int32_t *obj, const uint16_t *rel, bool update, const int32_t *list_tail,
                        const RowSegment *list_seg, const unsigned long long *ctr, hipStream_t st) {
    const size_t plane = (size_t)r->Epad * W;
    const unsigned long long *prev = r->levels + plane * (h - 1);
    unsigned long long *cur = r->levels + plane * h;
    uint32_t *act_cur = r->act + (size_t)(r->Epad / 32) * h;
    long long nt = (long long)hc[C_NTAIL], ns = (long long)hc[C_NSEG];
    const unsigned long long *known = r->walk_exact ? cur : h == 1 ? nullptr : r->visited;
    if (ns > 0) {
        ProfScope ps(g->prof, KK_PUSH_SEG, st);
        k_push_seg<W, MASK><<<dim3(blocks_for(ns, 4)), dim3(256), 0, st>>>(
            list_seg, ctr, g->out_off, g->row_begin, obj, rel, r->allow, prev, known, cur, act_cur);
        g->prof.acc[KK_PUSH_SEG].units[0] += g->prof.on ? ns : 0;
    }
    if (nt > 0) {
        ProfScope ps(g->prof, KK_PUSH_TAIL, st);
        constexpr int G = push_tail_lanes<W>();
        launch_ranges(nt, 256 / G, [&](long long first, long long n) {
            k_push_tail<W, MASK><<<dim3(blocks_for(n * G, 256)), dim3(256), 0, st>>>(
                list_tail, first, ctr, g->out_off, g->row_begin, obj, rel, r->allow, prev, known, cur, act_cur);
        });
        g->prof.acc[KK_PUSH_TAIL].units[0] += g->prof.on ? nt : 0;
    }
    const bool keep = W < 16 || r->keep_visited;
    if (!update || (!keep && r->walk_exact)) return;  // (walk-exact levels ask for nothing that was reached)
    ProfScope ps(g->prof, KK_UPDATE, st);
    const dim3 grid(blocks_for(r->Epad / 64, 4)), block(256);
    if (!keep && !known) {
        k_drop_seeds<<<dim3(blocks_for((long long)(r->Epad / 64), 256)), block, 0, st>>>(r->Epad / 64, r->act, act_cur, r->levels, cur);
        return;
    }
    if (known) k_update_visited<W, false><<<grid, block, 0, st>>>(r->Epad, act_cur, cur, r->visited);
    else k_update_visited<W, true><<<grid, block, 0, st>>>(r->Epad, act_cur, cur, r->visited);
}

// STATS: the counting mode runs instantiations of its own, so that kernel statistics of the
// ordinary ones are not mixed with it.
// When most triples leave the frontier the kernels gather every edge's line without asking for
// its frontier bit first (never in the counting mode: its statistics count frontier lines).
static inline bool dense_pull(const logoskg_graph *g, const unsigned long long *hc, bool want_stats) {
    return !want_stats && dense_rule((long long)hc[C_FEDGES], g->T);
}

// live[h-1] of 16-word planes: the queries this hop can still reach something for (once per hop; of a dense one by the census).
static void launch_live(logoskg_graph *g, logoskg_result *r, int h, hipStream_t st) {
    const size_t plane = (size_t)r->Epad * 16;
    ProfScope ps(g->prof, KK_LIVE, st);
    unsigned nb = std::min<unsigned>(2048u, std::max(1u, blocks_for(g->E, 256)));
    unsigned long long *live = r->live + (size_t)16 * (h - 1);
    k_live<16><<<dim3(nb), dim3(256), 0, st>>>(r->act + (size_t)(r->Epad / 32) * (h - 1), g->E, g->out_off,
                                               r->levels + plane * (h - 1), live);
}

// Pull over the object rows of the work lists `rc`, whose entries index in_sub / in_rel (the whole
// object-sorted CSR of a resident graph, or one object range of a sharded one in a cache slot).
template <int W, bool MASK, bool STATS>
static void launch_pull_rows(logoskg_graph *g, logoskg_result *r, int h, const RowClasses &rc, const int32_t *in_sub,
                             const uint16_t *in_rel, bool dense, const unsigned long long *go, hipStream_t st) {
    const size_t plane = (size_t)r->Epad * W;
    const unsigned long long *prev = r->levels + plane * (h - 1);
    unsigned long long *cur = r->levels + plane * h;
    const uint32_t *act_prev = r->act + (size_t)(r->Epad / 32) * (h - 1);
    uint32_t *act_cur = r->act + (size_t)(r->Epad / 32) * h;
    const unsigned long long *live = r->live + (size_t)16 * (h - 1);
    auto stats = [&](int kind) { return STATS ? g->d_ctr + C_STATS + 4 * kind : nullptr; };
    const int walk = r->walk_exact ? 1 : 0;
    Seen seen = W == 16 && (!walk || r->keep_visited) ? seen_levels(r, h) : Seen{};
    seen.sure = h > 1 && 2 * r->stats[(size_t)h - 2].entities_reached > (long long)(g->in_rows.n_tail + g->in_rows.n_long);
    if constexpr (W <= 4 && !STATS) {
        if (rc.n_seg + rc.n_tail == 0) return;
        ProfScope ps(g->prof, KK_PULL_TAIL, st);
        constexpr int rows_per_block = 256 / kNarrowTailLanes;
        auto launch = [&](long long n_seg, long long first, long long n_rows) {
            const unsigned seg_blocks = blocks_for(n_seg, 4);
            const dim3 grid(seg_blocks + blocks_for(n_rows, rows_per_block)), block(256);
            k_pull_narrow<W, MASK><<<grid, block, 0, st>>>(rc.seg, n_seg, seg_blocks, rc.tail + first, n_rows, in_sub, in_rel,
                                                           r->allow, act_prev, prev, live, r->visited, cur, walk, dense, go);
        };
        if ((rc.n_seg + 3) / 4 + (rc.n_tail + rows_per_block - 1) / rows_per_block <= kMaxBlocks) {
            launch(rc.n_seg, 0, rc.n_tail);
        } else {  // (as many segments as triple indices allow fit one launch)
            if (rc.n_seg > 0) launch(rc.n_seg, 0, 0);
            launch_ranges(rc.n_tail, rows_per_block, [&](long long first, long long n) { launch(0, first, n); });
        }
        return;
    } else {
    if (rc.n_seg > 0) {
        ProfScope ps(g->prof, KK_PULL_SEG, st);
        const dim3 grid(blocks_for(rc.n_seg, 4)), block(256);
        if (dense)
            k_pull_seg<W, MASK, STATS, true><<<grid, block, 0, st>>>(rc.seg, rc.n_seg, in_sub, in_rel,
                                                                     r->allow, act_prev, prev, live, r->visited, seen, cur,
                                                                     act_cur, stats(KK_PULL_SEG), walk);
        else
            k_pull_seg<W, MASK, STATS, false><<<grid, block, 0, st>>>(rc.seg, rc.n_seg, in_sub, in_rel,
                                                                      r->allow, act_prev, prev, live, r->visited, seen, cur,
                                                                      act_cur, stats(KK_PULL_SEG), walk);
    }
    if (rc.n_tail > 0) {
        ProfScope ps(g->prof, KK_PULL_TAIL, st);
        const long long groups = (rc.n_tail + kTailRows - 1) / kTailRows;
        const dim3 grid(blocks_for(groups * W, 256)), block(256);
        if (dense)
            k_pull_tail<W, MASK, STATS, true><<<grid, block, 0, st>>>(rc.tail, rc.n_tail, in_sub, in_rel, r->allow,
                                                                      act_prev, prev, live, r->visited, seen, cur, act_cur,
                                                                      stats(KK_PULL_TAIL), walk);
        else
            k_pull_tail<W, MASK, STATS, false><<<grid, block, 0, st>>>(rc.tail, rc.n_tail, in_sub, in_rel, r->allow,
                                                                       act_prev, prev, live, r->visited, seen, cur, act_cur,
                                                                       stats(KK_PULL_TAIL), walk);
    }
    if (rc.n_multi > 0) {
        ProfScope ps(g->prof, KK_PULL_FINISH, st);
        k_pull_finish<W><<<dim3(blocks_for(rc.n_multi * W, 256)), dim3(256), 0, st>>>(rc.multi, rc.n_multi,
                                                                                      r->visited, cur, act_cur, W < 16 || r->keep_visited);
    }
    }
}

template <int W>
static void pull_rows_w(logoskg_graph *g, logoskg_result *r, int h, const RowClasses &rc, const int32_t *in_sub,
                        const uint16_t *in_rel, bool dense, bool want_stats, hipStream_t st,
                        const unsigned long long *go = nullptr) {
    if (r->has_mask) {
        if (want_stats) launch_pull_rows<W, true, true>(g, r, h, rc, in_sub, in_rel, dense, go, st);
        else launch_pull_rows<W, true, false>(g, r, h, rc, in_sub, in_rel, dense, go, st);
    } else {
        if (want_stats) launch_pull_rows<W, false, true>(g, r, h, rc, in_sub, in_rel, dense, go, st);
        else launch_pull_rows<W, false, false>(g, r, h, rc, in_sub, in_rel, dense, go, st);
    }
}

// One object range of a pull hop (a sharded graph visits them one after the other; `first`: the
// live words of the hop are computed before the range).
void launch_pull_range(logoskg_graph *g, logoskg_result *r, int h, const RowClasses &rc, const int32_t *in_sub,
                       const uint16_t *in_rel, const unsigned long long *hc, bool want_stats, bool first,
                       hipStream_t st) {
    const bool dense = dense_pull(g, hc, want_stats);
    switch (r->W) {
        case 1:
            pull_rows_w<1>(g, r, h, rc, in_sub, in_rel, dense, want_stats, st);
            break;
        case 4:
            pull_rows_w<4>(g, r, h, rc, in_sub, in_rel, dense, want_stats, st);
            break;
        default:
            if (first && !dense) launch_live(g, r, h, st);
            pull_rows_w<16>(g, r, h, rc, in_sub, in_rel, dense, want_stats, st);
            break;
    }
}

// What a pulled hop of a resident graph walks: the distinct pairs, under whitelists all triples, both with the subjects that
// most queries have reached first (where the graph has them so).
struct PullArrays {
    const RowClasses &rows;
    const int32_t *sub;
    const uint16_t *rel;
};

static PullArrays pull_arrays(const logoskg_graph *g, const logoskg_result *r) {
    if (!g->pairs.off) return {g->in_rows, g->in_sub, g->in_rel};
    if (r->has_mask) return {g->in_rows, g->pairs.all_sub, g->pairs.all_rel};
    return {g->pairs.rows, g->pairs.pull_sub, nullptr};
}

template <int W>
static void run_hop(logoskg_graph *g, logoskg_result *r, int h, bool pull, bool want_stats,
                    const unsigned long long *hc, hipStream_t st) {
    if (pull) {
        const PullArrays p = pull_arrays(g, r);
        launch_pull_range(g, r, h, p.rows, p.sub, p.rel, hc, want_stats, true, st);
    } else {
        if (r->has_mask) launch_push<W, true>(g, r, h, hc, g->out_obj, g->out_rel, true, g->fr_tail, g->fr_seg, level_counters(r, h - 1), st);
        else launch_push<W, false>(g, r, h, hc, g->out_obj, g->out_rel, true, g->fr_tail, g->fr_seg, level_counters(r, h - 1), st);
    }
}

// Push of prepared work lists (short rows, segments; ctr[0], ctr[1] = their lengths on the
// device), reading the edge arrays through the given base pointers (a shard slot, shifted so
// that grouped edge indices apply).
void launch_push_lists(logoskg_graph *g, logoskg_result *r, int h, const unsigned long long *hc,
                       const int32_t *obj, const uint16_t *rel, bool update, const int32_t *list_tail,
                       const RowSegment *list_seg, const unsigned long long *ctr, hipStream_t st) {
    switch (r->W) {
        case 1:
            if (r->has_mask) launch_push<1, true>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            else launch_push<1, false>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            break;
        case 4:
            if (r->has_mask) launch_push<4, true>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            else launch_push<4, false>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            break;
        default:
            if (r->has_mask) launch_push<16, true>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            else launch_push<16, false>(g, r, h, hc, obj, rel, update, list_tail, list_seg, ctr, st);
            break;
    }
}

void launch_resident_hop(logoskg_graph *g, logoskg_result *r, int h, bool pull, bool want_stats,
                         const unsigned long long *hc, hipStream_t st) {
    switch (r->W) {
        case 1: run_hop<1>(g, r, h, pull, want_stats, hc, st); break;
        case 4: run_hop<4>(g, r, h, pull, want_stats, hc, st); break;
        default: run_hop<16>(g, r, h, pull, want_stats, hc, st); break;
    }
}

// A pulled hop of a resident graph on narrow planes, for the case that *go says so.
static void launch_pull_ahead(logoskg_graph *g, logoskg_result *r, int h, const unsigned long long *go, hipStream_t st) {
    const PullArrays p = pull_arrays(g, r);
    if (r->W == 1) pull_rows_w<1>(g, r, h, p.rows, p.sub, p.rel, false, false, st, go);
    else pull_rows_w<4>(g, r, h, p.rows, p.sub, p.rel, false, false, st, go);
}

__global__ void k_clear_cursors(unsigned long long *ctr) { ctr[threadIdx.x] = 0ull; }

// Push lists of level h into g->fr_tail / g->fr_seg.  ctr: two words that hold zeros (a level's own counters, once),
// or NULL for the graph's, which are cleared first.
logoskg_status census_lists(logoskg_graph *g, logoskg_result *r, int h, unsigned long long *ctr, hipStream_t st, int prof_kind) {
    if (!ctr) {
        ctr = g->d_ctr;
        // (a kernel: a fetch that a stream capture records comes by here, and a memset node that is not run again in
        // a later replay would let the lists grow past their ends)
        k_clear_cursors<<<dim3(1), dim3(2), 0, st>>>(ctr);
    }
    ProfScope ps(g->prof, prof_kind, st);
    const unsigned nb = std::min<unsigned>(512u, std::max(1u, blocks_for(g->E, 1024 * kCensusEntities)));
    k_census_lists<<<dim3(nb), dim3(1024), 0, st>>>(r->act + (size_t)(r->Epad / 32) * h, g->E, g->out_off, g->fr_tail,
                                                   g->fr_seg, ctr);
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

// Census of level h into `host` (pinned).  pulled: the level comes from the pull kernels; go: the hop in front was
// launched ahead, and so is this.
static logoskg_status launch_census(logoskg_graph *g, logoskg_result *r, int h, bool pulled, unsigned long long *host,
                                    const unsigned long long *go, hipStream_t st) {
    ProfScope ps(g->prof, KK_CENSUS, st);
    auto launch = [&](auto *kernel, int threads, int per_thread) {
        const unsigned nb = std::min<unsigned>(kCensusBlocks, std::max(1u, blocks_for(g->E, threads * per_thread)));
        kernel<<<dim3(nb), dim3((unsigned)threads), 0, st>>>(r->act + (size_t)(r->Epad / 32) * h, g->E, g->out_off,
                                                             level_counters(r, h), g->d_ctr + C_TOTAL, host,
                                                             r->levels + (size_t)r->Epad * r->W * h, r->live + (size_t)16 * h,
                                                             go, (long long)g->T, push_most(g, r, h + 1), g->prof.counters ? 0 : r->Q);
    };
    if (r->W == 16) launch(k_census<0, false>, 1024, kCensusEntities);
    else if (pulled) launch(r->W == 1 ? k_census<1, true> : k_census<4, true>, 512, 4);
    else launch(r->W == 1 ? k_census<1, false> : k_census<4, false>, 512, kCensusEntities);
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

// The counters that a census has written to `host`: waits for its word kCensusDone and not for the stream, behind whose
// census the next hop may be running.  After a few milliseconds the host stops polling and waits for the stream, which
// also ends where a launch failed.
constexpr int kCensusPolls = 1 << 18;  // some 10 ns each

static logoskg_status await_census(const unsigned long long *host, hipStream_t st) {
    auto done = [&]() { return __atomic_load_n(&host[kCensusDone], __ATOMIC_ACQUIRE) != 0; };
    for (int turn = 0; turn < kCensusPolls; ++turn) {
        if (done()) return LOGOSKG_OK;
        __builtin_ia32_pause();
    }
    LKG_HIP(hipStreamSynchronize(st));
    if (done()) return LOGOSKG_OK;
    set_error("the frontier census did not run");
    return LOGOSKG_EINTERNAL;
}

static unsigned long long *census_slot(logoskg_graph *g, int h) { return g->h_census + (h & 1) * kCensusSlot; }

// ... into g->h_ctr, when everything in front of it is done.  (Waiting for the word instead of the stream: the host is back
// and the next hop on its way while the census kernel ends.)
static logoskg_status census(logoskg_graph *g, logoskg_result *r, int h, bool pulled, hipStream_t st) {
    unsigned long long *host = census_slot(g, h);
    host[kCensusDone] = 0;
    LKG_TRY(launch_census(g, r, h, pulled, host, nullptr, st));
    if (g->prof.counters) {
        LKG_HIP(hipMemcpyAsync(g->h_ctr + C_STATS, g->d_ctr + C_STATS, 4 * KK_NUM * sizeof(unsigned long long),
                               hipMemcpyDeviceToHost, st));
        LKG_HIP(hipStreamSynchronize(st));
    }
    LKG_TRY(await_census(host, st));
    memcpy(g->h_ctr, host, C_STATS * sizeof(host[0]));
    return LOGOSKG_OK;
}

logoskg_status count_reached(logoskg_result *r, hipStream_t st);  // result.hip

// The hops of a narrow batch on a resident graph (direction by rule).  The host needs each level's counters to choose the
// next hop's direction, and on a graph of a few million triples a hop is 20 us of kernels, about what a wait, a
// launch and the GPU's way back to work take.  Behind a pulled hop, whose successor nearly always pulls as well, the next
// one is therefore launched before its turn is known: the census leaves its decision on the device (push_most, dense_rule:
// the host's own), and kernels launched ahead of a hop that is not pulled return at once (about 4 us).  The last level's
// counters, which only feed the statistics, are read behind the counts of the lists.  `pending`: that is still to be done.
static logoskg_status narrow_hops(logoskg_graph *g, logoskg_result *r, int first_hop, bool *pending, hipStream_t st) {
    unsigned long long hc[C_TOTAL] = {};
    memcpy(hc, g->h_ctr, C_STATS * sizeof(hc[0]));
    auto slot = [&](int h) { return census_slot(g, h); };
    bool running = false;  // hop h is on its way already
    for (int h = first_hop; h <= r->k; ++h) {
        logoskg_hop_stats &hs = r->stats[(size_t)h - 1];
        if (hc[C_NROWS] == 0) break;
        hs.active_rows = (long long)hc[C_NROWS];
        hs.frontier_edges = (long long)hc[C_FEDGES];
        hs.shards_touched = 1;
        const bool pull = hs.frontier_edges > push_most(g, r, h);
        hs.direction = pull ? LOGOSKG_DIR_PULL : LOGOSKG_DIR_PUSH;
        if (!pull) hs.edges_scanned = hs.lines_gathered = hs.frontier_edges;
        if (!running) {
            if (!pull) LKG_TRY(census_lists(g, r, h - 1, level_counters(r, h - 1), st));
            launch_resident_hop(g, r, h, pull, false, hc, st);
            LKG_HIP(hipGetLastError());
            slot(h)[kCensusDone] = 0;
            LKG_TRY(launch_census(g, r, h, pull, slot(h), nullptr, st));
        }
        const bool ahead = pull && h < r->k;
        if (ahead) {
            const unsigned long long *go = level_counters(r, h) + L_PULL;
            launch_pull_ahead(g, r, h + 1, go, st);
            LKG_HIP(hipGetLastError());
            slot(h + 1)[kCensusDone] = 0;
            LKG_TRY(launch_census(g, r, h + 1, true, slot(h + 1), go, st));
        }
        if (h == r->k) {
            *pending = true;
            break;
        }
        LKG_TRY(await_census(slot(h), st));
        memcpy(hc, slot(h), C_STATS * sizeof(hc[0]));
        hs.entities_reached = (long long)hc[C_NACTIVE];
        running = ahead && (long long)hc[C_FEDGES] > push_most(g, r, h + 1);
    }
    return LOGOSKG_OK;
}

}  // namespace lkg

using namespace lkg;

extern "C" void logoskg_result_free(logoskg_result *r) {
    if (!r) return;
    logoskg_graph *g = r->g;
    (void)hipSetDevice(g->device);
    drop_walk_tables(r);
    // levels follows visited and live follows act in one allocation each
    void *ptrs[] = {r->visited, r->act, r->allow, r->seed_off, r->small_off, r->tile_base,
                    r->super_base, r->mega_base, r->d_reached_off, r->lvl_tile_base, r->lvl_super_base,
                    r->lvl_mega_base, r->d_level_off, r->trip_ent, r->trip_off,
                    r->trip_chunk_entry, r->trip_chunk_first, r->tile_ent, r->cpos, r->act_chunk};
    constexpr int n = (int)(sizeof(ptrs) / sizeof(ptrs[0]));
    bool zeroed[n] = {};
    const hipStream_t st = r->last_stream;
    if (r->vis_made) {
        if (hipStreamWaitEvent(st, r->vis_made, 0) != hipSuccess) (void)hipGetLastError();
        (void)hipEventDestroy(r->vis_made);
    }
    if (r->complete && r->visited && r->act) {  // hand the planes and the bitmaps back as zeros
        ProfScope ps(g->prof, KK_CLEAR, st);
        const long long plane = r->Epad * r->W, actw = r->Epad / 32;
        const dim3 grid(blocks_for(r->Epad / 64, 4)), block(256);
        const int vis = r->W == 16 ? r->vis_dirty.load() : r->k + 1;
        switch (r->W) {
            case 1: k_sparse_clear<1><<<grid, block, 0, st>>>(r->Epad, r->k + 1, vis, r->act, actw, r->visited, r->levels, plane, r->live); break;
            case 4: k_sparse_clear<4><<<grid, block, 0, st>>>(r->Epad, r->k + 1, vis, r->act, actw, r->visited, r->levels, plane, r->live); break;
            default: k_sparse_clear<16><<<grid, block, 0, st>>>(r->Epad, r->k + 1, vis, r->act, actw, r->visited, r->levels, plane, r->live); break;
        }
        if (hipGetLastError() == hipSuccess) zeroed[0] = zeroed[1] = true;
        if (g->prof.on && r->n_active > 0) g->prof.acc[KK_CLEAR].units[3] += (vis > r->k ? 2 : 1) * r->n_active * r->W;
    }
    // the blocks may still be in use by work on the stream of the result's last call
    g->pool.release_after(ptrs, zeroed, n, st);
    delete r;
}

extern "C" logoskg_status logoskg_khop(logoskg_graph *g, const logoskg_query_batch *b, logoskg_result **out) {
    if (!g || !b || !out) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    *out = nullptr;
    if (b->struct_size != sizeof(logoskg_query_batch)) {
        set_error("logoskg_query_batch.struct_size is %u, expected %zu", b->struct_size, sizeof(*b));
        return LOGOSKG_EINVAL;
    }
    if (b->num_queries < 1 || b->num_queries > LOGOSKG_MAX_QUERIES || b->k < 0 || b->k > LOGOSKG_MAX_K ||
        b->num_seeds < 0 || !b->seed_off || (b->num_seeds > 0 && !b->seeds)) {
        set_error("bad query batch: Q=%d k=%d num_seeds=%lld", b->num_queries, b->k, (long long)b->num_seeds);
        return LOGOSKG_EINVAL;
    }
    uint32_t dir = b->flags & LOGOSKG_DIR_MASK;
    const bool walk_exact = (b->flags & LOGOSKG_WALK_EXACT) != 0;
    if (dir == 3u) { set_error("bad direction flags"); return LOGOSKG_EINVAL; }
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)b->stream;

    logoskg_result *r = new (std::nothrow) logoskg_result();
    if (!r) { set_error("out of host memory"); return LOGOSKG_ENOMEM; }
    r->g = g;
    r->Q = b->num_queries;
    r->k = b->k;
    r->W = words_for_queries(r->Q);
    r->Epad = g->Epad;
    r->has_mask = b->rel_mask != nullptr;
    r->walk_exact = walk_exact;
    r->stats.assign((size_t)r->k, logoskg_hop_stats{});
    const int W = r->W, k = r->k;
    const size_t plane = (size_t)r->Epad * W;
    const size_t actw = (size_t)r->Epad / 32;
    logoskg_status s;
    // From the first census on a failed call ends with its stream idle, like one that succeeds: what is still queued
    // writes the graph's pinned words and would be taken for the next call's census.
    bool censused = false;
    auto fail = [&](logoskg_status e) {
        if (censused) (void)hipStreamSynchronize(st);
        logoskg_result_free(r);
        return e;
    };
    // visited and the level planes are one allocation, the active bitmaps, the live words and the levels'
    // counters another: each is cleared by one fill
    const size_t act_bytes = actw * 4 * (size_t)(k + 1), live_bytes = (size_t)(16 + kLevelCounters) * 8 * (size_t)(k + 1);
    r->last_stream = st;
    if (g->pairs.wanted) (void)give_up_pairs(g);
    bool planes_zero = false, act_zero = false;  // a block released by an earlier result comes back cleared
    if ((s = g->pool.alloc((void **)&r->visited, plane * 8 * (size_t)(k + 2), st, &planes_zero)) != LOGOSKG_OK) return fail(s);
    r->levels = r->visited + plane;
    if ((s = g->pool.alloc((void **)&r->act, act_bytes + live_bytes, st, &act_zero)) != LOGOSKG_OK) return fail(s);
    r->live = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(r->act) + act_bytes);
    if (r->has_mask && (s = g->pool.alloc((void **)&r->allow, (size_t)g->R * W * 8, st)) != LOGOSKG_OK) return fail(s);

    // (offsets, then the seeds)
    if ((s = g->pool.alloc((void **)&r->seed_off, ((size_t)r->Q + 1) * 8 + (size_t)b->num_seeds * 4, st)) != LOGOSKG_OK) return fail(s);
    r->seeds = reinterpret_cast<int32_t *>(r->seed_off + r->Q + 1);

#define KH(call)                                  \
    do {                                          \
        logoskg_status s2_ = [&]() -> logoskg_status { LKG_HIP(call); return LOGOSKG_OK; }(); \
        if (s2_ != LOGOSKG_OK) return fail(s2_);  \
    } while (0)

    {
        ProfScope ps(g->prof, KK_CLEAR, st);
        if (!planes_zero) {
            KH(hipMemsetAsync(r->visited, 0, plane * 8 * (size_t)(k + 2), st));
            g->prof.acc[KK_CLEAR].units[3] += g->prof.on ? (long long)(plane * (size_t)(k + 2)) : 0;
        }
        if (!act_zero) KH(hipMemsetAsync(r->act, 0, act_bytes + live_bytes, st));
    }
    // Up to 64 queries with few seeds: the first hops - all of them when the search stays small - run in one
    // launch (not where the caller asked for pulled hops or for the kernels' work counters).
    const bool want_stats = g->prof.counters;
    const bool want_counts = !(b->flags & LOGOSKG_NO_COUNTS);
    const bool small = W == 1 && g->num_shards <= 1 && !want_stats && dir != LOGOSKG_DIR_PULL &&
                       b->num_seeds <= kSmallEdges;
    if (r->has_mask) {
        ProfScope ps(g->prof, KK_SEED, st);
        const int rel_words = (g->R + 63) / 64;
        k_allow<<<dim3(blocks_for(rel_words * W, 4)), dim3(256), 0, st>>>(r->Q, g->R, W, rel_words,
                                                                          (const unsigned long long *)b->rel_mask,
                                                                          (unsigned long long *)r->allow);
    }
    int first_hop = 1;
    r->vis_levels = r->vis_dirty = W == 16 ? 1 : k + 1;  // the seeds
    r->keep_visited = keeps_visited(g, r);
    g->visited_asked = false;
    r->n_levels = 1;
    if (small && (s = small_search(g, r, b, want_counts, dir == LOGOSKG_DIR_PUSH, &first_hop, st)) != LOGOSKG_OK) return fail(s);
    if (!small) {
        g->prof.begin(KK_SEED, st);
        k_seed<<<dim3((r->Q + 255) / 256), dim3(256), 0, st>>>(r->Q, (long long)b->num_seeds,
                                                               (const long long *)b->seed_off, b->seeds, g->E, W,
                                                               (unsigned long long *)r->levels,
                                                               (unsigned long long *)r->visited, r->act, level_counters(r, 0),
                                                               r->seed_off, r->seeds);
        g->prof.end(st);
        KH(hipGetLastError());
        censused = true;
        if ((s = census(g, r, 0, false, st)) != LOGOSKG_OK) return fail(s);
        if (g->h_ctr[C_ERR]) {
            set_error("seed_off / seeds are inconsistent or out of range (device check, code %llu)", g->h_ctr[C_ERR]);
            return fail(LOGOSKG_EINVAL);
        }
    }
    const bool narrow = W <= 4 && g->num_shards <= 1 && !want_stats && dir == LOGOSKG_DIR_AUTO;
    bool pending = false;
    censused = true;
    if (narrow && (s = narrow_hops(g, r, first_hop, &pending, st)) != LOGOSKG_OK) return fail(s);
    for (int h = first_hop; !narrow && h <= k; ++h) {
        logoskg_hop_stats &hs = r->stats[h - 1];
        long long rows = (long long)g->h_ctr[C_NROWS];
        long long fedges = (long long)g->h_ctr[C_FEDGES];
        if (rows == 0) break;  // nothing can be reached any more: the remaining levels stay empty
        hs.active_rows = rows;
        hs.frontier_edges = fedges;
        const bool pull = dir == LOGOSKG_DIR_PULL || (dir == LOGOSKG_DIR_AUTO && fedges > push_most(g, r, h));
        hs.direction = pull ? LOGOSKG_DIR_PULL : LOGOSKG_DIR_PUSH;
        unsigned long long hc[C_TOTAL] = {};
        memcpy(hc, g->h_ctr, C_STATS * sizeof(hc[0]));
        if (W == 16 && !walk_exact && !pull && (s = fold_visited(r, h, st)) != LOGOSKG_OK) return fail(s);
        if (want_stats)
            KH(hipMemsetAsync(g->d_ctr + C_STATS, 0, 4 * KK_NUM * sizeof(unsigned long long), st));
        if (g->num_shards > 1) {
            // Alg. 1: the hop visits sub-graphs one after the other through the cache -- the
            // subject shards that hold a frontier row (push) or every object range (pull)
            if ((s = run_sharded_hop(g, r, h, pull, want_stats, hc, st, &hs)) != LOGOSKG_OK) return fail(s);
            KH(hipGetLastError());
        } else {
            hs.shards_touched = 1;
            if (!pull && (s = census_lists(g, r, h - 1, level_counters(r, h - 1), st)) != LOGOSKG_OK) return fail(s);
            launch_resident_hop(g, r, h, pull, want_stats, hc, st);
            KH(hipGetLastError());
        }
        r->n_levels = h + 1;
        if (W == 16 && (r->keep_visited || (!walk_exact && !pull && h > 1))) r->vis_levels = r->vis_dirty = h + 1;
        if (h == k && !want_stats) {  // (its counters only feed the statistics: read behind the counts)
            census_slot(g, h)[kCensusDone] = 0;
            if ((s = launch_census(g, r, h, pull, census_slot(g, h), nullptr, st)) != LOGOSKG_OK) return fail(s);
            pending = true;
        } else {
            if ((s = census(g, r, h, pull, st)) != LOGOSKG_OK) return fail(s);
            hs.entities_reached = (long long)g->h_ctr[C_NACTIVE];
        }
        if (hs.direction == LOGOSKG_DIR_PULL) {
            if (want_stats) for (int kind : {KK_PULL_TAIL, KK_PULL_SEG}) {
                const unsigned long long *c = g->h_ctr + C_STATS + 4 * kind;
                hs.rows_scanned += (long long)c[0];
                hs.edges_scanned += (long long)c[1];
                hs.lines_gathered += (long long)c[2];
                for (int u = 0; u < 3; ++u) g->prof.acc[kind].units[u] += (long long)c[u];
                // distinct frontier lines this kernel can have gathered
                g->prof.acc[kind].units[3] += std::min<long long>((long long)c[2], (long long)hs.active_rows);
            }
        } else {
            hs.edges_scanned = fedges;
            hs.lines_gathered = fedges;
        }
    }
    if (want_counts && !r->has_counts) {
        if ((s = count_reached(r, st)) != LOGOSKG_OK) return fail(s);
    }
    // Without counts nothing has waited for the stream yet: a census is polled while its kernel ends, and what the kernel's
    // other blocks have written (a pulled level's bitmap) other streams see behind its end only.
    if (!want_counts) KH(hipStreamSynchronize(st));
    if (pending) {
        const unsigned long long *host = census_slot(g, k);
        if ((s = await_census(host, st)) != LOGOSKG_OK) return fail(s);
        r->stats[(size_t)k - 1].entities_reached = (long long)host[C_NACTIVE];
    }
#undef KH
    r->complete = true;
    *out = r;
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_get_info(const logoskg_result *r, logoskg_result_info *o) {
    if (!r || !o) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    o->num_queries = r->Q;
    o->k = r->k;
    o->words_per_entity = r->W;
    o->num_levels = r->k + 1;
    o->padded_entities = r->Epad;
    if (r->W == 16) r->g->visited_asked = true;
    if (!visited_by_search(r)) LKG_TRY(finish_visited(const_cast<logoskg_result *>(r)));
    o->visited = (const uint64_t *)r->visited;
    o->levels = (const uint64_t *)r->levels;
    o->total_reached = r->has_counts ? r->reached_off.back() : -1;
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_hop_stats(const logoskg_result *r, logoskg_hop_stats *o) {
    if (!r || (r->k > 0 && !o)) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    for (int i = 0; i < r->k; ++i) o[i] = r->stats[(size_t)i];
    return LOGOSKG_OK;
}

// ---------------------------------------------------------------- measurement aid
// The line gathers of a dense pull hop and nothing else: for every entry of the object-sorted CSR,
// in order, the 128-byte line of its subject is loaded with the access shape of k_pull_seg (one
// wavefront per 1,024 entries, eight lanes per line, eight lines per load instruction, four rounds
// in flight, the ids of the next 64 entries requested ahead) and ORed into sixteen words.  No row
// bounds, no visited or level lines, no writes: what this takes is what the memory system needs
// for the gathers of such a hop on this graph.
namespace lkg {
__global__ void __launch_bounds__(256)
k_probe_gather(const int32_t *__restrict__ in_sub, long long T, const ulonglong2 *__restrict__ lines,
               unsigned long long *out) {
    const long long lo = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * kPullSegment;
    if (lo >= T) return;  // wavefront-uniform
    const long long hi = min(T, lo + (long long)kPullSegment);
    const int l8 = lane() & 7, grp = lane() >> 3;
    unsigned long long a0 = 0, a1 = 0;
    int s_next = lo + lane() < hi ? in_sub[lo + lane()] : 0;
    for (long long j0 = lo; j0 < hi; j0 += 64) {
        const int s = s_next;
        const long long jn = j0 + 64 + lane();
        s_next = jn < hi ? in_sub[jn] : 0;
        const int n = (int)min(64ll, hi - j0);
        for (int base = 0; base < n; base += 32) {
            ulonglong2 l[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int i = base + 8 * x + grp;
                const int sx = __shfl(s, i & 63);
                l[x] = make_ulonglong2(0, 0);
                if (i < n) l[x] = lines[(size_t)sx * 8 + l8];
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                a0 |= l[x].x;
                a1 |= l[x].y;
            }
        }
    }
#pragma unroll
    for (int m = 8; m < 64; m <<= 1) {
        a0 |= shfl_xor64(a0, m);
        a1 |= shfl_xor64(a1, m);
    }
    if (lane() < 8) {
        if (a0) atomicOr(&out[2 * lane()], a0);
        if (a1) atomicOr(&out[2 * lane() + 1], a1);
    }
}
}  // namespace lkg

extern "C" logoskg_status logoskg_probe_gather(const logoskg_graph *g, const uint64_t *lines, uint64_t *out16,
                                               void *stream) {
    if (!g || !lines || !out16) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    if (g->num_shards > 1 || !g->in_sub) {
        set_error("the gather probe needs a resident graph");
        return LOGOSKG_EINVAL;
    }
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = static_cast<hipStream_t>(stream);
    LKG_HIP(hipMemsetAsync(out16, 0, 16 * sizeof(uint64_t), st));
    const long long nseg = (g->T + kPullSegment - 1) / kPullSegment;
    if (nseg > 0)
        k_probe_gather<<<dim3((unsigned)((nseg + 3) / 4)), dim3(256), 0, st>>>(
            g->in_sub, g->T, reinterpret_cast<const ulonglong2 *>(lines), reinterpret_cast<unsigned long long *>(out16));
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}
