// Bulk export of complete paths (paper Sec. 3.3, "Path reconstruction": the
// active triples of hop 1 are extended hop by hop, whenever the object of a
// triple is the subject of a triple of the next hop, into complete paths of
// length k; Eq. 5-7).
//
// For one query and a length d this file lists EVERY chain (t_1, .., t_d) of
// allowed triples with s_{t_1} a seed, o_{t_i} = s_{t_{i+1}} and the subject of
// t_i in level i-1 -- on a LOGOSKG_WALK_EXACT result all walks of d triples from
// a seed, on a minimum-hop result all shortest paths to the entities at hop d --
// without a bound per target: the chains are numbered, and a caller fetches any
// range of numbers (a page) into a buffer of its own.
//
// Order: by target (ascending entity id), chains of one target ordered
// lexicographically by (t_d, t_{d-1}, .., t_1), the order of logoskg_paths and
// logoskg_walks.  Numbering needs no enumeration: c_0[v] = 1 for the seeds,
// c_h[v] = sum over the allowed triples (s, r, v) of c_{h-1}[s] counts the chains
// that end in v after h triples (c_{h-1} is zero outside level h-1), and the
// running sums of a row of OBJ say which chain numbers pass through each of its
// triples.  Chain number x is then decoded by d binary searches, one thread per
// chain, whatever the degree of the entities on it.
#include <rocprim/device/device_scan.hpp>

#include "common.h"

namespace lkg {

// Counts stay below 2^56 (7.2 x 10^16), so up to 256 of them add up without wrapping.  Whoever adds more looks at
// the sums in between: `high` collects the upper halves of all of them, and a bit from 24 on in it says that one
// reached the limit (the tables are not used then, so what wrapped later does not matter).  No min() with the limit:
// where a min and a branch on the same comparison of two uniform 64-bit values met, the compiler's scalar select read
// a condition bit that the comparison had not written.
constexpr unsigned long long kWalkCountLimit = 1ull << 56;
constexpr int kWalkSummands = 256;

__device__ __forceinline__ unsigned long long wave_incl_scan64(unsigned long long v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = shfl_up64(v, d);
        if (lane() >= d) v += y;
    }
    return v;
}

__global__ void __launch_bounds__(256)
k_walk_seeds(int32_t E, int W, int w, unsigned long long bit, const unsigned long long *__restrict__ level0,
             unsigned long long *__restrict__ cnt0) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) cnt0[e] = (level0[(size_t)e * W + w] & bit) ? 1ull : 0ull;
}

// One hop of the count over the object rows of the entities in level h of the query: cum[j] = chains
// that pass through the row's entries before j (exclusive running sum inside the row), cnt_cur[v] =
// the row's total.
//
// Rows of up to kTailMaxDegree entries: a thread per entity walks its row, eight entries' loads
// together (neighbouring rows are contiguous in OBJ, so a wavefront's loads share their lines).
// Longer rows have a block each.  One wavefront per 64 entities, row after row, took 1.0 ms
// a hop on a 3.4M-triple graph whatever the level held (a 10^5-entry row is 1,500 turns of one
// wavefront); count and page of 10^6 chains of three triples together went from 3.2 ms to 0.30 ms there.
template <bool MASK>
__device__ __forceinline__ unsigned long long walk_entry(uint32_t j, int W, int w, unsigned long long bit,
                                                         const unsigned long long *__restrict__ allow,
                                                         const int32_t *__restrict__ in_sub,
                                                         const uint16_t *__restrict__ in_rel,
                                                         const unsigned long long *__restrict__ cnt_prev) {
    if (MASK && !(allow[(size_t)in_rel[j] * W + w] & bit)) return 0ull;
    return cnt_prev[in_sub[j]];
}

__device__ __forceinline__ uint32_t upper_half(unsigned long long x) { return (uint32_t)(x >> 32); }

// a sum on the way was past the limit: reported by the host
__device__ __forceinline__ unsigned long long capped(unsigned long long total, uint32_t high, unsigned int *overflow) {
    static_assert(kWalkCountLimit >> 32 == 1ull << 24, "the bits of `high` from 24 on");
    if ((high >> 24) == 0u) return total;
    atomicOr(overflow, 1u);
    return kWalkCountLimit - 1;
}

template <bool MASK>
__device__ __forceinline__ void walk_count_short(long long e, int32_t E, int W, int w, unsigned long long bit,
                                                 const unsigned long long *__restrict__ level_h,
                                                 const unsigned long long *__restrict__ allow,
                                                 const uint32_t *__restrict__ in_off, const int32_t *__restrict__ in_sub,
                                                 const uint16_t *__restrict__ in_rel,
                                                 const unsigned long long *__restrict__ cnt_prev,
                                                 unsigned long long *__restrict__ cnt_cur,
                                                 unsigned long long *__restrict__ cum, unsigned int *overflow) {
    if (e >= E || !(level_h[(size_t)e * W + w] & bit)) return;
    const uint32_t lo = in_off[e], hi = in_off[e + 1];
    if (hi - lo > (uint32_t)kTailMaxDegree) return;
    constexpr int U = 8;
    static_assert(kTailMaxDegree <= kWalkSummands, "a short row's sum cannot wrap");
    unsigned long long running = 0;
    for (uint32_t j0 = lo; j0 < hi; j0 += U) {
        int32_t sub[U];
        uint16_t rel[U];
        bool ok[U];
        unsigned long long c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = j0 + u < hi;
            sub[u] = ok[u] ? in_sub[j0 + u] : 0;
            if (MASK) rel[u] = ok[u] ? in_rel[j0 + u] : (uint16_t)0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (MASK && ok[u]) ok[u] = (allow[(size_t)rel[u] * W + w] & bit) != 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = ok[u] ? cnt_prev[sub[u]] : 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + u < hi) cum[j0 + u] = running;
            running += c[u];
        }
    }
    cnt_cur[e] = capped(running, upper_half(running), overflow);
}

// Entries [lo, hi) of one row by a block of NW wavefronts, U entries per lane and turn (one wavefront apart, so
// that every load and store is contiguous): cum = running sums from the first one on; returns the total.
template <bool MASK, int NW, int U>
__device__ __forceinline__ unsigned long long walk_count_span(uint32_t lo, uint32_t hi, int W, int w, unsigned long long bit,
                                                              const unsigned long long *__restrict__ allow,
                                                              const int32_t *__restrict__ in_sub,
                                                              const uint16_t *__restrict__ in_rel,
                                                              const unsigned long long *__restrict__ cnt_prev,
                                                              unsigned long long *__restrict__ cum,
                                                              unsigned long long (*part)[NW], int &buf, uint32_t &high) {
    constexpr int NT = 64 * NW;
    static_assert(64 * U <= kWalkSummands, "a wavefront's sum of one turn cannot wrap");
    static_assert(NW + 1 <= kWalkSummands, "nor can the turn's, while its parts are below the limit");
    const int wave = threadIdx.x >> 6;
    unsigned long long running = 0;
    for (uint32_t j0 = lo; j0 < hi; j0 += NT * U, buf ^= 1) {  // (buf: the half of `part` of this turn, the caller's next one too)
        const uint32_t base = j0 + (uint32_t)(wave * 64 * U + lane());
        unsigned long long c[U], incl[U], sum = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = base + u * 64 < hi ? walk_entry<MASK>(base + u * 64, W, w, bit, allow, in_sub, in_rel, cnt_prev) : 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            incl[u] = sum + wave_incl_scan64(c[u]);
            sum = shfl64(incl[u], 63);
        }
        if (lane() == 0) part[buf][wave] = sum;
        __syncthreads();  // (the other half of `part` is written in the next turn)
        unsigned long long before = running, total = running;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            const unsigned long long p = part[buf][x];
            if (x < wave) before += p;
            total += p;
            high |= upper_half(p);
        }
        high |= upper_half(total);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (base + u * 64 < hi) cum[base + u * 64] = before + (incl[u] - c[u]);
        running = total;
    }
    return running;
}

__device__ __forceinline__ long long giant_row_of(const uint32_t *__restrict__ seg_first, long long n, uint32_t seg) {
    long long lo = 0, hi = n;  // the last row whose first segment is <= seg
    while (hi - lo > 1) {
        const long long m = (lo + hi) >> 1;
        if (seg_first[m] <= seg) lo = m; else hi = m;
    }
    return lo;
}

// One launch for all rows, blocks of four wavefronts: the first n_segs take a segment of kGiantSegment entries of a
// giant row each (the first n_giant rows of the list; the segment's own running sums, its total to seg_total and to the
// row's count), the next n_long_blocks the longer rows, the others 256 entities, a thread for each short row.  A block
// of longer rows looks at every n_long_blocks-th of them (so the longest spread over the blocks) and walks those that are
// in the level: mostly few are, and a block per row took 445 us for two counts of 3 hops of a query that reaches little
// of 30M triples, kWalkBlocks blocks take 350.  The giants' running sums are joined over their segments once, behind the
// last hop (k_walk_join_giant): the hops need the counts only.
// A block per giant row was a chain of 4,096-entry turns, 140 .. 176 us a hop on 3.4M triples.  Segments, their join,
// longer and short rows in a launch each were 4 launches a hop: the whole call of three hops there 583 us, 495 us now,
// and two counts (2 and 3 hops) of a query that reaches nothing 258 us, 205 us now.
constexpr unsigned kWalkBlocks = 4096;  // at most; twice what the GPU holds at once

template <bool MASK>
__global__ void __launch_bounds__(256)
k_walk_count(const int32_t *__restrict__ rows, const uint32_t *__restrict__ seg_first, unsigned n_giant, unsigned n_segs,
             unsigned n_long, unsigned n_long_blocks, int32_t E, int W, int w, unsigned long long bit,
             const unsigned long long *__restrict__ level_h, const unsigned long long *__restrict__ allow,
             const uint32_t *__restrict__ in_off, const int32_t *__restrict__ in_sub, const uint16_t *__restrict__ in_rel,
             const unsigned long long *__restrict__ cnt_prev, unsigned long long *__restrict__ cnt_cur,
             unsigned long long *__restrict__ cum, unsigned long long *__restrict__ seg_total, unsigned int *overflow) {
    __shared__ unsigned long long part[2][4];
    const unsigned b = blockIdx.x;
    if (b >= n_segs + n_long_blocks) {
        walk_count_short<MASK>((long long)(b - n_segs - n_long_blocks) * 256 + threadIdx.x, E, W, w, bit, level_h, allow,
                               in_off, in_sub, in_rel, cnt_prev, cnt_cur, cum, overflow);
        return;
    }
    int buf = 0;
    if (b < n_segs) {
        const long long i = giant_row_of(seg_first, n_giant, b);
        const int32_t v = rows[i];
        if (!(level_h[(size_t)v * W + w] & bit)) return;  // block-uniform
        const uint32_t lo = in_off[v] + (b - seg_first[i]) * (uint32_t)kGiantSegment;
        const uint32_t hi = min(lo + (uint32_t)kGiantSegment, in_off[v + 1]);
        uint32_t high = 0;
        const unsigned long long total =
            walk_count_span<MASK, 4, 4>(lo, hi, W, w, bit, allow, in_sub, in_rel, cnt_prev, cum, part, buf, high);
        if (threadIdx.x == 0) {
            const unsigned long long x = capped(total, high, overflow);
            seg_total[b] = x;
            atomicAdd(&cnt_cur[v], x);  // (whether the row's sum passed the limit shows in the join)
        }
        return;
    }
    for (unsigned first = b - n_segs; first < n_long; first += 64u * n_long_blocks) {  // lane = one of the block's rows
        const unsigned at = first + (unsigned)lane() * n_long_blocks;
        int32_t mine = 0;
        bool in = at < n_long;
        if (in) {
            mine = rows[n_giant + at];
            in = (level_h[(size_t)mine * W + w] & bit) != 0ull;
        }
        for (unsigned long long m = __ballot(in); m; m &= m - 1) {  // the same rows in every wavefront
            const int32_t v = __shfl(mine, __builtin_ctzll(m));
            uint32_t high = 0;
            const unsigned long long total = walk_count_span<MASK, 4, 2>(in_off[v], in_off[v + 1], W, w, bit, allow, in_sub,
                                                                         in_rel, cnt_prev, cum, part, buf, high);
            if (threadIdx.x == 0) cnt_cur[v] = capped(total, high, overflow);
        }
    }
}

// Every segment of a giant row adds what lies before it in its row, for the hops whose level holds the row (lane = hop).
// Small blocks that look at all hops: in blocks of 1,024 threads per segment and hop the search for the row alone, again in
// each, was 40 us of a count of 3 hops on 30M triples.
__global__ void __launch_bounds__(256)
k_walk_join_giant(const int32_t *__restrict__ rows, const uint32_t *__restrict__ seg_first, long long n_rows, int W, int w,
                  unsigned long long bit, const unsigned long long *__restrict__ levels, size_t plane, int d,
                  const uint32_t *__restrict__ in_off, const unsigned long long *__restrict__ seg_totals, long long T,
                  unsigned long long *__restrict__ cums, unsigned int *overflow) {
    constexpr int U = 8;
    const long long i = giant_row_of(seg_first, n_rows, blockIdx.x);
    const int32_t v = rows[i];
    const uint32_t lo = in_off[v] + (blockIdx.x - seg_first[i]) * (uint32_t)kGiantSegment;
    const uint32_t hi = min(lo + (uint32_t)kGiantSegment, in_off[v + 1]);
    for (int h0 = 0; h0 < d; h0 += 64) {
        const int mine = h0 + lane();  // hop - 1
        for (unsigned long long m = __ballot(mine < d && (levels[(size_t)(mine + 1) * plane + (size_t)v * W + w] & bit)); m;
             m &= m - 1) {  // the same hops in every wavefront
            const int h = h0 + __builtin_ctzll(m);
            const unsigned long long *seg_total = seg_totals + (size_t)h * gridDim.x;
            unsigned long long *cum = cums + (size_t)h * T;
            unsigned long long before = 0;
            uint32_t high = 0;
            for (uint32_t x = seg_first[i]; x < blockIdx.x; ++x) {
                before += seg_total[x];
                high |= upper_half(before);
            }
            if (before)
                for (uint32_t j = lo + threadIdx.x; j < hi; j += 256 * U) {  // eight loads ahead of their stores
                    unsigned long long c[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) c[u] = j + u * 256 < hi ? cum[j + u * 256] : 0ull;
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (j + u * 256 < hi) cum[j + u * 256] = c[u] + before;
                }
            if (threadIdx.x == 0) (void)capped(before, high | upper_half(before + seg_total[blockIdx.x]), overflow);
        }
    }
}

// pref[0] = 0 and the running sum over the entities must not have wrapped
__global__ void __launch_bounds__(256)
k_walk_check_prefix(int32_t E, unsigned long long *pref, unsigned int *overflow) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e == 0) pref[0] = 0ull;
    if (e >= 1 && e < E && pref[e + 1] < pref[e]) atomicOr(overflow, 1u);
}

// One thread per chain of the page: the target from the prefix over the entities, then one
// triple per hop, from the last to the first, by a binary search in the running sums of the row.
__global__ void __launch_bounds__(256)
k_walk_page(long long first, long long count, int d, int32_t E, long long T, const unsigned long long *__restrict__ pref,
            const unsigned long long *__restrict__ cum, const uint32_t *__restrict__ in_off,
            const int32_t *__restrict__ in_sub, const int32_t *__restrict__ in_eid, int32_t *__restrict__ walk_edges,
            int32_t *__restrict__ walk_target) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    unsigned long long x = (unsigned long long)(first + i);
    // the last entity whose prefix is <= x (it has at least one chain: x < pref[E])
    long long a = 0, b = E;  // pref[a] <= x < pref[b]
    while (b - a > 1) {
        const long long m = (a + b) >> 1;
        if (pref[m] <= x) a = m; else b = m;
    }
    int32_t v = (int32_t)a;
    x -= pref[a];
    if (walk_target) walk_target[i] = v;
    for (int h = d; h >= 1; --h) {
        const unsigned long long *c = cum + (size_t)(h - 1) * (size_t)T;
        uint32_t lo = in_off[v], hi = in_off[v + 1];  // c[lo] = 0 <= x, and x < the row's total
        while (hi - lo > 1) {
            const uint32_t m = lo + ((hi - lo) >> 1);
            if (c[m] <= x) lo = m; else hi = m;
        }
        walk_edges[(size_t)i * d + (h - 1)] = in_eid[lo];
        x -= c[lo];
        v = in_sub[lo];
    }
}

void drop_walk_tables(logoskg_result *r) {
    logoskg_graph *g = r->g;
    r->walk_q = r->walk_d = -1;
    r->walk_total = 0;
    if (!r->walk_cnt && !r->walk_cum && !r->walk_pref) return;
    void *ptrs[] = {r->walk_cnt, r->walk_cum, r->walk_pref};
    const bool zeroed[3] = {false, false, false};
    g->pool.release_after(ptrs, zeroed, 3, r->last_stream);
    r->walk_cnt = r->walk_cum = r->walk_pref = nullptr;
}

template <bool MASK>
static void launch_walk_hop(logoskg_graph *g, int W, int w, unsigned long long bit, const unsigned long long *level_h,
                            const unsigned long long *allow, const int32_t *in_sub, const uint16_t *in_rel,
                            const unsigned long long *prev, unsigned long long *cur, unsigned long long *cum,
                            unsigned int *overflow, unsigned long long *seg_total, hipStream_t st) {
    const RowClasses &rc = g->in_rows;
    const unsigned giants = seg_total ? (unsigned)rc.n_giant : 0u, segs = giants ? (unsigned)rc.n_giant_segs : 0u;
    // (at most T / 8192 + n_giant segments and E / 256 blocks of entities: below the grid's limit)
    const unsigned n_long = (unsigned)rc.n_long - giants, n_long_blocks = std::min(n_long, kWalkBlocks);
    k_walk_count<MASK><<<dim3(segs + n_long_blocks + (unsigned)((g->E + 255) / 256)), dim3(256), 0, st>>>(
        rc.longrows, rc.giant_seg_first, giants, segs, n_long, n_long_blocks, g->E, W, w, bit, level_h, allow, g->in_off,
        in_sub, in_rel, prev, cur, cum, seg_total, overflow);
}

static logoskg_status prepare_walk_tables(logoskg_result *r, int q, int d, hipStream_t st) {
    logoskg_graph *g = r->g;
    if (r->walk_q == q && r->walk_d == d) return LOGOSKG_OK;
    drop_walk_tables(r);
    const int W = r->W, w = q >> 6;
    const unsigned long long bit = 1ull << (q & 63);
    const int32_t E = g->E;
    const size_t Epad = (size_t)r->Epad, T = (size_t)std::max<int64_t>(g->T, 1);
    const int32_t *in_sub = g->in_sub, *in_eid = g->in_eid;
    const uint16_t *in_rel = g->in_rel;
    if (g->num_shards > 1 && !shard_in_arrays(g, &in_sub, &in_rel, &in_eid)) {
        set_error("the object-sorted triples of the sharded graph are not available");
        return LOGOSKG_EINTERNAL;
    }
    // cnt: d + 1 levels, then one word of flags and the giant rows' segment totals of d hops; cum: d rows of T; pref: E + 1
    // (a sharded graph has no list of all its giant rows: they are long rows like the others)
    const size_t segs = g->num_shards > 1 ? 0 : (size_t)g->in_rows.n_giant_segs;
    LKG_TRY(g->pool.alloc((void **)&r->walk_cnt, ((size_t)(d + 1) * Epad + 8 + (size_t)d * segs) * 8, st));
    LKG_TRY(g->pool.alloc((void **)&r->walk_cum, (size_t)std::max(d, 1) * T * 8, st));
    LKG_TRY(g->pool.alloc((void **)&r->walk_pref, (Epad + 8) * 8, st));
    unsigned int *overflow = (unsigned int *)(r->walk_cnt + (size_t)(d + 1) * Epad);
    unsigned long long *seg_total = segs ? r->walk_cnt + (size_t)(d + 1) * Epad + 8 : nullptr;
    LKG_HIP(hipMemsetAsync(r->walk_cnt, 0, ((size_t)(d + 1) * Epad + 8) * 8, st));
    const size_t plane = Epad * (size_t)W;
    {
        ProfScope ps(g->prof, KK_PATHS, st);
        k_walk_seeds<<<dim3((unsigned)((E + 255) / 256)), dim3(256), 0, st>>>(E, W, w, bit, r->levels, r->walk_cnt);
        for (int h = 1; h <= d; ++h) {
            const unsigned long long *lvl = r->levels + plane * (size_t)h;
            unsigned long long *prev = r->walk_cnt + (size_t)(h - 1) * Epad, *cur = r->walk_cnt + (size_t)h * Epad;
            unsigned long long *cum = r->walk_cum + (size_t)(h - 1) * T;
            unsigned long long *totals = seg_total ? seg_total + (size_t)(h - 1) * segs : nullptr;
            if (r->has_mask) launch_walk_hop<true>(g, W, w, bit, lvl, r->allow, in_sub, in_rel, prev, cur, cum, overflow, totals, st);
            else launch_walk_hop<false>(g, W, w, bit, lvl, nullptr, in_sub, in_rel, prev, cur, cum, overflow, totals, st);
        }
        if (seg_total && d > 0)
            k_walk_join_giant<<<dim3((unsigned)segs), dim3(256), 0, st>>>(
                g->in_rows.longrows, g->in_rows.giant_seg_first, g->in_rows.n_giant, W, w, bit, r->levels, plane, d, g->in_off,
                seg_total, (long long)T, r->walk_cum, overflow);
    }
    LKG_HIP(hipGetLastError());
    // pref[e + 1] = chains that end in an entity <= e
    const unsigned long long *last = r->walk_cnt + (size_t)d * Epad;
    size_t bytes = 0;
    auto check = [&](hipError_t e, const char *what) -> logoskg_status {
        if (e != hipSuccess) { set_error("%s failed: %s", what, hipGetErrorString(e)); return LOGOSKG_EDEVICE; }
        return LOGOSKG_OK;
    };
    LKG_TRY(check(rocprim::inclusive_scan(nullptr, bytes, last, r->walk_pref + 1, (size_t)E,
                                          rocprim::plus<unsigned long long>(), st), "sizing the prefix sum"));
    void *tmp = nullptr;
    LKG_TRY(g->pool.alloc(&tmp, std::max<size_t>(bytes, 8), st));
    logoskg_status s = check(rocprim::inclusive_scan(tmp, bytes, last, r->walk_pref + 1, (size_t)E,
                                                     rocprim::plus<unsigned long long>(), st), "prefix sum");
    {
        void *ptrs[] = {tmp};
        const bool z[1] = {false};
        g->pool.release_after(ptrs, z, 1, st);
    }
    LKG_TRY(s);
    k_walk_check_prefix<<<dim3((unsigned)((E + 255) / 256)), dim3(256), 0, st>>>(E, r->walk_pref, overflow);
    LKG_HIP(hipGetLastError());
    unsigned long long total = 0;
    unsigned int ovf = 0;
    LKG_HIP(hipMemcpyAsync(&total, r->walk_pref + E, 8, hipMemcpyDeviceToHost, st));
    LKG_HIP(hipMemcpyAsync(&ovf, overflow, 4, hipMemcpyDeviceToHost, st));
    LKG_HIP(hipStreamSynchronize(st));
    if (ovf || total >= (1ull << 62)) {
        drop_walk_tables(r);
        set_error("query %d has 2^56 or more chains of %d triples into one entity: too many to number", q, d);
        return LOGOSKG_ERANGE;
    }
    r->walk_q = q;
    r->walk_d = d;
    r->walk_total = (int64_t)total;
    return LOGOSKG_OK;
}

}  // namespace lkg

using namespace lkg;

extern "C" logoskg_status logoskg_result_walks_count(logoskg_result *r, int32_t query, int32_t length, int64_t *total,
                                                     void *stream) {
    if (!r || !total) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    if (query < 0 || query >= r->Q) { set_error("query %d outside [0, %d)", query, r->Q); return LOGOSKG_EINVAL; }
    if (length < 0 || length > r->k) { set_error("length %d outside [0, %d]", length, r->k); return LOGOSKG_EINVAL; }
    logoskg_graph *g = r->g;
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    r->last_stream = st;
    LKG_TRY(prepare_walk_tables(r, query, length, st));
    *total = r->walk_total;
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_result_walks_fetch(logoskg_result *r, int32_t query, int32_t length, int64_t first,
                                                     int64_t count, int32_t *walk_edges, int32_t *walk_target,
                                                     void *stream) {
    if (!r) { set_error("NULL result"); return LOGOSKG_EINVAL; }
    if (r->walk_q != query || r->walk_d != length || query < 0) {
        set_error("the chains of %d triples of query %d were not counted: call logoskg_result_walks_count for them first",
                  length, query);
        return LOGOSKG_EINVAL;
    }
    if (first < 0 || count < 0 || first + count > r->walk_total) {
        set_error("chains [%lld, %lld) outside [0, %lld)", (long long)first, (long long)(first + count),
                  (long long)r->walk_total);
        return LOGOSKG_ERANGE;
    }
    if (count == 0) return LOGOSKG_OK;
    if (count > (1ll << 36)) { set_error("at most 2^36 chains per call"); return LOGOSKG_ERANGE; }
    if ((length > 0 && !walk_edges) || (length == 0 && !walk_target)) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    logoskg_graph *g = r->g;
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    r->last_stream = st;
    const int32_t *in_sub = g->in_sub, *in_eid = g->in_eid;
    const uint16_t *in_rel = g->in_rel;
    if (g->num_shards > 1 && !shard_in_arrays(g, &in_sub, &in_rel, &in_eid)) {
        set_error("the object-sorted triples of the sharded graph are not available");
        return LOGOSKG_EINTERNAL;
    }
    ProfScope ps(g->prof, KK_PATHS, st);
    k_walk_page<<<dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st>>>(
        first, count, length, g->E, std::max<int64_t>(g->T, 1), r->walk_pref, r->walk_cum, g->in_off, in_sub, in_eid,
        walk_edges, walk_target);
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}
