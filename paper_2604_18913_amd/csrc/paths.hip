// logoskg_paths: shortest-path listing from the level planes (paper Sec. 3.3,
// "Path reconstruction", Eq. 5-7).  A triple t is on a shortest path of query q
// to its object when its subject sits exactly one hop closer to the seeds and
// q allows its relation; chaining such triples backward from the target always
// ends at a seed, so a depth-first walk over the object rows (edge ids
// ascending) lists the paths in (t_d, t_{d-1}, .., t_1) order and can stop at
// max_paths.
//
// logoskg_walks lists walks of a given number of triples on a result of the
// plain iteration (no visited set) with the same kernel: there level h holds
// the ends of the walks of h triples, so the backward walk from level d of the
// target through levels d-1 .. 0 meets exactly the walks of d allowed triples
// from a seed (Sec. 3.3: complete paths, extended hop by hop).
#include <algorithm>

#include "common.h"

namespace lkg {

// What the listing kernel needs besides the level planes.
struct PathArgs {
    long long first_pair;  // of this launch
    int Q, k, W;
    int32_t E, R;
    long long plane, actw;
    const unsigned long long *levels, *allow;
    const uint32_t *act;
    const uint32_t *in_off;
    const int32_t *in_sub;
    const uint16_t *in_rel;
    const int32_t *in_eid;
    // the queries' seeds and SUB's rows with their triple indices, or NULL out_eid
    const long long *seed_off;
    const int32_t *seeds;
    const uint32_t *out_off;
    const int32_t *out_obj;
    const uint16_t *out_rel;
    const int32_t *out_eid;
    const int32_t *query_idx, *target, *length;
    int max_paths;
    int32_t *path_count, *path_edges;
};

// Wavefronts per pair on graphs with rows longer than kPathShortRow: 16 up to kPathWidePairs pairs, 4 up to
// kPathNarrowPairs, then one.  What counts are the scans of long rows: few pairs need many wavefronts each to fill the
// GPU, many pairs fill it by themselves.  us for 16 paths each on a 30M-triple graph (k = 3 with whitelists; without):
//    pairs     16 wavefronts       4               1
//       64       749     250      982     172     3,161     449
//      256     1,777     614    2,262     753     6,769   2,344
//    1,024     2,600   1,973    2,579   2,253     8,003   6,880
//    4,096     5,216   3,504    3,301   2,395     9,810   6,671
//   65,536    69,857  38,151   18,755   9,009    21,416  14,278
//  131,072   138,171  74,066   37,363  15,773    40,212  19,234
//  262,144   276,567 147,159   70,130  29,416    67,812  29,837
// With k = 2 the rows of a pair are fewer: 4 are better than 16 from 512 pairs on (without whitelists from 64 on: 46
// against 117 us), one than 4 from 131,072 on.
constexpr int64_t kPathWidePairs = 1024;
constexpr int64_t kPathNarrowPairs = 65536;
constexpr int kPathSeeds = 64;    // queries with more seeds than this keep to the object rows at level 1
constexpr int kPathRelations = 2048; // up to so many relations the query's whitelist is held in LDS
constexpr int kPathMatches = 256; // triples from the seeds into one entity that are sorted in LDS
constexpr uint32_t kPathShortRow = 128;  // what is left of a row up to this length: one wavefront, two entries per lane

// Triples of the pair's paths: -1 = none, 0 = the target is a seed.
__device__ __forceinline__ int path_length(const PathArgs &a, long long i, int v, int w, unsigned long long bit) {
    if (a.length) {  // walks of exactly that many triples: the target has to sit in that level
        const int want = a.length[i];
        return want >= 0 && want <= a.k && (a.levels[(size_t)want * a.plane + (size_t)v * a.W + w] & bit) ? want : -1;
    }
    for (int h0 = 0; h0 <= a.k; h0 += 64) {  // shortest paths: the first level that holds the target, 64 levels at a time
        const int h = h0 + lane();
        const unsigned long long m = __ballot(h <= a.k && (a.levels[(size_t)min(h, a.k) * a.plane + (size_t)v * a.W + w] & bit));
        if (m) return h0 + __builtin_ctzll(m);
    }
    return -1;
}

// writes path number `at`: the edges chosen at levels d .. 2, and `eid` in front of them
__device__ __forceinline__ void write_path(int32_t *out, int k, int d, const int32_t *se, int at, int32_t eid) {
    int32_t *row = out + (size_t)at * k;
    row[0] = eid;
    for (int x = 2; x <= d; ++x) row[x - 1] = se[x];
}

// The search from entry j of vertex x's row at level lev on by one wavefront alone, until it is over or the next row is a
// long one: subject, relation and triple index of two entries per lane are requested together, then the subjects' level
// words.  The stacks hold every entry but the current one (x, j) while this runs; n = paths found.
template <typename Allowed>
__device__ __forceinline__ void path_short_rows(const PathArgs &a, int w, unsigned long long bit, int d, int32_t *out,
                                                int32_t *sv, uint32_t *sp, int32_t *se, Allowed allowed, int x, uint32_t j,
                                                uint32_t hi, int &lev, int &n) {
    const int k = a.k, W = a.W, max_paths = a.max_paths;
    while (true) {
        if (hi - j > kPathShortRow) break;
        const unsigned long long *lv = a.levels + (size_t)(lev - 1) * a.plane;
        const uint32_t at0 = j + (uint32_t)lane(), at1 = at0 + 64u;
        const bool in0 = at0 < hi, in1 = at1 < hi;
        const int32_t s0 = in0 ? a.in_sub[at0] : 0, s1 = in1 ? a.in_sub[at1] : 0;
        const int32_t e0 = in0 ? a.in_eid[at0] : 0, e1 = in1 ? a.in_eid[at1] : 0;
        int r0 = 0, r1 = 0;
        if (a.allow) {
            r0 = in0 ? a.in_rel[at0] : 0;
            r1 = in1 ? a.in_rel[at1] : 0;
        }
        const unsigned long long w0 = in0 ? lv[(size_t)s0 * W + w] : 0ull, w1 = in1 ? lv[(size_t)s1 * W + w] : 0ull;
        bool ok0 = (w0 & bit) != 0ull, ok1 = (w1 & bit) != 0ull;
        if (a.allow) {
            ok0 &= allowed(r0);
            ok1 &= allowed(r1);
        }
        const unsigned long long m0 = __ballot(ok0), m1 = __ballot(ok1);
        if (lev == 1) {  // every admissible entry ends a path
            if (d > 8) {  // long paths: one after the other, their entries by all lanes
                for (int half = 0, at = n; half < 2; ++half)
                    for (unsigned long long m = half ? m1 : m0; m && at < max_paths; m &= m - 1, ++at) {
                        const int32_t eid = __shfl(half ? e1 : e0, __builtin_ctzll(m));
                        int32_t *row = out + (size_t)at * k;
                        for (int x = lane(); x < d; x += 64) row[x] = x ? se[x + 1] : eid;
                    }
            } else {
                const unsigned long long below = (1ull << lane()) - 1ull;
                const int p0 = n + __popcll(m0 & below), p1 = n + __popcll(m0) + __popcll(m1 & below);
                if (ok0 && p0 < max_paths) write_path(out, k, d, se, p0, e0);
                if (ok1 && p1 < max_paths) write_path(out, k, d, se, p1, e1);
            }
            n = min(max_paths, n + __popcll(m0) + __popcll(m1));
        } else if (m0 | m1) {  // the first one is descended into
            const int f = m0 ? __builtin_ctzll(m0) : __builtin_ctzll(m1);
            const int32_t sf = __shfl(m0 ? s0 : s1, f), ef = __shfl(m0 ? e0 : e1, f);
            se[lev] = ef;  // (all lanes write the same)
            sv[lev] = x;
            sp[lev] = j + (m0 ? 0u : 64u) + (uint32_t)f + 1u;
            --lev;
            x = sf;
            j = a.in_off[sf];
            hi = a.in_off[sf + 1];
            continue;
        }
        // this vertex's row is exhausted: back to the vertex after it
        ++lev;
        if (lev > d || n >= max_paths) break;
        x = sv[lev];
        j = sp[lev];
        hi = a.in_off[x + 1];
    }
    if (lev <= d) {
        sv[lev] = x;
        sp[lev] = j;
    }
}

// A graph whose object rows are all short: a wavefront per pair, four pairs per block, nothing shared between them.
// What bounds it is the chain of gathers down a path and, with many pairs, the rows of -1 that are written first (80,000
// pairs on 50,000 entities and 250,000 triples, 16 paths of up to four triples: 20 MB in 89 us; 113 us with a block of
// one wavefront for every pair).
__global__ void __launch_bounds__(256) k_paths_short(PathArgs a, long long n_pairs) {
    __shared__ int32_t sv_all[4][LOGOSKG_MAX_K + 1], se_all[4][LOGOSKG_MAX_K + 1];
    __shared__ uint32_t sp_all[4][LOGOSKG_MAX_K + 1];
    const int wave = threadIdx.x >> 6;
    const long long i = a.first_pair + (long long)blockIdx.x * 4 + wave;
    if (i >= n_pairs) return;  // wavefront-uniform
    int32_t *out = a.path_edges + (size_t)i * a.max_paths * a.k;
    for (long long x = lane(); x < (long long)a.max_paths * a.k; x += 64) out[x] = -1;
    const int q = a.query_idx[i], v = a.target[i];
    int n = 0;
    if ((uint32_t)q < (uint32_t)a.Q && (uint32_t)v < (uint32_t)a.E) {
        const int w = q >> 6;
        const unsigned long long bit = 1ull << (q & 63);
        const int d = path_length(a, i, v, w, bit);
        if (d == 0) n = 1;  // a seed: one empty path
        auto allowed = [&](int r) -> bool { return (a.allow[(size_t)r * a.W + w] & bit) != 0ull; };
        int lev = d;
        if (d > 0)
            path_short_rows(a, w, bit, d, out, sv_all[wave], sp_all[wave], se_all[wave], allowed, v, a.in_off[v],
                            a.in_off[v + 1], lev, n);
    }
    if (lane() == 0) a.path_count[i] = n;
}

// NW wavefronts (one block) per (query, target) pair.  The depth-first state - per level the vertex,
// the next row position and the chosen edge - is block-uniform and lives in LDS (k <= 254).
//
// An object row is scanned in steps of NT = 64 NW entries (the first step after a descent) or four
// times as many: every lane tests its entries (relation allowed, the subject's bit in the level's
// active bitmap, then the query's bit in the subject's level line - each test spares the rest the
// next, dearer gather), and the ballots of all wavefronts give the admissible entries in ascending
// position = ascending edge id.  At level 1 every admissible entry ends a path and the entries' own
// lanes write them; above, the first one is descended into.
//
// Where at most kPathShortRow entries of a row are left, the block's barriers and its steps would be all that
// it costs: one wavefront goes on alone then, two entries per lane, until the next long row.  (16 paths of up to 40
// triples through rows of two entries: 228 us with a wavefront per pair, 1,810 us with sixteen that take every
// row together, 230 us now.)
//
// The last triple on the way down leaves a seed, and a query has few seeds: when their out-rows
// together are shorter than the vertex's object row, the block walks those instead and sorts the
// matches by edge id.  What bounds the kernel are hub targets and the hub subjects of level 1, whose
// rows hold 10^5 entries.  4,096 pairs of a 30M-triple graph with whitelists, k = 2, 16 paths each:
// 19.1 ms with one wavefront per pair and 64 entries per step (every path scanned the whole object
// row of its level-1 subject for a seed), 0.46 ms now (0.65 with the whitelist's words gathered from global
// memory for every entry), with the rows' entries and the gathers of their subjects' bits for a floor:
// sixteen wavefronts per pair took 0.96 ms against those 0.65 (the short rows leave them idle), so it is the
// scans' work and no longer one block's chain of steps that counts.
template <int NW>
__global__ void __launch_bounds__(64 * NW) k_paths(PathArgs a) {
    constexpr int NT = 64 * NW, U = 4;
    __shared__ int32_t sv[LOGOSKG_MAX_K + 1], se[LOGOSKG_MAX_K + 1];
    __shared__ uint32_t sp[LOGOSKG_MAX_K + 1];
    __shared__ unsigned long long hit[2][U][NW];
    __shared__ uint32_t s_lo[kPathSeeds], s_end[kPathSeeds];  // out-rows of the seeds: begin, running total of the lengths
    __shared__ int32_t s_id[kPathSeeds];
    __shared__ int32_t match[kPathMatches];
    __shared__ unsigned long long s_allow[kPathRelations / 64];
    __shared__ int n_match, s_l, s_found;
    const long long i = a.first_pair + blockIdx.x;
    const int t = threadIdx.x, wave = t >> 6, k = a.k, W = a.W, max_paths = a.max_paths;
    int32_t *out = a.path_edges + (size_t)i * max_paths * k;
    for (long long x = t; x < (long long)max_paths * k; x += NT) out[x] = -1;
    const int q = a.query_idx[i], v = a.target[i];
    if ((uint32_t)q >= (uint32_t)a.Q || (uint32_t)v >= (uint32_t)a.E) {
        if (t == 0) a.path_count[i] = 0;
        return;
    }
    const int w = q >> 6;
    const unsigned long long bit = 1ull << (q & 63);
    const int d = path_length(a, i, v, w, bit);
    if (d <= 0) {  // not reached: no path; a seed: one empty path
        if (t == 0) a.path_count[i] = d == 0 ? 1 : 0;
        return;
    }
    // The whitelist test is the first of every entry.  Where the target's row is longer than the list of relations
    // (only then are there more gathers to save than the collecting makes), the query's bits are collected in LDS
    // once: 0.65 -> 0.46 ms for the 4,096 pairs above.
    const bool lds_allow = a.allow && a.R <= kPathRelations && a.in_off[v + 1] - a.in_off[v] > (uint32_t)a.R;  // block-uniform
    if (lds_allow) {
        for (int r0 = wave * 64; r0 < a.R; r0 += NT) {
            const int r = r0 + lane();
            const unsigned long long m = __ballot(r < a.R && (a.allow[(size_t)(r < a.R ? r : 0) * W + w] & bit));
            if (lane() == 0) s_allow[r0 >> 6] = m;
        }
        __syncthreads();
    }
    auto allowed = [&](int r) -> bool {
        return lds_allow ? (s_allow[r >> 6] >> (r & 63)) & 1ull : (a.allow[(size_t)r * W + w] & bit) != 0ull;
    };
    int found = 0, l = d, buf = 0, n_seeds = -1;
    uint32_t seed_edges = 0;
    if (t == 0) {
        sv[d] = v;
        sp[d] = a.in_off[v];
    }
    __syncthreads();
    while (l <= d && found < max_paths) {  // (all wavefronts have the same l and found)
        const int x = sv[l];
        uint32_t j = sp[l];
        const uint32_t hi = a.in_off[x + 1];
        if (hi - j <= kPathShortRow) {
            __syncthreads();  // (the last reads of the stacks)
            if (wave == 0) {
                int lev = l, n = found;
                path_short_rows(a, w, bit, d, out, sv, sp, se, allowed, x, j, hi, lev, n);
                s_l = lev;  // (all lanes write the same)
                s_found = n;
            }
            __syncthreads();
            l = s_l;
            found = s_found;
            continue;
        }
        bool descended = false;
        if (l == 1 && n_seeds < 0) {
            // the seeds' out-rows (a repeated seed counts once), looked at when the first long row asks for them;
            // n_seeds = 0: not usable for this query
            n_seeds = 0;
            if (a.out_eid) {  // block-uniform
                const long long b0 = a.seed_off[q], n = a.seed_off[q + 1] - b0;
                if (n > 0 && n <= kPathSeeds) {
                    n_seeds = (int)n;
                    if (t < n_seeds) s_id[t] = a.seeds[b0 + t];
                    __syncthreads();
                    if (t < n_seeds) {
                        const int32_t s = s_id[t];
                        bool again = false;
                        for (int x = 0; x < t; ++x) again |= s_id[x] == s;
                        s_lo[t] = a.out_off[s];
                        s_end[t] = again ? 0u : a.out_off[s + 1] - s_lo[t];
                    }
                    __syncthreads();
                    if (t == 0) {
                        uint32_t sum = 0;
                        for (int x = 0; x < n_seeds; ++x) s_end[x] = sum += s_end[x];  // < 2^31: distinct rows of one graph
                    }
                    __syncthreads();
                    seed_edges = s_end[n_seeds - 1];
                }
            }
        }
        if (l == 1 && n_seeds > 0 && seed_edges < hi - j) {
            __syncthreads();  // (the last reads of n_match and match)
            if (t == 0) n_match = 0;
            __syncthreads();
            for (uint32_t p = t; p < seed_edges; p += NT) {
                int r = 0;
                while (s_end[r] <= p) ++r;
                const uint32_t jj = s_lo[r] + (p - (r ? s_end[r - 1] : 0u));
                if (a.out_obj[jj] != x) continue;
                if (a.allow && !allowed(a.out_rel[jj])) continue;
                const int m = atomicAdd(&n_match, 1);
                if (m < kPathMatches) match[m] = a.out_eid[jj];
            }
            __syncthreads();
            const int n = n_match;
            if (n <= kPathMatches) {
                for (int m = t; m < n; m += NT) {
                    const int32_t eid = match[m];
                    int rank = 0;
                    for (int y = 0; y < n; ++y) rank += match[y] < eid;
                    if (found + rank < max_paths) write_path(out, k, d, se, found + rank, eid);
                }
                found = min(max_paths, found + n);
                ++l;
                continue;
            }
        }
        const unsigned long long *lv = a.levels + (size_t)(l - 1) * a.plane;
        const uint32_t *act = a.act + (size_t)(l - 1) * a.actw;
        // The first step after a descent takes an entry per lane, the next ones U; from the second on the ids of the step
        // behind it are on their way while the bits of this one are gathered.  With many pairs the longest rows outlast
        // everything else, and their steps are chains of gathers: a row of 123,361 entries by four wavefronts 306 -> 236 us.
        int steps = 1, s_next[U], r_next[U];
        auto request = [&](uint32_t j0, int n) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t jj = j0 + (uint32_t)(u * NT + t);
                const uint32_t at = u < n && jj < hi ? jj : j;  // (an entry of the row in any case)
                s_next[u] = a.in_sub[at];
                r_next[u] = a.allow ? a.in_rel[at] : 0;
            }
        };
        request(j, 1);
        while (j < hi && found < max_paths) {
            int32_t s[U], r[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s[u] = s_next[u];
                r[u] = r_next[u];
                ok[u] = u < steps && j + (uint32_t)(u * NT + t) < hi;
            }
            const uint32_t j_next = j + (uint32_t)(steps * NT);
            if (steps > 1) request(j_next, j_next < hi ? U : 0);
            // Lanes that are out read what stands for entity or relation 0: with a branch around every gather, the U gathers
            // of a kind waited for each other.
            if (a.allow) {
                unsigned long long x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = lds_allow ? s_allow[r[u] >> 6] >> (r[u] & 63) : a.allow[(size_t)r[u] * W + w] >> (q & 63);
#pragma unroll
                for (int u = 0; u < U; ++u) ok[u] &= (x[u] & 1ull) != 0ull;
            }
            {
                uint32_t x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = act[(ok[u] ? s[u] : 0) >> 5] >> (s[u] & 31);
#pragma unroll
                for (int u = 0; u < U; ++u) ok[u] &= (x[u] & 1u) != 0u;
            }
            {
                unsigned long long x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = lv[(size_t)(ok[u] ? s[u] : 0) * W + w];
#pragma unroll
                for (int u = 0; u < U; ++u) ok[u] &= (x[u] & bit) != 0ull;
            }
            unsigned long long mine[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mine[u] = __ballot(ok[u]);
                if (lane() == 0) hit[buf][u][wave] = mine[u];
            }
            __syncthreads();  // the other half of `hit` is written next: no barrier needed after the reads
            if (l == 1) {
                int before = found;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    int at = before;
                    for (int y = 0; y < NW; ++y) {
                        const int c = __popcll(hit[buf][u][y]);
                        if (y < wave) at += c;
                        before += c;
                    }
                    if (ok[u]) {
                        at += __popcll(mine[u] & ((1ull << lane()) - 1ull));
                        if (at < max_paths) write_path(out, k, d, se, at, a.in_eid[j + (uint32_t)(u * NT + t)]);
                    }
                }
                found = min(max_paths, before);
            } else {  // take the first one and go down; the rest of the row is tried after coming back
                int pos = -1;
                for (int y = U * NW - 1; y >= 0; --y) {
                    const unsigned long long m = hit[buf][y / NW][y % NW];
                    if (m) pos = y * 64 + __builtin_ctzll(m);
                }
                if (pos >= 0) {
                    if (t == 0) {
                        const uint32_t jj = j + (uint32_t)pos;
                        const int32_t sf = a.in_sub[jj];
                        se[l] = a.in_eid[jj];
                        sp[l] = jj + 1u;
                        sv[l - 1] = sf;
                        sp[l - 1] = a.in_off[sf];
                    }
                    buf ^= 1;
                    --l;
                    descended = true;
                    __syncthreads();
                    break;
                }
            }
            buf ^= 1;
            if (steps == 1) request(j_next, U);
            j = j_next;
            steps = U;
        }
        if (!descended) ++l;  // this vertex's row is exhausted: back to the vertex after it
    }
    if (t == 0) a.path_count[i] = found;
}

}  // namespace lkg

using namespace lkg;

// `may_allocate`: the triple indices of SUB's rows may be built on this call (4 bytes per triple, kept
// with the graph); without them the seeds' side is not used.
static logoskg_status launch_paths(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                   const int32_t *target, const int32_t *length, int64_t n_pairs, int32_t max_paths,
                                   int32_t *path_count, int32_t *path_edges, bool may_allocate, hipStream_t st) {
    r->last_stream = st;
    PathArgs a = {};
    // a sharded graph keeps its object-sorted triples in pinned host memory: the kernel reads the
    // rows it walks from there
    a.in_sub = g->in_sub; a.in_eid = g->in_eid; a.in_rel = g->in_rel;
    if (g->num_shards > 1 && !shard_in_arrays(g, &a.in_sub, &a.in_rel, &a.in_eid)) {
        set_error("the object-sorted triples of the sharded graph are not available");
        return LOGOSKG_EINTERNAL;
    }
    if (g->num_shards <= 1 && r->seeds) {
        if (may_allocate) (void)ensure_out_eid(g, st);  // no room: the object rows serve
        a.seed_off = r->seed_off; a.seeds = r->seeds;
        a.out_off = g->out_off; a.out_obj = g->out_obj; a.out_rel = g->out_rel; a.out_eid = g->out_eid;
    }
    a.Q = r->Q; a.k = r->k; a.W = r->W; a.E = g->E; a.R = g->R;
    a.plane = r->Epad * r->W; a.actw = r->Epad / 32;
    a.levels = r->levels; a.act = r->act; a.allow = r->has_mask ? r->allow : nullptr;
    a.in_off = g->in_off;
    a.query_idx = query_idx; a.target = target; a.length = length;
    a.max_paths = max_paths; a.path_count = path_count; a.path_edges = path_edges;
    ProfScope ps(g->prof, KK_PATHS, st);
    // A graph without a row for the whole block: k_paths_short, whatever the pairs' number (10,000 pairs on that graph, whose
    // rows have up to 14 entries: 61 us with four wavefronts per pair, of which three wait, 38 with one, 35 with four pairs
    // to a block).
    const bool short_rows = g->in_rows.longest <= kPathShortRow;
    // (a launch takes fewer than 2^32 threads)
    for (int64_t first = 0; first < n_pairs; first += 1ll << 25) {
        const dim3 grid((unsigned)std::min<int64_t>(n_pairs - first, 1ll << 25));
        a.first_pair = first;
        if (short_rows) k_paths_short<<<dim3((grid.x + 3) / 4), dim3(256), 0, st>>>(a, n_pairs);
        else if (n_pairs <= kPathWidePairs) k_paths<16><<<grid, dim3(1024), 0, st>>>(a);
        else if (n_pairs <= kPathNarrowPairs) k_paths<4><<<grid, dim3(256), 0, st>>>(a);
        else k_paths<1><<<grid, dim3(64), 0, st>>>(a);
    }
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

static logoskg_status check_path_args(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                      const int32_t *target, int64_t n_pairs, int32_t max_paths,
                                      const int32_t *path_count, const int32_t *path_edges) {
    if (n_pairs < 0 || max_paths < 1 || max_paths > LOGOSKG_MAX_PATHS) {
        set_error("bad n_pairs / max_paths");
        return LOGOSKG_EINVAL;
    }
    if (n_pairs > 0 && (!query_idx || !target || !path_count || (r->k > 0 && !path_edges))) {
        set_error("NULL argument");
        return LOGOSKG_EINVAL;
    }
    return LOGOSKG_OK;
}

static logoskg_status list_paths(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                 const int32_t *target, const int32_t *length, int64_t n_pairs, int32_t max_paths,
                                 int32_t *path_count, int32_t *path_edges, void *stream) {
    LKG_TRY(check_path_args(g, r, query_idx, target, n_pairs, max_paths, path_count, path_edges));
    if (n_pairs == 0) return LOGOSKG_OK;
    LKG_HIP(hipSetDevice(g->device));
    hipStream_t st = (hipStream_t)stream;
    LKG_TRY(launch_paths(g, r, query_idx, target, length, n_pairs, max_paths, path_count, path_edges, true, st));
    LKG_HIP(hipStreamSynchronize(st));
    return LOGOSKG_OK;
}

// ---------------------------------------------------------------- listing without any allocation
// logoskg_paths needs no working memory beside the block's LDS, but may build the triple indices of
// SUB's rows on first use and waits for the stream; logoskg_paths_static does neither.
extern "C" logoskg_status logoskg_paths_static(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                               const int32_t *target, int64_t n_pairs, int32_t max_paths,
                                               int32_t *path_count, int32_t *path_edges, void *stream) {
    if (!g || !r || r->g != g) { set_error("graph / result mismatch"); return LOGOSKG_EINVAL; }
    if (r->walk_exact) {
        set_error("shortest paths are not defined for a LOGOSKG_WALK_EXACT result");
        return LOGOSKG_EINVAL;
    }
    LKG_TRY(check_path_args(g, r, query_idx, target, n_pairs, max_paths, path_count, path_edges));
    const long long slots = (long long)n_pairs * std::max(r->k, 1);
    if (slots > (long long)LOGOSKG_STATIC_PATH_SLOTS) {
        set_error("logoskg_paths_static: n_pairs * max(k, 1) = %lld exceeds LOGOSKG_STATIC_PATH_SLOTS = %lld; "
                  "split the pair list or use logoskg_paths", slots, (long long)LOGOSKG_STATIC_PATH_SLOTS);
        return LOGOSKG_ERANGE;
    }
    if (n_pairs == 0) return LOGOSKG_OK;
    LKG_HIP(hipSetDevice(g->device));
    return launch_paths(g, r, query_idx, target, nullptr, n_pairs, max_paths, path_count, path_edges, false,
                        (hipStream_t)stream);
}

extern "C" logoskg_status logoskg_paths(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                        const int32_t *target, int64_t n_pairs, int32_t max_paths,
                                        int32_t *path_count, int32_t *path_edges, void *stream) {
    if (!g || !r || r->g != g) { set_error("graph / result mismatch"); return LOGOSKG_EINVAL; }
    if (r->walk_exact) {
        set_error("shortest paths are not defined for a LOGOSKG_WALK_EXACT result: use logoskg_walks");
        return LOGOSKG_EINVAL;
    }
    return list_paths(g, r, query_idx, target, nullptr, n_pairs, max_paths, path_count, path_edges, stream);
}

extern "C" logoskg_status logoskg_walks(logoskg_graph *g, const logoskg_result *r, const int32_t *query_idx,
                                        const int32_t *target, const int32_t *length, int64_t n_pairs,
                                        int32_t max_paths, int32_t *path_count, int32_t *path_edges, void *stream) {
    if (!g || !r || r->g != g) { set_error("graph / result mismatch"); return LOGOSKG_EINVAL; }
    if (!r->walk_exact) {
        set_error("walks of a given length need a LOGOSKG_WALK_EXACT result (levels = ends of the walks of h triples)");
        return LOGOSKG_EINVAL;
    }
    if (n_pairs > 0 && !length) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    return list_paths(g, r, query_idx, target, length, n_pairs, max_paths, path_count, path_edges, stream);
}
