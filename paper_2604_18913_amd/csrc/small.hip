// Small searches: the first hops of a batch of up to 64 queries (one plane word per entity) in one
// launch of one block, and the lists of a search that ended inside it in another.
//
// A question to a knowledge graph starts at a handful of entities, and its first hops - often all of
// them - touch a few hundred triples.  Hop by hop, such a search is nothing but launches (a dozen per
// hop) and a read-back of the frontier's size per hop, 30 us each.  Here one block of sixteen wavefronts
// scatters the seeds, keeps the frontier as a list in LDS and pushes it, until the search is done or
// a frontier is too large for one CU (kSmallEdges triples) or dense enough that
// the hop should pull; the host reads one report and goes on from there.  The planes, bitmaps and
// visited words are the ones the general kernels write, so every other call works on such a result.
//
// When the whole search fits, the same launch sorts the reached entities and counts per query, and
// logoskg_result_fetch takes a block per query: the reached entities' out-rows are walked once
// more and offer their triple indices to the objects one hop further (LDS atomicMin), which
// costs the triples of the search and not the object rows of what it reached - one reached hub has
// 10^5 entries in its object row.
//
// One question, two hops, 10,000 entities: 30 launches and 4 read-backs, 216 .. 242 us with the lists; now 3
// launches and one read-back, 55 us.  64 questions: 306 .. 322 -> 77 us (k_small_search 17 .. 42 us, a chain of
// dependent reads per hop; k_small_fetch 5 .. 16 us; the rest is the binding and the read-back).
#include <algorithm>
#include <climits>

#include "common.h"

namespace lkg {

namespace {

constexpr int kSmallThreads = 1024;

__device__ __forceinline__ unsigned long long load_l2(const unsigned long long *p) {  // (atomics write past the L1)
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Atomics without a result and stores of the wavefront have been performed when this returns; a barrier
// behind it makes them visible to the block's reads past the L1.
__device__ __forceinline__ void drain_writes() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// exclusive prefix over one value per thread of a block; *total receives the sum
template <int NT>
__device__ __forceinline__ int block_excl_scan(int v, int *part, int &total) {
    const int wave = threadIdx.x >> 6;
    int sum;
    const int x = wave_excl_scan(v, sum);
    __syncthreads();  // (the last reads of part)
    if (lane() == 0) part[wave] = sum;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        if (i < wave) before += part[i];
        total += part[i];
    }
    return before + x;
}

// the last i in [0, n) with pre[i] <= p (pre ascending, pre[0] = 0); rows without triples share their
// prefix with the next one and are skipped that way
__device__ __forceinline__ int row_of(const int *pre, int n, int p) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct SmallArgs {
    int Q, hops, more, want_counts, walk_exact, force_push;  // more: the search is deeper than `hops`
    int32_t E;
    long long T, num_seeds, plane, actw;
    const long long *seed_off;
    const int32_t *seeds;
    const uint32_t *out_off;
    const int32_t *out_obj;
    const uint16_t *out_rel;
    const unsigned long long *allow;
    unsigned long long *visited, *levels;
    uint32_t *act;
    long long *kept_off;
    int32_t *kept_seeds;
    int32_t *ent;      // [kSmallEntities] reached entities, ascending
    long long *off;    // [65] offsets of the lists
    SmallReport *rep;  // pinned host memory
    unsigned long long *live;  // [levels][16] live words, of the level the general path goes on with (or NULL)
};

// ids[0 .. n) in ascending order (different ids, n <= kSmallEntities), by all threads of a block of kSmallThreads; behind it
// the block has met at a barrier.  tmp: kSmallEntities ints, count: 2 kSmallThreads ints.  The ids are dealt to one bucket per
// thread by their place between the smallest and the largest, and ranked inside their bucket: eight barriers where
// a bitonic sort of 2,048 ids has 66 (64 questions on 10,000 entities: k_small_search 41 -> 27 us).  That sort remains for ids
// so uneven that a bucket gets more than kSortBucket.
constexpr int kSortBucket = 32;

__device__ __forceinline__ void sort_ids(int32_t *ids, int n, int32_t *tmp, int *count, int *part, unsigned int *flag) {
    const int t = threadIdx.x;
    int *start = count + kSmallThreads;
    constexpr int PER = kSmallEntities / kSmallThreads;
    int32_t lo = INT_MAX, not_hi = INT_MAX;  // (~largest)
    __syncthreads();  // (the last use of tmp, count and *flag)
    for (int i = t; i < n; i += kSmallThreads) {
        lo = min(lo, ids[i]);
        not_hi = min(not_hi, ~ids[i]);
    }
    count[t] = 0;
    if (t == 0) {
        tmp[0] = tmp[1] = INT_MAX;
        *flag = 0;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        lo = min(lo, __shfl_xor(lo, m));
        not_hi = min(not_hi, __shfl_xor(not_hi, m));
    }
    __syncthreads();
    if (lane() == 0 && lo != INT_MAX) {
        atomicMin(&tmp[0], lo);
        atomicMin(&tmp[1], not_hi);
    }
    __syncthreads();
    lo = tmp[0];
    const unsigned long long span = (unsigned long long)((unsigned)~tmp[1] - (unsigned)lo) + 1ull;
    const unsigned long long scale = ((unsigned long long)kSmallThreads << 32) / span;  // (x < span: x * scale >> 32 < kSmallThreads)
    int32_t id[PER];
    int bucket[PER], rank[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = t + u * kSmallThreads;
        bucket[u] = -1;
        if (i < n) {
            id[u] = ids[i];
            bucket[u] = (int)((((unsigned)id[u] - (unsigned)lo) * scale) >> 32);
            rank[u] = atomicAdd(&count[bucket[u]], 1);
        }
    }
    __syncthreads();
    const int c = count[t];
    if (c > kSortBucket) *flag = 1;
    int total;
    start[t] = block_excl_scan<kSmallThreads>(c, part, total);
    __syncthreads();
    if (*flag) {  // block-uniform: bitonic over the next power of two
        int pow2 = 64;
        while (pow2 < n) pow2 <<= 1;
        for (int i = n + t; i < pow2; i += kSmallThreads) ids[i] = INT_MAX;
        for (int size = 2; size <= pow2; size <<= 1)
            for (int d = size >> 1; d > 0; d >>= 1) {
                __syncthreads();
                for (int p = t; p < pow2 / 2; p += kSmallThreads) {
                    const int i = ((p & -d) << 1) | (p & (d - 1)), j = i + d;
                    const int32_t x = ids[i], y = ids[j];
                    if ((x > y) == ((i & size) == 0)) {
                        ids[i] = y;
                        ids[j] = x;
                    }
                }
            }
        __syncthreads();
        return;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (bucket[u] >= 0) tmp[start[bucket[u]] + rank[u]] = id[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (bucket[u] < 0) continue;
        const int first = start[bucket[u]], k = count[bucket[u]];
        int smaller = 0;
        for (int i = 0; i < k; ++i) smaller += tmp[first + i] < id[u];
        ids[first + smaller] = id[u];
    }
    __syncthreads();
}

// One word per entity.  A level's list is bounded by the triples pushed into it, the list of all
// reached entities by the sum: both are checked before a hop is taken.
__global__ void __launch_bounds__(kSmallThreads) k_small_search(SmallArgs a) {
    __shared__ int32_t s_list[2][kSmallEdges];
    __shared__ int s_pre[kSmallEdges];
    __shared__ unsigned long long s_line[kSmallEdges];
    __shared__ int32_t s_all[kSmallEntities];
    __shared__ int part[16], s_n[2], s_nall, s_err;
    __shared__ unsigned int s_work;
    __shared__ int s_rows, s_tail, s_seg;
    __shared__ int s_count[64];
    __shared__ long long s_off[65];
    const int t = threadIdx.x;
    if (t == 0) s_n[0] = s_n[1] = s_nall = s_err = 0;
    if (t < 64) s_count[t] = 0;
    __syncthreads();
    // ---- seeds: a thread each
    if (t <= a.Q) {
        const long long x = a.seed_off[t];
        s_off[t] = x;
        a.kept_off[t] = x;
    }
    __syncthreads();
    if (t < a.Q) {
        const long long lo = s_off[t], hi = s_off[t + 1];
        if (lo < 0 || hi < lo || hi > a.num_seeds || (t == 0 && lo != 0) || (t == a.Q - 1 && hi != a.num_seeds)) atomicOr(&s_err, 1);
    }
    __syncthreads();
    if (!s_err)
        for (int i = t; i < (int)a.num_seeds; i += kSmallThreads) {
            const int32_t e = a.seeds[i];
            a.kept_seeds[i] = e;
            if ((uint32_t)e >= (uint32_t)a.E) {
                atomicOr(&s_err, 2);
                continue;
            }
            int lo = 0, hi = a.Q - 1;  // the seed's query: the last one that starts at or before it
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_off[mid] <= i) lo = mid;
                else hi = mid - 1;
            }
            const unsigned long long bit = 1ull << lo;
            atomicOr(&a.levels[e], bit);
            atomicOr(&a.visited[e], bit);
            const uint32_t b = 1u << (e & 31);
            if (!(atomicOr(&a.act[e >> 5], b) & b)) {
                s_list[0][atomicAdd(&s_n[0], 1)] = e;  // at most num_seeds <= kSmallEdges
                s_all[atomicAdd(&s_nall, 1)] = e;
            }
        }
    drain_writes();
    __syncthreads();
    int h = 0, cur = 0, status = kSmallDone;
    if (s_err) {
        if (t == 0) {
            a.rep->status = kSmallBad;
            a.rep->err = s_err;
        }
        return;
    }
    for (int i = t; i < s_n[0]; i += kSmallThreads) s_line[i] = load_l2(&a.levels[s_list[0][i]]);
    // ---- hops
    for (;; ++h) {
        // the frontier's rows: where each starts in their concatenation, and what a general hop wants to know
        // (the length of s_all is read ahead of the barriers below: the pushes behind them grow it, and the
        // decision between them has to be the same in every wavefront)
        const int n = s_n[cur], n_all = s_nall;
        int edges = 0;
        __syncthreads();
        if (t == 0) {
            s_work = 0;
            s_rows = s_tail = s_seg = 0;
            s_n[cur ^ 1] = 0;
        }
        __syncthreads();
        bool large = false;
        for (int i0 = 0; i0 < n; i0 += kSmallThreads) {  // block-uniform
            const int i = i0 + t;
            uint32_t d = 0;
            if (i < n) d = a.out_off[s_list[cur][i] + 1] - a.out_off[s_list[cur][i]];
            const int dc = (int)min(d, (uint32_t)kSmallEdges + 1u);  // (a sum of capped degrees cannot overflow)
            int sum;
            const int x = block_excl_scan<kSmallThreads>(dc, part, sum);
            if (i < n) s_pre[i] = min(edges + x, kSmallEdges + 1);
            edges = min(edges + sum, 1 << 24);
            if (d > 0) {
                atomicAdd(&s_rows, 1);
                if (d <= (uint32_t)kTailMaxDegree) atomicAdd(&s_tail, 1);
                else atomicAdd(&s_seg, (int)((d + kPushSegment - 1) / kPushSegment));
                atomicAdd(&s_work, (unsigned)dc * (unsigned)__popcll(s_line[i]));
            }
        }
        __syncthreads();
        const int rows = s_rows;
        if (t == 0) a.rep->reached[h] = n;
        const bool last = h == a.hops;
        if (rows == 0 || (last && !a.more)) break;
        large = last || edges > kSmallEdges || s_work > (unsigned)kSmallPairs || n_all + edges > kSmallEntities ||
                (!a.force_push && (long long)edges * 12 > a.T);
        if (large) {
            // the general path goes on with this frontier: its exact size
            unsigned long long fe = 0;
            for (int i = t; i < n; i += kSmallThreads) fe += a.out_off[s_list[cur][i] + 1] - a.out_off[s_list[cur][i]];
            fe = (unsigned long long)wave_sum((long long)fe);
            unsigned long long lv = 0;  // the queries whose frontier has an out-edge
            for (int i = t; i < n; i += kSmallThreads)
                if (a.out_off[s_list[cur][i] + 1] > a.out_off[s_list[cur][i]]) lv |= s_line[i];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) lv |= shfl_xor64(lv, m);
            unsigned long long *sum = s_line;  // (not needed any more)
            __syncthreads();
            if (lane() == 0) {
                sum[t >> 6] = fe;
                sum[16 + (t >> 6)] = lv;
            }
            __syncthreads();
            if (t == 0) {
                fe = lv = 0;
                for (int i = 0; i < kSmallThreads / 64; ++i) {
                    fe += sum[i];
                    lv |= sum[16 + i];
                }
                if (a.live) a.live[(size_t)16 * h] = lv;
                a.rep->rows[h] = rows;
                a.rep->edges[h] = (long long)fe;
                a.rep->n_tail = s_tail;
                a.rep->n_seg = s_seg;
            }
            status = kSmallGoOn;
            break;
        }
        if (t == 0) {
            a.rep->rows[h] = rows;
            a.rep->edges[h] = edges;
        }
        unsigned long long *lv = a.levels + (size_t)(h + 1) * a.plane;
        uint32_t *act = a.act + (size_t)(h + 1) * a.actw;
        for (int p = t; p < edges; p += kSmallThreads) {
            const int i = row_of(s_pre, n, p);
            const uint32_t j = a.out_off[s_list[cur][i]] + (uint32_t)(p - s_pre[i]);
            const int32_t o = a.out_obj[j];
            unsigned long long m = s_line[i];
            if (a.allow) m &= a.allow[a.out_rel[j]];
            if (!m) continue;
            const unsigned long long vis = load_l2(&a.visited[o]);  // changes between the hops only
            if (!a.walk_exact) m &= ~vis;
            if (!m) continue;
            if (!(m & ~atomicOr(&lv[o], m))) continue;  // (whoever set these bits marks the object as well)
            const uint32_t b = 1u << (o & 31);
            if (!(atomicOr(&act[o >> 5], b) & b)) {  // one thread per object comes by here
                s_list[cur ^ 1][atomicAdd(&s_n[cur ^ 1], 1)] = o;
                if (!vis) s_all[atomicAdd(&s_nall, 1)] = o;
            }
        }
        drain_writes();
        __syncthreads();
        cur ^= 1;
        const int m = s_n[cur];
        for (int i = t; i < m; i += kSmallThreads) {
            const int32_t o = s_list[cur][i];
            const unsigned long long x = load_l2(&lv[o]);
            s_line[i] = x;
            atomicOr(&a.visited[o], x);
        }
        drain_writes();
        __syncthreads();
    }
    if (t == 0) {
        a.rep->status = status;
        a.rep->err = 0;
        a.rep->hops = h;
        a.rep->n_all = s_nall;
    }
    if (status != kSmallDone || !a.want_counts) return;
    // ---- reached entities in ascending order, counts per query
    const int n = s_nall;
    sort_ids(s_all, n, &s_list[0][0], s_pre, part, &s_work);
    for (int i0 = (t & ~63); i0 < n; i0 += kSmallThreads) {  // wavefront-uniform: lane = entity, then lane = query
        const int i = i0 + lane();
        unsigned long long x = 0;
        if (i < n) {
            a.ent[i] = s_all[i];
            x = load_l2(&a.visited[s_all[i]]);
        }
        atomicAdd(&s_count[lane()], __popcll(transpose64(x)));
    }
    __syncthreads();
    if (t < 64) {
        int total;
        const int c = s_count[t], x = wave_excl_scan(c, total);
        a.off[t] = x;
        a.rep->off[t] = x;
        if (t == 63) {
            a.off[64] = total;
            a.rep->off[64] = total;
        }
    }
}

// One block per fetched query: its reached entities (ascending), their hops, and the smallest
// triple index from an entity one hop closer.
constexpr int kFetchThreads = 256;

__global__ void __launch_bounds__(kFetchThreads)
k_small_fetch(int q0, int n_all, int k, int last_level, long long plane, const int32_t *__restrict__ ent,
              const long long *__restrict__ off, const unsigned long long *__restrict__ visited,
              const unsigned long long *__restrict__ levels, const unsigned long long *__restrict__ allow,
              const uint32_t *__restrict__ out_off, const int32_t *__restrict__ out_obj,
              const uint16_t *__restrict__ out_rel, const int32_t *__restrict__ out_eid, int32_t *__restrict__ entity,
              uint8_t *__restrict__ hop, int32_t *__restrict__ pred) {
    __shared__ int32_t s_ent[kSmallEntities];
    __shared__ uint8_t s_hop[kSmallEntities];
    __shared__ int32_t s_pred[kSmallEntities];
    __shared__ int s_pre[kSmallEntities];
    __shared__ int part[kFetchThreads / 64];
    const int q = q0 + blockIdx.x, t = threadIdx.x;
    const unsigned long long bit = 1ull << q;
    int n = 0;
    for (int i0 = 0; i0 < n_all; i0 += kFetchThreads) {  // block-uniform
        const int i = i0 + t;
        int32_t e = 0;
        bool in = false;
        if (i < n_all) {
            e = ent[i];
            in = (visited[e] & bit) != 0ull;
        }
        int total;
        const int at = n + block_excl_scan<kFetchThreads>(in ? 1 : 0, part, total);
        n += total;
        if (in) {
            int h = 0;
            if (hop || pred)  // (entities alone: no look at the levels)
                while (h < last_level && !(levels[(size_t)h * plane + e] & bit)) ++h;
            s_ent[at] = e;
            s_hop[at] = (uint8_t)h;
            s_pred[at] = h == 0 ? -1 : INT_MAX;
        }
    }
    __syncthreads();
    if (pred) {
        int edges = 0;
        for (int i0 = 0; i0 < n; i0 += kFetchThreads) {
            const int i = i0 + t;
            int d = 0;
            if (i < n && (int)s_hop[i] < k) d = (int)(out_off[s_ent[i] + 1] - out_off[s_ent[i]]);
            int total;
            const int x = block_excl_scan<kFetchThreads>(d, part, total);
            if (i < n) s_pre[i] = edges + x;
            edges += total;
        }
        __syncthreads();
        for (int p = t; p < edges; p += kFetchThreads) {
            const int i = row_of(s_pre, n, p);
            const uint32_t j = out_off[s_ent[i]] + (uint32_t)(p - s_pre[i]);
            const int32_t o = out_obj[j];
            if (allow && !(allow[out_rel[j]] & bit)) continue;
            int lo = 0, hi = n;  // o's place in the list
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (s_ent[mid] < o) lo = mid + 1;
                else hi = mid;
            }
            if (lo < n && s_ent[lo] == o && s_hop[lo] == s_hop[i] + 1) atomicMin(&s_pred[lo], out_eid[j]);
        }
        __syncthreads();
    }
    const long long base = off[q] - off[q0];
    for (int i = t; i < n; i += kFetchThreads) {
        entity[base + i] = s_ent[i];
        if (hop) hop[base + i] = s_hop[i];
        if (pred) pred[base + i] = s_pred[i];
    }
}

}  // namespace

logoskg_status small_search(logoskg_graph *g, logoskg_result *r, const logoskg_query_batch *b, bool want_counts,
                            bool force_push, int *next_hop, hipStream_t st) {
    LKG_TRY(g->pool.alloc((void **)&r->small_off, 65 * 8 + (size_t)kSmallEntities * 4, st));
    r->small_ent = reinterpret_cast<int32_t *>(r->small_off + 65);
    SmallArgs a = {};
    a.Q = r->Q; a.hops = std::min(r->k, kSmallHops); a.more = r->k > kSmallHops;
    // (the lists' predecessors come from SUB's triple indices: a graph that does not hold them - built on the host -
    // keeps to the general kernels' tables, so that a fetch allocates nothing and waits for nothing)
    a.want_counts = want_counts && !a.more && g->out_eid;
    a.walk_exact = r->walk_exact; a.force_push = force_push;
    a.E = g->E; a.T = g->T; a.num_seeds = b->num_seeds; a.plane = r->Epad; a.actw = r->Epad / 32;
    a.seed_off = reinterpret_cast<const long long *>(b->seed_off); a.seeds = b->seeds;
    a.out_off = g->out_off; a.out_obj = g->out_obj; a.out_rel = g->out_rel;
    a.allow = r->has_mask ? r->allow : nullptr;
    a.visited = r->visited; a.levels = r->levels; a.act = r->act;
    a.kept_off = r->seed_off; a.kept_seeds = r->seeds;
    a.ent = r->small_ent; a.off = r->small_off; a.rep = g->h_small; a.live = r->live;
    {
        ProfScope ps(g->prof, KK_SEED, st);
        k_small_search<<<dim3(1), dim3(kSmallThreads), 0, st>>>(a);
    }
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipStreamSynchronize(st));
    const SmallReport &rep = *g->h_small;
    if (rep.status == kSmallBad) {
        set_error("seed_off / seeds are inconsistent or out of range (device check, code %d)", rep.err);
        return LOGOSKG_EINVAL;
    }
    for (int h = 0; h < rep.hops; ++h) {
        logoskg_hop_stats &hs = r->stats[(size_t)h];
        hs.direction = LOGOSKG_DIR_PUSH;
        hs.shards_touched = 1;
        hs.active_rows = rep.rows[h];
        hs.frontier_edges = hs.edges_scanned = hs.lines_gathered = rep.edges[h];
        hs.entities_reached = rep.reached[h + 1];
    }
    if (rep.status == kSmallGoOn) {
        g->h_ctr[C_NROWS] = (unsigned long long)rep.rows[rep.hops];
        g->h_ctr[C_FEDGES] = (unsigned long long)rep.edges[rep.hops];
        g->h_ctr[C_NTAIL] = (unsigned long long)rep.n_tail;
        g->h_ctr[C_NSEG] = (unsigned long long)rep.n_seg;
        *next_hop = rep.hops + 1;
        return LOGOSKG_OK;
    }
    *next_hop = r->k + 1;
    if (a.want_counts) {
        r->reached_off.assign(rep.off, rep.off + r->Q + 1);
        r->has_counts = true;
        r->small_n = rep.n_all;
        r->small_levels = rep.hops;
    }
    return LOGOSKG_OK;
}

logoskg_status small_fetch(logoskg_result *r, int q0, int q1, int32_t *entity, uint8_t *hop, int32_t *pred,
                           hipStream_t st) {
    logoskg_graph *g = r->g;
    ProfScope ps(g->prof, KK_PRED, st);
    k_small_fetch<<<dim3((unsigned)(q1 - q0)), dim3(kFetchThreads), 0, st>>>(
        q0, (int)r->small_n, r->k, r->small_levels, r->Epad, r->small_ent, r->small_off, r->visited, r->levels,
        r->has_mask ? r->allow : nullptr, g->out_off, g->out_obj, g->out_rel, g->out_eid, entity, hop, pred);
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

}  // namespace lkg
