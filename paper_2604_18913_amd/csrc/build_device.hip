// Device-side part of logoskg_build: the two stable sorts of the triple list
// (by subject for SUB, by object for OBJ, Sec. 3.2, Eq. 1-3) run on the GPU, for
// a resident graph (the sorted arrays stay in HBM) and for a sharded one (the
// sorted arrays go to pinned host memory, the subject order grouped by shard).  A least-significant-digit radix sort of (key, triple index)
// pairs is stable, so triple indices ascend inside a row exactly as in the host
// counting sort; the row offsets come from a histogram and a prefix sum.  The
// sort and the scan are rocPRIM's device-wide primitives; everything else is a
// handful of streaming kernels.
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "common.h"

namespace lkg {

// Device temporaries, freed on every way out.  With an arena they are pieces of one block, which the steps of a build use
// one after the other (restart): taking and giving back each by itself was a millisecond on 3.4M triples.
struct Scratch {
    std::vector<void *> ptrs;
    char *arena = nullptr;
    size_t size = 0, used = 0;
    ~Scratch() { release(); }
    void reserve(size_t bytes) {  // (without room for it the pieces are taken by themselves)
        if (hipMalloc((void **)&arena, bytes) == hipSuccess) {
            ptrs.push_back(arena);
            size = bytes;
        } else {
            (void)hipGetLastError();
            arena = nullptr;
        }
    }
    void restart() { used = 0; }
    void release() {
        for (void *p : ptrs)
            if (p) (void)hipFree(p);
        ptrs.clear();
        arena = nullptr;
        size = used = 0;
    }
    static size_t rounded(size_t bytes) { return (std::max<size_t>(bytes, 1) + 255) / 256 * 256; }
    template <typename T>
    logoskg_status get(T **p, size_t n) {
        const size_t bytes = rounded(n * sizeof(T));
        if (used + bytes <= size) {
            *p = reinterpret_cast<T *>(arena + used);
            used += bytes;
            return LOGOSKG_OK;
        }
        LKG_HIP(hipMalloc((void **)p, bytes));
        ptrs.push_back(*p);
        return LOGOSKG_OK;
    }
};

namespace {

constexpr int kBlock = 256;

inline unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + kBlock - 1) / kBlock); }

// index of the first triple with an id out of range (INT64_MAX-like sentinel = none)
__global__ void k_check_triples(const int32_t *__restrict__ subj, const int32_t *__restrict__ rel,
                                const int32_t *__restrict__ obj, long long T, int32_t E, int32_t R,
                                unsigned long long *first_bad) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    if ((uint32_t)subj[t] >= (uint32_t)E || (uint32_t)obj[t] >= (uint32_t)E || (uint32_t)rel[t] >= (uint32_t)R)
        atomicMin(first_bad, (unsigned long long)t);
}

__global__ void k_iota(uint32_t *v, long long n) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = (uint32_t)i;
}

// cnt[key + 1] += 1: after an inclusive prefix sum cnt[e] is the first place of row e
__global__ void k_degrees(const int32_t *__restrict__ key, long long T, uint32_t *cnt) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) atomicAdd(&cnt[key[t] + 1], 1u);
}

__global__ void k_gather_sub_rows(const uint32_t *__restrict__ eid, long long T, const int32_t *__restrict__ obj,
                                  const int32_t *__restrict__ rel, int32_t *out_obj, uint16_t *out_rel) {
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= T) return;
    const uint32_t t = eid[p];
    out_obj[p] = obj[t];
    out_rel[p] = (uint16_t)rel[t];
}

// (in_eid NULL: the triple indices stay in eid)
__global__ void k_gather_obj_rows(const uint32_t *__restrict__ eid, long long T, const int32_t *__restrict__ subj,
                                  const int32_t *__restrict__ rel, int32_t *in_sub, uint16_t *in_rel,
                                  int32_t *in_eid) {
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= T) return;
    const uint32_t t = eid[p];
    in_sub[p] = subj[t];
    in_rel[p] = (uint16_t)rel[t];
    if (in_eid) in_eid[p] = (int32_t)t;
}

// subject_of[t] = subject of triple t, from the object-sorted arrays (which keep the triple index)
__global__ void k_subject_of_triple(const int32_t *__restrict__ in_sub, const int32_t *__restrict__ in_eid,
                                    long long T, uint32_t *subject_of) {
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < T) subject_of[in_eid[p]] = (uint32_t)in_sub[p];
}

// The one instantiation of the 32-bit sort, for rows, in-degrees and classes.  The sorts are most of what a process's first
// build on the device loads: with a byte-wide, a descending and a const-keyed one beside it they were 9.9 MB and a first build
// of 500,000 / 3.4M triples took 48 / 55 ms; 5.5 MB and 31 / 36 ms, later builds the same.  (The sort only reads keys and vals.)
hipError_t sort_u32(void *d_tmp, size_t &bytes, const uint32_t *keys, uint32_t *keys_out, const uint32_t *vals, uint32_t *vals_out, int64_t n, unsigned bits,
                    hipStream_t stream = nullptr) {
    return rocprim::radix_sort_pairs(d_tmp, bytes, const_cast<uint32_t *>(keys), keys_out, const_cast<uint32_t *>(vals), vals_out, (size_t)n, 0u, bits, stream);
}

hipError_t sort_u32(void *d_tmp, size_t &bytes, rocprim::double_buffer<uint32_t> &keys, rocprim::double_buffer<uint32_t> &vals, int64_t n, unsigned bits) {
    return rocprim::radix_sort_pairs(d_tmp, bytes, keys, vals, (size_t)n, 0u, bits);
}

// sorted_eid = triple indices in (key, index) order; off = row offsets of that order
logoskg_status sort_by(const int32_t *d_key, int64_t T, int32_t E, unsigned key_bits, uint32_t *d_iota,
                       uint32_t *d_keys_out, uint32_t *d_sorted_eid, uint32_t *d_off, void *d_tmp, size_t tmp_bytes) {
    LKG_HIP(hipMemsetAsync(d_off, 0, ((size_t)E + 1) * sizeof(uint32_t), nullptr));
    if (T > 0) {
        k_degrees<<<dim3(grid_for(T)), dim3(kBlock)>>>(d_key, T, d_off);
        size_t need = tmp_bytes;
        LKG_HIP(sort_u32(d_tmp, need, reinterpret_cast<const uint32_t *>(d_key), d_keys_out, d_iota, d_sorted_eid, T, key_bits));
    }
    size_t need = tmp_bytes;
    LKG_HIP(rocprim::inclusive_scan(d_tmp, need, d_off, d_off, (size_t)E + 1, rocprim::plus<uint32_t>()));
    LKG_HIP(hipGetLastError());
    return LOGOSKG_OK;
}

}  // namespace

static unsigned bits_for(int32_t E) {
    unsigned bits = 1;
    while (bits < 32 && (1ull << bits) < (unsigned long long)E) ++bits;
    return bits;
}

static logoskg_status csr_sort_bytes(int64_t T, int32_t E, size_t *bytes) {
    size_t sort_bytes = 0, scan_bytes = 0;
    uint32_t *none = nullptr;
    LKG_HIP(sort_u32(nullptr, sort_bytes, none, none, none, none, std::max<int64_t>(T, 1), bits_for(E)));
    LKG_HIP(rocprim::inclusive_scan(nullptr, scan_bytes, none, none, (size_t)E + 1, rocprim::plus<uint32_t>()));
    *bytes = std::max(sort_bytes, scan_bytes);
    return LOGOSKG_OK;
}

struct PairBuffers {
    rocprim::double_buffer<unsigned long long> keys{nullptr, nullptr};
    rocprim::double_buffer<uint32_t> vals{nullptr, nullptr}, degrees{nullptr, nullptr}, ids{nullptr, nullptr};
};

static logoskg_status pair_sort_bytes(int64_t T, int32_t E, size_t (&bytes)[3]) {
    PairBuffers b;
    uint32_t *none = nullptr;
    LKG_HIP(rocprim::radix_sort_pairs(nullptr, bytes[0], b.keys, b.vals, (size_t)T, 0u, 2 * bits_for(E)));
    LKG_HIP(sort_u32(nullptr, bytes[1], b.degrees, b.ids, E, 32u));
    LKG_HIP(rocprim::inclusive_scan(nullptr, bytes[2], none, none, 2 * (size_t)T, rocprim::plus<uint32_t>()));
    return LOGOSKG_OK;
}

// One block for the temporaries of a resident graph's build on the device: the two sorts', then the distinct pairs'.
logoskg_status scratch_create(logoskg_graph *g, bool resident, Scratch **out) {
    *out = nullptr;
    std::unique_ptr<Scratch> s(new (std::nothrow) Scratch());
    if (!s) { set_error("out of host memory"); return LOGOSKG_ENOMEM; }
    const int64_t T = g->T;
    if (!resident) {
        *out = s.release();
        return LOGOSKG_OK;
    }
    size_t csr = 0, pair[3] = {};
    LKG_TRY(csr_sort_bytes(T, g->E, &csr));
    if (T > 0) LKG_TRY(pair_sort_bytes(T, g->E, pair));
    const size_t for_sorts = (size_t)T * 20 + csr;
    const size_t for_pairs = (size_t)T * 24 + (size_t)g->E * 16 + std::max({pair[0], pair[1], pair[2]});
    size_t bytes = std::max(for_sorts, for_pairs) + 16 * 256;
    constexpr size_t kNeverShort = (size_t)256 << 20;
    if (bytes > kNeverShort) {  // no more than the sorts take where the graph's own arrays need the room
        const size_t arrays = (size_t)T * 20 + (size_t)g->E * 40;
        size_t free_bytes = 0, all_bytes = 0;
        if (hipMemGetInfo(&free_bytes, &all_bytes) != hipSuccess) (void)hipGetLastError();
        if (bytes + arrays + arrays / 8 > free_bytes) bytes = for_sorts + 16 * 256;
    }
    s->reserve(bytes);
    *out = s.release();
    return LOGOSKG_OK;
}

void scratch_destroy(Scratch *s) { delete s; }
void scratch_release(Scratch *s) { s->release(); }
size_t scratch_bytes(const Scratch *s) { return s->size; }

// Fills g->out_off/out_obj/out_rel/out_eid and g->in_off/in_sub/in_rel/in_eid from host triple arrays.
logoskg_status build_csr_on_device(logoskg_graph *g, const int32_t *subj, const int32_t *rel, const int32_t *obj, Scratch &tmp) {
    const int64_t T = g->T;
    const int32_t E = g->E;
    tmp.restart();
    int32_t *d_subj = nullptr, *d_rel = nullptr, *d_obj = nullptr;
    uint32_t *d_iota = nullptr, *d_keys = nullptr;
    unsigned long long *d_bad = nullptr;
    LKG_TRY(tmp.get(&d_subj, (size_t)T));
    LKG_TRY(tmp.get(&d_rel, (size_t)T));
    LKG_TRY(tmp.get(&d_obj, (size_t)T));
    LKG_TRY(tmp.get(&d_iota, (size_t)T));
    LKG_TRY(tmp.get(&d_keys, (size_t)T));
    LKG_TRY(tmp.get(&d_bad, 1));
    if (T > 0) {
        LKG_HIP(hipMemcpy(d_subj, subj, (size_t)T * 4, hipMemcpyHostToDevice));
        LKG_HIP(hipMemcpy(d_rel, rel, (size_t)T * 4, hipMemcpyHostToDevice));
        LKG_HIP(hipMemcpy(d_obj, obj, (size_t)T * 4, hipMemcpyHostToDevice));
    }
    const unsigned long long none = ~0ull;
    LKG_HIP(hipMemcpy(d_bad, &none, sizeof(none), hipMemcpyHostToDevice));
    if (T > 0) {
        k_check_triples<<<dim3(grid_for(T)), dim3(kBlock)>>>(d_subj, d_rel, d_obj, T, E, g->R, d_bad);
        k_iota<<<dim3(grid_for(T)), dim3(kBlock)>>>(d_iota, T);
    }
    unsigned long long bad = none;
    LKG_HIP(hipMemcpy(&bad, d_bad, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad != none) {
        set_error("triple %llu = (%d, %d, %d) is out of range", bad, subj[bad], rel[bad], obj[bad]);
        return LOGOSKG_EINVAL;
    }
    const unsigned key_bits = bits_for(E);
    size_t tmp_bytes = 0;  // one temporary buffer that serves the sort and the scan
    LKG_TRY(csr_sort_bytes(T, E, &tmp_bytes));
    char *d_tmp = nullptr;
    LKG_TRY(tmp.get(&d_tmp, tmp_bytes));

    // (the arrays of a small graph are one allocation: eight of them are 60 us of a build of half a millisecond)
    constexpr size_t kSmallArrays = (size_t)16 << 20;
    const size_t all = 2 * Scratch::rounded(((size_t)E + 1) * 4) + 4 * Scratch::rounded((size_t)T * 4) + 2 * Scratch::rounded((size_t)T * 2);
    char *at = nullptr;
    auto keep = [&](void **p, size_t bytes) -> logoskg_status {
        if (g->csr_block) {
            *p = at;
            at += Scratch::rounded(bytes);
            return LOGOSKG_OK;
        }
        LKG_HIP(hipMalloc(p, std::max<size_t>(bytes, 4)));
        g->static_bytes += std::max<size_t>(bytes, 4);
        return LOGOSKG_OK;
    };
    if (all <= kSmallArrays) {
        LKG_HIP(hipMalloc(&g->csr_block, all));
        g->static_bytes += all;
        at = static_cast<char *>(g->csr_block);
    }
    // Both sorts leave the triple indices where the graph keeps them, so that they need no column of their own beside
    // it (40 bytes per triple and the sort's buffers at the peak; 44 with one).
    // SUB: rows by subject
    LKG_TRY(keep((void **)&g->out_off, ((size_t)E + 1) * 4));
    LKG_TRY(keep((void **)&g->out_obj, (size_t)T * 4));
    LKG_TRY(keep((void **)&g->out_rel, (size_t)T * 2));
    LKG_TRY(keep((void **)&g->out_eid, (size_t)T * 4));
    uint32_t *const d_out_eid = reinterpret_cast<uint32_t *>(g->out_eid);
    LKG_TRY(sort_by(d_subj, T, E, key_bits, d_iota, d_keys, d_out_eid, g->out_off, d_tmp, tmp_bytes));
    if (T > 0) k_gather_sub_rows<<<dim3(grid_for(T)), dim3(kBlock)>>>(d_out_eid, T, d_obj, d_rel, g->out_obj, g->out_rel);
    // OBJ: rows by object, triple indices kept as edge ids
    LKG_TRY(keep((void **)&g->in_off, ((size_t)E + 1) * 4));
    LKG_TRY(keep((void **)&g->in_sub, (size_t)T * 4));
    LKG_TRY(keep((void **)&g->in_rel, (size_t)T * 2));
    LKG_TRY(keep((void **)&g->in_eid, (size_t)T * 4));
    uint32_t *const d_in_eid = reinterpret_cast<uint32_t *>(g->in_eid);
    LKG_TRY(sort_by(d_obj, T, E, key_bits, d_iota, d_keys, d_in_eid, g->in_off, d_tmp, tmp_bytes));
    if (T > 0)
        k_gather_obj_rows<<<dim3(grid_for(T)), dim3(kBlock)>>>(d_in_eid, T, d_subj, d_rel, g->in_sub, g->in_rel, nullptr);
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipDeviceSynchronize());
    return LOGOSKG_OK;
}

// ---------------------------------------------------------------- distinct pairs
// One stable radix sort of (object, rank of the subject by in-degree) keys with the positions of OBJ as values: equal
// keys are parallel triples, the first of them has the smallest triple index, and the keys' order is pull_sub's.  A row
// keeps its extent in the sorted order, so prefix sums over the first ones of each run give the rows of both orders.
__global__ void k_row_starts(const uint32_t *__restrict__ off, int32_t E, uint32_t *obj_of) {
    const int32_t e = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (e < E && off[e + 1] > off[e]) obj_of[off[e]] = (uint32_t)e;
}

// (inverted: the sort ascends, the highest degree comes first)
__global__ void k_in_degrees(const uint32_t *__restrict__ off, int32_t E, uint32_t *deg) {
    const int32_t e = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (e < E) deg[e] = ~(off[e + 1] - off[e]);
}

__global__ void k_rank_of(const uint32_t *__restrict__ by_rank, int32_t E, uint32_t *rank_of) {
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < E) rank_of[by_rank[i]] = (uint32_t)i;
}

// (obj_of NULL: the last row that begins at or before p; rank_of NULL: the subjects by id)
__global__ void k_pair_keys(const uint32_t *__restrict__ obj_of, const uint32_t *__restrict__ off, int32_t E, const int32_t *__restrict__ in_sub,
                            const uint32_t *__restrict__ rank_of, long long T, unsigned bits, unsigned long long *key, uint32_t *pos) {
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= T) return;
    uint32_t o = 0;
    if (obj_of) {
        o = obj_of[p];
    } else {
        for (uint32_t hi = (uint32_t)E; hi - o > 1;) {
            const uint32_t m = o + (hi - o) / 2;
            if (off[m] <= p) o = m; else hi = m;
        }
    }
    const uint32_t s = (uint32_t)in_sub[p];
    key[p] = ((unsigned long long)o << bits) | (rank_of ? rank_of[s] : s);
    pos[p] = (uint32_t)p;
}

// is_new[i]: the i-th key differs from the one before; is_first[p]: position p of OBJ holds the first triple of its pair
__global__ void k_pair_flags(const unsigned long long *__restrict__ key, const uint32_t *__restrict__ pos, long long T,
                             uint32_t *is_new, uint32_t *is_first) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T) return;
    const uint32_t n = i == 0 || key[i] != key[i - 1];
    is_new[i] = n;
    is_first[pos[i]] = n;
}

// (the flags have become inclusive prefix sums, is_first's behind is_new's)
__global__ void k_pair_rows(const uint32_t *__restrict__ off, int32_t E, const uint32_t *__restrict__ new_upto, uint32_t *pair_off) {
    const int32_t e = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (e <= E) pair_off[e] = off[e] ? new_upto[off[e] - 1] : 0u;
}

__global__ void k_pair_fill(const unsigned long long *__restrict__ key, const uint32_t *__restrict__ new_upto,
                            const uint32_t *__restrict__ first_upto, long long T, unsigned bits,
                            const uint32_t *__restrict__ by_rank, const int32_t *__restrict__ in_sub,
                            const int32_t *__restrict__ in_eid, int32_t *pull_sub, int32_t *sub, int32_t *eid,
                            const uint32_t *__restrict__ pos, const uint16_t *__restrict__ in_rel, int32_t *all_sub, uint16_t *all_rel) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T) return;
    const uint32_t pairs = new_upto[T - 1], n = new_upto[i], f = first_upto[i] - pairs;
    const uint32_t of_key = (uint32_t)(key[i] & ((1ull << bits) - 1ull));
    const int32_t s = (int32_t)(by_rank ? by_rank[of_key] : of_key);
    all_sub[i] = s;
    all_rel[i] = in_rel[pos[i]];
    if (n != (i ? new_upto[i - 1] : 0u)) pull_sub[n - 1] = s;
    if (f != (i ? first_upto[i - 1] - pairs : 0u)) {
        sub[f - 1] = in_sub[i];
        eid[f - 1] = in_eid[i];
    }
}

// Graphs up to so many triples have pull_sub by id, which takes a dozen launches less; the rows' first subjects matter where a
// hop's lines come from far.  Build of 80,000 / 400,000 / 1.6M triples 804 / 1,881 / 4,091 us by in-degree, 748 / 1,822 / 4,003
// by id; searches of 1 .. 1,024 questions with their lists the same within 1 % (20,000 triples, 1,024 questions: 3 % longer by id).
constexpr int64_t kFewPairTriples = 1 << 21;

logoskg_status build_pairs_on_device(logoskg_graph *g, const int32_t *in_sub, const uint16_t *in_rel, const int32_t *in_eid, Scratch &tmp) {
    const int64_t T = g->T;
    const int32_t E = g->E;
    if (T == 0) return LOGOSKG_OK;
    const unsigned bits = bits_for(E);
    size_t bytes[3] = {};
    LKG_TRY(pair_sort_bytes(T, E, bytes));
    tmp.restart();
    bool room = true;
    auto get = [&](auto **p, size_t n) {  // (without them the graph works as well)
        if (room && tmp.get(p, n) != LOGOSKG_OK) {
            (void)hipGetLastError();
            room = false;
        }
    };
    unsigned long long *key[2] = {};
    uint32_t *pos[2] = {}, *rank[4] = {};
    char *d_tmp = nullptr;
    for (auto &p : key) get(&p, (size_t)T);
    for (auto &p : pos) get(&p, (size_t)T);
    for (auto &p : rank) get(&p, (size_t)E);
    get(&d_tmp, std::max({bytes[0], bytes[1], bytes[2]}));
    if (!room) return LOGOSKG_OK;
    rocprim::double_buffer<unsigned long long> keys(key[0], key[1]);
    rocprim::double_buffer<uint32_t> vals(pos[0], pos[1]), degrees(rank[0], rank[1]), ids(rank[2], rank[3]);

    const dim3 block(kBlock), per_triple(grid_for(T)), per_entity(grid_for((int64_t)E + 1));
    uint32_t *const obj_of = pos[1];
    const bool few = T <= kFewPairTriples;
    if (!few) {
        LKG_HIP(hipMemsetAsync(obj_of, 0, (size_t)T * 4, nullptr));
        k_row_starts<<<per_entity, block>>>(g->in_off, E, obj_of);
        LKG_HIP(rocprim::inclusive_scan(d_tmp, bytes[2], obj_of, obj_of, (size_t)T, rocprim::maximum<uint32_t>()));
        k_in_degrees<<<per_entity, block>>>(g->in_off, E, degrees.current());
        k_iota<<<per_entity, block>>>(ids.current(), E);
        LKG_HIP(sort_u32(d_tmp, bytes[1], degrees, ids, E, 32u));
        k_rank_of<<<per_entity, block>>>(ids.current(), E, degrees.current());
    }
    const uint32_t *const by_rank = few ? nullptr : ids.current();
    k_pair_keys<<<per_triple, block>>>(few ? nullptr : obj_of, g->in_off, E, in_sub, few ? nullptr : degrees.current(), T, bits, key[0], pos[0]);
    LKG_HIP(rocprim::radix_sort_pairs(d_tmp, bytes[0], keys, vals, (size_t)T, 0u, 2 * bits));
    uint32_t *const is_new = reinterpret_cast<uint32_t *>(keys.alternate()), *const is_first = is_new + T;
    k_pair_flags<<<per_triple, block>>>(keys.current(), vals.current(), T, is_new, is_first);
    LKG_HIP(rocprim::inclusive_scan(d_tmp, bytes[2], is_new, is_new, 2 * (size_t)T, rocprim::plus<uint32_t>()));
    LKG_HIP(hipGetLastError());
    uint32_t n = 0;
    LKG_HIP(hipMemcpy(&n, is_new + T - 1, sizeof(n), hipMemcpyDeviceToHost));
    if ((int64_t)n * 100 > T * (T < kPairManyTriples ? kPairShareFew : kPairShare)) return LOGOSKG_OK;

    PairRows p;
    const size_t of_pairs = Scratch::rounded((size_t)n * 4), of_triples = Scratch::rounded((size_t)T * 4), of_rels = Scratch::rounded((size_t)T * 2),
                 of_rows = Scratch::rounded(((size_t)E + 1) * 4), all = 3 * of_pairs + of_triples + of_rels + of_rows;
    if (hipMalloc(&p.block, all) != hipSuccess) {
        (void)hipGetLastError();
        return LOGOSKG_OK;
    }
    char *at = static_cast<char *>(p.block);
    auto piece = [&](auto **out, size_t size) {
        *out = reinterpret_cast<std::remove_reference_t<decltype(*out)>>(at);
        at += size;
    };
    piece(&p.pull_sub, of_pairs);
    piece(&p.sub, of_pairs);
    piece(&p.eid, of_pairs);
    piece(&p.all_sub, of_triples);
    piece(&p.all_rel, of_rels);
    piece(&p.off, of_rows);
    g->pairs = p;
    g->static_bytes += all;
    k_pair_rows<<<per_entity, block>>>(g->in_off, E, is_new, p.off);
    k_pair_fill<<<per_triple, block>>>(keys.current(), is_new, is_first, T, bits, by_rank, in_sub, in_eid, p.pull_sub,
                                       p.sub, p.eid, vals.current(), in_rel, p.all_sub, p.all_rel);
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipDeviceSynchronize());  // (the scratch goes)
    return LOGOSKG_OK;
}

// ---------------------------------------------------------------- row classes
// counts[0 .. 2] += rows with an entry, of more than kTailMaxDegree, of at least hub_min
__global__ void __launch_bounds__(kBlock) k_row_counts(const uint32_t *__restrict__ off, int32_t E, uint32_t hub_min, unsigned int *counts) {
    unsigned n[3] = {};
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < E; e += (long long)gridDim.x * kBlock) {
        const uint32_t d = off[e + 1] - off[e];
        n[0] += d > 0;
        n[1] += d > (uint32_t)kTailMaxDegree;
        n[2] += d >= hub_min;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const unsigned x = (unsigned)wave_sum(n[i]);
        if (lane() == 0 && x) atomicAdd(&counts[i], x);
    }
}

logoskg_status count_rows_on_device(const uint32_t *d_off, int32_t E, int hub_min, Scratch &tmp, unsigned int (&n)[3]) {
    unsigned int *d_n = nullptr;
    LKG_TRY(tmp.get(&d_n, 3));
    LKG_HIP(hipMemsetAsync(d_n, 0, sizeof(n), nullptr));
    // (its wavefronts' sums meet in three words: 1,024 blocks over 407,000 rows were 91 us, 128 are 22)
    k_row_counts<<<dim3(std::min(128u, grid_for(E))), dim3(kBlock)>>>(d_off, E, (uint32_t)hub_min, d_n);
    LKG_HIP(hipMemcpy(n, d_n, sizeof(n), hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

// short rows by descending length, then the longer ones, then the empty ones
__global__ void k_row_class(const uint32_t *__restrict__ off, int32_t E, uint32_t *key, uint32_t *id) {
    const long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (e >= E) return;
    const uint32_t d = off[e + 1] - off[e];
    key[e] = d == 0 ? kTailMaxDegree + 1 : d > (uint32_t)kTailMaxDegree ? kTailMaxDegree : kTailMaxDegree - d;
    id[e] = (uint32_t)e;
}

__global__ void k_row_records(const uint32_t *__restrict__ id, long long n, const uint32_t *__restrict__ off, ShortRow *out) {
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) out[i] = ShortRow{(int32_t)id[i], off[id[i]], off[id[i] + 1]};
}

// The rows behind d_off: counts into rc, the short ones by descending length and then the longer ones as records on the
// device (*records, in the scratch), the longer ones on the host as well.  (A stable sort of one digit.  On the host, with
// the offsets copied back, 20M rows were a quarter of a second.)
logoskg_status classify_on_device(const uint32_t *d_off, int32_t E, int hub_min, Scratch &tmp, RowClasses *rc, ShortRow **records, std::vector<ShortRow> *longer) {
    tmp.restart();
    unsigned int n[3];
    LKG_TRY(count_rows_on_device(d_off, E, hub_min, tmp, n));
    rc->n_tail = (int64_t)n[0] - n[1];
    rc->n_hub = n[2];
    longer->resize(n[1]);
    *records = nullptr;
    if (n[0] == 0) return LOGOSKG_OK;
    uint32_t *key[2] = {}, *id[2] = {};
    for (auto &p : key) LKG_TRY(tmp.get(&p, (size_t)E));
    for (auto &p : id) LKG_TRY(tmp.get(&p, (size_t)E));
    rocprim::double_buffer<uint32_t> keys(key[0], key[1]), ids(id[0], id[1]);
    size_t bytes = 0;
    LKG_HIP(sort_u32(nullptr, bytes, keys, ids, E, 6u));
    char *d_tmp = nullptr;
    LKG_TRY(tmp.get(&d_tmp, bytes));
    LKG_TRY(tmp.get(records, n[0]));
    k_row_class<<<dim3(grid_for(E)), dim3(kBlock)>>>(d_off, E, key[0], id[0]);
    LKG_HIP(sort_u32(d_tmp, bytes, keys, ids, E, 6u));
    k_row_records<<<dim3(grid_for(n[0])), dim3(kBlock)>>>(ids.current(), n[0], d_off, *records);
    LKG_HIP(hipGetLastError());
    if (n[1]) LKG_HIP(hipMemcpy(longer->data(), *records + rc->n_tail, (size_t)n[1] * sizeof(ShortRow), hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

// ---------------------------------------------------------------- sharded graphs
// The triple list on the device with the scratch of the sorts, alive during logoskg_build only.
struct TripleSorter {
    int64_t T = 0;
    int32_t E = 0;
    unsigned key_bits = 1;
    Scratch tmp;
    int32_t *d_subj = nullptr, *d_rel = nullptr, *d_obj = nullptr;
    uint32_t *d_iota = nullptr, *d_keys = nullptr, *d_eid = nullptr, *d_off = nullptr, *d_key_in = nullptr;
    int32_t *d_a = nullptr, *d_b = nullptr;  // gathered 4-byte columns
    uint16_t *d_r = nullptr;                 // gathered relation ids
    char *d_tmp = nullptr;
    size_t tmp_bytes = 0;
};

__global__ void k_row_keys(const int32_t *subj, long long T, const uint32_t *__restrict__ row_begin,
                           uint32_t *key) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < T) key[t] = row_begin[subj[t]];
}

logoskg_status sorter_create(logoskg_graph *g, const int32_t *subj, const int32_t *rel, const int32_t *obj,
                             TripleSorter **out) {
    *out = nullptr;
    std::unique_ptr<TripleSorter> s(new (std::nothrow) TripleSorter());
    if (!s) { set_error("out of host memory"); return LOGOSKG_ENOMEM; }
    const int64_t T = g->T;
    s->T = T;
    s->E = g->E;
    unsigned long long *d_bad = nullptr;
    LKG_TRY(s->tmp.get(&s->d_subj, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_rel, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_obj, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_iota, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_keys, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_eid, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_key_in, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_a, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_b, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_r, (size_t)T));
    LKG_TRY(s->tmp.get(&s->d_off, (size_t)g->E + 1));
    LKG_TRY(s->tmp.get(&d_bad, 1));
    if (T > 0) {
        LKG_HIP(hipMemcpy(s->d_subj, subj, (size_t)T * 4, hipMemcpyHostToDevice));
        LKG_HIP(hipMemcpy(s->d_rel, rel, (size_t)T * 4, hipMemcpyHostToDevice));
        LKG_HIP(hipMemcpy(s->d_obj, obj, (size_t)T * 4, hipMemcpyHostToDevice));
    }
    const unsigned long long none = ~0ull;
    LKG_HIP(hipMemcpy(d_bad, &none, sizeof(none), hipMemcpyHostToDevice));
    if (T > 0) {
        k_check_triples<<<dim3(grid_for(T)), dim3(kBlock)>>>(s->d_subj, s->d_rel, s->d_obj, T, g->E, g->R, d_bad);
        k_iota<<<dim3(grid_for(T)), dim3(kBlock)>>>(s->d_iota, T);
    }
    unsigned long long bad = none;
    LKG_HIP(hipMemcpy(&bad, d_bad, sizeof(bad), hipMemcpyDeviceToHost));
    if (bad != none) {
        set_error("triple %llu = (%d, %d, %d) is out of range", bad, subj[bad], rel[bad], obj[bad]);
        return LOGOSKG_EINVAL;
    }
    while (s->key_bits < 32 && (1ull << s->key_bits) < (unsigned long long)g->E) ++s->key_bits;
    size_t sort_bytes = 0, scan_bytes = 0;
    LKG_HIP(sort_u32(nullptr, sort_bytes, s->d_key_in, s->d_keys, s->d_iota, s->d_eid, std::max<int64_t>(T, 1), 32u));
    LKG_HIP(rocprim::inclusive_scan(nullptr, scan_bytes, (uint32_t *)nullptr, (uint32_t *)nullptr, (size_t)g->E + 1,
                                    rocprim::plus<uint32_t>()));
    s->tmp_bytes = std::max(sort_bytes, scan_bytes);
    LKG_TRY(s->tmp.get(&s->d_tmp, s->tmp_bytes));
    *out = s.release();
    return LOGOSKG_OK;
}

void sorter_destroy(TripleSorter *s) { delete s; }

// Row offsets of SUB (by_object = false) or OBJ on the host: off[e] = triples of smaller keys.
logoskg_status sorter_offsets(TripleSorter *s, bool by_object, std::vector<uint32_t> *off) {
    const int32_t *key = by_object ? s->d_obj : s->d_subj;
    LKG_HIP(hipMemsetAsync(s->d_off, 0, ((size_t)s->E + 1) * sizeof(uint32_t), nullptr));
    if (s->T > 0) k_degrees<<<dim3(grid_for(s->T)), dim3(kBlock)>>>(key, s->T, s->d_off);
    size_t need = s->tmp_bytes;
    LKG_HIP(rocprim::inclusive_scan(s->d_tmp, need, s->d_off, s->d_off, (size_t)s->E + 1, rocprim::plus<uint32_t>()));
    off->resize((size_t)s->E + 1);
    LKG_HIP(hipMemcpy(off->data(), s->d_off, ((size_t)s->E + 1) * 4, hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

// Objects and relation ids in the shard-grouped subject order: triples sorted (stably, so triple
// indices ascend inside a subject) by the place where their subject's run begins.
logoskg_status sorter_subject_order(TripleSorter *s, const uint32_t *d_row_begin, int32_t *h_obj, uint16_t *h_rel) {
    const int64_t T = s->T;
    if (T == 0) return LOGOSKG_OK;
    k_row_keys<<<dim3(grid_for(T)), dim3(kBlock)>>>(s->d_subj, T, d_row_begin, s->d_key_in);
    size_t need = s->tmp_bytes;
    LKG_HIP(sort_u32(s->d_tmp, need, s->d_key_in, s->d_keys, s->d_iota, s->d_eid, T, 32u));
    k_gather_sub_rows<<<dim3(grid_for(T)), dim3(kBlock)>>>(s->d_eid, T, s->d_obj, s->d_rel, s->d_a, s->d_r);
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipMemcpy(h_obj, s->d_a, (size_t)T * 4, hipMemcpyDeviceToHost));
    LKG_HIP(hipMemcpy(h_rel, s->d_r, (size_t)T * 2, hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

// Subjects, relation ids and triple indices in object order (rows of OBJ, indices ascending inside a row).
logoskg_status sorter_object_order(TripleSorter *s, int32_t *h_sub, uint16_t *h_rel, int32_t *h_eid) {
    const int64_t T = s->T;
    if (T == 0) return LOGOSKG_OK;
    size_t need = s->tmp_bytes;
    LKG_HIP(sort_u32(s->d_tmp, need, reinterpret_cast<const uint32_t *>(s->d_obj), s->d_keys, s->d_iota, s->d_eid, T, s->key_bits));
    k_gather_obj_rows<<<dim3(grid_for(T)), dim3(kBlock)>>>(s->d_eid, T, s->d_subj, s->d_rel, s->d_a, s->d_r, s->d_b);
    LKG_HIP(hipGetLastError());
    LKG_HIP(hipMemcpy(h_sub, s->d_a, (size_t)T * 4, hipMemcpyDeviceToHost));
    LKG_HIP(hipMemcpy(h_rel, s->d_r, (size_t)T * 2, hipMemcpyDeviceToHost));
    LKG_HIP(hipMemcpy(h_eid, s->d_b, (size_t)T * 4, hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

void sorter_object_arrays(const TripleSorter *s, const int32_t **sub, const uint16_t **rel, const int32_t **eid) {
    *sub = s->d_a;
    *rel = s->d_r;
    *eid = s->d_b;
}

// g->out_eid[p] = index of the triple behind entry p of the subject-sorted CSR (SUB's rows, Eq. 1).
// The build keeps triple indices only with the object-sorted arrays; this repeats the stable sort
// by subject on (subject, triple index) pairs, so the order is the one of out_obj / out_rel.
static logoskg_status build_out_eid(logoskg_graph *g, hipStream_t st) {
    // a sharded graph keeps the object-sorted triples in pinned host memory (read in place here) and
    // its rows of SUB in the shard-grouped order: the sort key is the place where a subject's run begins
    const int32_t *in_sub = g->in_sub, *in_eid = g->in_eid;
    const uint16_t *in_rel = g->in_rel;
    const bool sharded = g->num_shards > 1;
    if (sharded && !shard_in_arrays(g, &in_sub, &in_rel, &in_eid)) {
        set_error("the object-sorted triples of the sharded graph are not available");
        return LOGOSKG_EINTERNAL;
    }
    const int64_t T = g->T;
    Scratch tmp;
    uint32_t *d_subject = nullptr, *d_iota = nullptr, *d_keys = nullptr;
    LKG_TRY(tmp.get(&d_subject, (size_t)T));
    LKG_TRY(tmp.get(&d_iota, (size_t)T));
    LKG_TRY(tmp.get(&d_keys, (size_t)T));
    int32_t *eid = nullptr;
    LKG_HIP(hipMalloc((void **)&eid, std::max<size_t>((size_t)T, 1) * 4));
    auto fail = [&](logoskg_status s) { (void)hipFree(eid); return s; };
    if (T > 0) {
        unsigned key_bits = 1;
        while (key_bits < 32 && (1ull << key_bits) < (unsigned long long)g->E) ++key_bits;
        if (sharded) key_bits = 32;
        k_subject_of_triple<<<dim3(grid_for(T)), dim3(kBlock), 0, st>>>(in_sub, in_eid, T, d_subject);
        if (sharded)
            k_row_keys<<<dim3(grid_for(T)), dim3(kBlock), 0, st>>>(reinterpret_cast<const int32_t *>(d_subject), T,
                                                                   g->row_begin, d_subject);
        k_iota<<<dim3(grid_for(T)), dim3(kBlock), 0, st>>>(d_iota, T);
        size_t bytes = 0;
        hipError_t e = sort_u32(nullptr, bytes, d_subject, d_keys, d_iota, (uint32_t *)eid, T, key_bits, st);
        char *d_tmp = nullptr;
        if (e == hipSuccess && tmp.get(&d_tmp, bytes) != LOGOSKG_OK) return fail(LOGOSKG_ENOMEM);
        if (e == hipSuccess)
            e = sort_u32(d_tmp, bytes, d_subject, d_keys, d_iota, (uint32_t *)eid, T, key_bits, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);  // the temporaries are freed on return
        if (e != hipSuccess) {
            set_error("sort of the triple indices failed: %s", hipGetErrorString(e));
            return fail(LOGOSKG_EDEVICE);
        }
    }
    g->out_eid = eid;
    g->static_bytes += std::max<size_t>((size_t)T, 1) * 4;
    return LOGOSKG_OK;
}

// Callers that can do without them go on after a failure, so it must not be what their own look at the runtime's
// last error finds.
logoskg_status ensure_out_eid(logoskg_graph *g, hipStream_t st) {
    if (g->out_eid) return LOGOSKG_OK;
    logoskg_status s = build_out_eid(g, st);
    if (s == LOGOSKG_ENOMEM) {
        (void)hipGetLastError();
        if (give_up_pairs(g)) s = build_out_eid(g, st);
    }
    if (s != LOGOSKG_OK) (void)hipGetLastError();
    return s;
}

}  // namespace lkg
