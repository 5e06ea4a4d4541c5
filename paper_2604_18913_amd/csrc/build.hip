// logoskg_build: triple list -> device CSR forms of the SUB and OBJ incidence
// matrices (paper Sec. 3.2, Eq. 1-3) plus degree classes.  A resident graph is
// sorted on the GPU (build_device.hip); the host counting sorts below serve
// sharded graphs, whose edge arrays stay in host memory, and the host_build
// option.
#include <algorithm>
#include <numeric>

#include "common.h"

namespace lkg {

static thread_local std::string g_err;

void set_error(const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_err = buf;
}

const char *get_error() { return g_err.c_str(); }

logoskg_status DevPool::alloc(void **out, size_t bytes, hipStream_t st, bool have_stream, bool *zeroed) {
    if (zeroed) *zeroed = false;
    const size_t asked = bytes;
    if (bytes == 0) bytes = 256;
    bytes = (bytes + 255) & ~size_t(255);
    auto it = free_.lower_bound(bytes);
    if (it != free_.end() && it->first <= bytes * 2) {
        Block b = it->second;
        live_[b.p] = Live{it->first, asked, b.zeros};
        free_.erase(it);
        if (b.after) {  // released behind work that may still run
            hipError_t e = hipSuccess;
            if (!have_stream) e = hipEventSynchronize(b.after->ev);
            else if (b.after->stream != st) e = hipStreamWaitEvent(st, b.after->ev, 0);
            if (e != hipSuccess) {
                set_error("waiting for a released block failed: %s", hipGetErrorString(e));
                return LOGOSKG_EDEVICE;
            }
        }
        if (zeroed) *zeroed = b.zeros >= asked;
        *out = b.p;
        return LOGOSKG_OK;
    }
    void *p = nullptr;
    if (!raw_alloc(&p, bytes)) {
        trim();  // give cached blocks back and retry once, then what else there is
        if (!raw_alloc(&p, bytes) && !(give_up_ && give_up_(give_up_ctx_) && raw_alloc(&p, bytes))) {
            set_error("device allocation of %zu bytes failed%s", bytes, alloc_fn_ ? " (caller's allocator)" : "");
            return LOGOSKG_ENOMEM;
        }
    }
    held_ += bytes;
    live_[p] = Live{bytes, asked, 0};
    *out = p;
    return LOGOSKG_OK;
}

bool DevPool::raw_alloc(void **p, size_t bytes) {
    if (alloc_fn_) {
        *p = alloc_fn_(bytes, ctx_);
        return *p != nullptr;
    }
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}

void DevPool::raw_free(void *p) {
    if (free_fn_) free_fn_(p, ctx_);
    else (void)hipFree(p);
}

void DevPool::release(void *p) {
    if (!p) return;
    auto it = live_.find(p);
    if (it == live_.end()) return;
    free_.emplace(it->second.size, Block{p, nullptr, 0});
    live_.erase(it);
}

// The blocks become reusable behind the work issued on `st` so far: one event for all of them
// (it goes back to the spare list when the last of these blocks has been handed out again).
void DevPool::release_after(void *const *ptrs, const bool *zeroed, int n, hipStream_t st) {
    hipEvent_t ev = nullptr;
    if (!spare_events_.empty()) {
        ev = spare_events_.back();
        spare_events_.pop_back();
    } else if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        ev = nullptr;
    }
    std::shared_ptr<After> after;
    if (ev && hipEventRecord(ev, st) == hipSuccess) {
        after = std::shared_ptr<After>(new After{ev, st}, [this](After *a) {
            spare_events_.push_back(a->ev);
            delete a;
        });
    } else {  // no event: wait here, then the blocks are free without conditions
        (void)hipGetLastError();
        (void)hipStreamSynchronize(st);
        if (ev) spare_events_.push_back(ev);
    }
    for (int i = 0; i < n; ++i) {
        if (!ptrs[i]) continue;
        auto it = live_.find(ptrs[i]);
        if (it == live_.end()) continue;
        const Live &l = it->second;  // (cleared: at least what was asked for; bytes behind it that were zero have stayed so)
        free_.emplace(l.size, Block{ptrs[i], after, zeroed && zeroed[i] ? std::max(l.asked, l.zeros) : 0});
        live_.erase(it);
    }
}

void DevPool::trim() {
    for (auto &kv : free_) {
        if (kv.second.after) (void)hipEventSynchronize(kv.second.after->ev);
        raw_free(kv.second.p);
        held_ -= kv.first;
    }
    free_.clear();
}

DevPool::~DevPool() {
    free_.clear();  // returns the events of pending releases to the spare list
    for (hipEvent_t e : spare_events_) (void)hipEventDestroy(e);
    spare_events_.clear();
}

const char *const kKernelNames[KK_NUM] = {
    "clear_planes", "seed_scatter", "frontier_census", "live_queries", "push_tail", "push_seg",
    "update_visited", "pull_tail", "pull_seg", "pull_finish", "count_tiles", "scan_counts",
    "lists", "pred", "pred_rows", "pred_mid_rows", "traversed", "paths", "shard_copy", "active_triples",
    "pred_walk"};

void Profiler::begin(int kind, hipStream_t st) {
    if (!on) return;
    hipEvent_t a = nullptr;
    if (!spare.empty()) { a = spare.back(); spare.pop_back(); }
    else if (hipEventCreate(&a) != hipSuccess) return;
    (void)hipEventRecord(a, st);
    cur_a = a;
    cur_kind = kind;
}

void Profiler::end(hipStream_t st) {
    if (!on || !cur_a) return;
    hipEvent_t b = nullptr;
    if (!spare.empty()) { b = spare.back(); spare.pop_back(); }
    else if (hipEventCreate(&b) != hipSuccess) { spare.push_back(cur_a); cur_a = nullptr; return; }
    (void)hipEventRecord(b, st);
    recs.push_back({cur_kind, cur_a, b});
    cur_a = nullptr;
}

void Profiler::drain() {
    for (auto &r : recs) {
        float ms = 0.f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            acc[r.kind].launches++;
            acc[r.kind].total_ms += ms;
            if (ms > acc[r.kind].max_ms) acc[r.kind].max_ms = ms;
        }
        spare.push_back(r.a);
        spare.push_back(r.b);
    }
    recs.clear();
}

void Profiler::release() {
    drain();
    for (hipEvent_t e : spare) (void)hipEventDestroy(e);
    spare.clear();
}

// The helper streams (two for the fetch's side work, one for shard copies, one for a plane that is
// made while those are part of a recorded sequence) are made once per
// device and shared by every graph on it; they live until the process ends.  Work of different
// graphs on one helper stream is only serialised: every dependency goes through events.
hipStream_t helper_stream(int device, int which) {
    static std::mutex mu;
    static std::map<int, std::array<hipStream_t, 4>> table;
    std::lock_guard<std::mutex> lock(mu);
    auto &row = table[device];  // value-initialised to null handles
    if (!row[which] && hipStreamCreateWithFlags(&row[which], hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        row[which] = nullptr;
    }
    return row[which];
}

template <typename T>
static logoskg_status upload(T **dst, const std::vector<T> &src, size_t *acct) {
    size_t bytes = std::max<size_t>(src.size(), 1) * sizeof(T);
    LKG_HIP(hipMalloc((void **)dst, bytes));
    if (!src.empty()) LKG_HIP(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
    *acct += bytes;
    return LOGOSKG_OK;
}

std::vector<uint32_t> segment_tables(const std::vector<ShortRow> &longer, uint32_t giant_min, RowClasses *rows) {
    std::vector<uint32_t> table(1, 0);
    auto count = [&](int64_t i, int segment) { return (longer[(size_t)i].end - longer[(size_t)i].begin + (uint32_t)segment - 1) / (uint32_t)segment; };
    rows->n_giant = 0;
    for (const ShortRow &r : longer) {
        if (r.end - r.begin < giant_min) break;
        table.push_back(table.back() + count(rows->n_giant++, kGiantSegment));
    }
    rows->n_giant_segs = table.back();
    rows->n_giant_places = rows->n_giant ? count(0, kGiantSegment) : 0;
    uint32_t first = 0;
    table.push_back(first);
    int64_t in = rows->n_giant;  // rows that reach a place
    for (int64_t place = 0; place < rows->n_giant_places; ++place) {
        while (count(in - 1, kGiantSegment) <= place) --in;
        table.push_back(first += (uint32_t)in);
    }
    rows->n_split = 0;
    rows->n_split_segs = 0;
    table.push_back(first = 0);
    for (int64_t i = 0; i < rows->n_hub; ++i) {
        const uint32_t n = count(i, kHubSegment);
        table.push_back(first += n);
        if (n > 1) {
            ++rows->n_split;
            rows->n_split_segs = first;  // (longest first: the split rows come before the others)
        }
    }
    rows->n_hub_segs = first;
    return table;
}

void set_segment_tables(RowClasses *rows, uint32_t *table) {
    rows->giant_seg_first = table;
    rows->giant_place_first = table + rows->n_giant + 1;
    rows->hub_seg_first = rows->giant_place_first + rows->n_giant_places + 1;
}

static void drop_pairs(logoskg_graph *g) {
    for (void *x : {g->pairs.block, g->pairs.rows.block, (void *)g->pairs.long_index})
        if (x) (void)hipFree(x);
    g->static_bytes -= g->pairs.bytes;
    g->pairs = PairRows();
}

size_t most_pair_bytes(const logoskg_graph *g) { return (size_t)g->T * 18 + (size_t)g->E * 24; }

bool give_up_pairs(logoskg_graph *g) {
    if (!g->pairs.off || g->pairs.recorded) return false;
    if (g->pairs.in_use) {
        g->pairs.wanted = true;
        return false;
    }
    if (hipDeviceSynchronize() != hipSuccess) {  // (kernels that read them may be queued on any stream)
        (void)hipGetLastError();
        return false;
    }
    drop_pairs(g);
    return true;
}

logoskg_status graph_alloc(logoskg_graph *g, void **p, size_t bytes) {
    if (hipMalloc(p, bytes) == hipSuccess) return LOGOSKG_OK;
    (void)hipGetLastError();
    if (give_up_pairs(g) && hipMalloc(p, bytes) == hipSuccess) return LOGOSKG_OK;
    (void)hipGetLastError();
    *p = nullptr;
    set_error("device allocation of %zu bytes failed", bytes);
    return LOGOSKG_ENOMEM;
}

// The rows of small graphs are counted and classified here: the device's way is a dozen launches and three waits.  us of a build
// with them on the device / here, by entities: 5,000: 738 / 598; 10,000: 909 / 816; 25,000: 1,237 / 1,252 and (hub-heavy)
// 1,577 / 1,491; 60,000: 1,026 / 1,127; 407,000: 7,614 / 11,019.
constexpr int32_t kHostRows = 1 << 14;

static logoskg_status read_offsets(const uint32_t *d_off, int32_t E, std::vector<uint32_t> *off) {
    off->resize((size_t)E + 1);
    LKG_HIP(hipMemcpy(off->data(), d_off, ((size_t)E + 1) * 4, hipMemcpyDeviceToHost));
    return LOGOSKG_OK;
}

// rows with an entry, of more than kTailMaxDegree, of at least hub_min
static logoskg_status count_rows(const logoskg_graph *g, const uint32_t *d_off, Scratch &tmp, unsigned int (&n)[3]) {
    if (g->E > kHostRows) return count_rows_on_device(d_off, g->E, g->hub_min, tmp, n);
    std::vector<uint32_t> off;
    LKG_TRY(read_offsets(d_off, g->E, &off));
    n[0] = n[1] = n[2] = 0;
    for (int32_t e = 0; e < g->E; ++e) {
        const uint32_t d = off[(size_t)e + 1] - off[e];
        n[0] += d > 0;
        n[1] += d > (uint32_t)kTailMaxDegree;
        n[2] += d >= (uint32_t)g->hub_min;
    }
    return LOGOSKG_OK;
}

// classify_on_device's lists, the short rows on the host as well
static logoskg_status classify_on_host(const logoskg_graph *g, const uint32_t *d_off, RowClasses *rc, std::vector<ShortRow> *tail, std::vector<ShortRow> *longer) {
    std::vector<uint32_t> off;
    LKG_TRY(read_offsets(d_off, g->E, &off));
    uint32_t at[kTailMaxDegree + 2] = {};  // of the rows of d entries at [kTailMaxDegree - d + 1], then where they begin
    rc->n_hub = 0;
    longer->clear();
    for (int32_t e = 0; e < g->E; ++e) {
        const uint32_t d = off[(size_t)e + 1] - off[e];
        if (d > (uint32_t)kTailMaxDegree) longer->push_back({e, off[e], off[(size_t)e + 1]});
        else if (d > 0) ++at[kTailMaxDegree - d + 1];
        rc->n_hub += d >= (uint32_t)g->hub_min;
    }
    for (int i = 1; i <= kTailMaxDegree; ++i) at[i] += at[i - 1];
    rc->n_tail = at[kTailMaxDegree];
    tail->resize((size_t)rc->n_tail);
    for (int32_t e = 0; e < g->E; ++e) {
        const uint32_t d = off[(size_t)e + 1] - off[e];
        if (d > 0 && d <= (uint32_t)kTailMaxDegree) (*tail)[at[kTailMaxDegree - d]++] = {e, off[e], off[(size_t)e + 1]};
    }
    return LOGOSKG_OK;
}

// Work lists over the rows of a CSR: short rows, segments of the longer ones (longest rows first; by_place:
// the first segments of all rows, then the second ones, ..), rows with several segments, giant and hub rows' segments.
static logoskg_status row_classes(logoskg_graph *g, const uint32_t *d_off, bool by_place, Scratch &tmp, RowClasses *rc) {
    std::vector<ShortRow> longer, tail;
    ShortRow *records = nullptr;
    bool on_host = g->E <= kHostRows;
    if (!on_host) {
        const logoskg_status s = classify_on_device(d_off, g->E, g->hub_min, tmp, rc, &records, &longer);
        if (s != LOGOSKG_OK && s != LOGOSKG_ENOMEM) return s;
        on_host = s == LOGOSKG_ENOMEM;  // no room for the device's temporaries
        if (on_host) (void)hipGetLastError();
    }
    if (on_host) LKG_TRY(classify_on_host(g, d_off, rc, &tail, &longer));
    std::stable_sort(longer.begin(), longer.end(), [](const ShortRow &a, const ShortRow &b) { return a.end - a.begin > b.end - b.begin; });
    std::vector<int32_t> rows, multi;
    std::vector<PullSegment> seg;
    rows.reserve(longer.size());
    for (const ShortRow &r : longer) {
        const uint32_t d = r.end - r.begin;
        rows.push_back(r.row);
        if (d > (uint32_t)kPullSegment) multi.push_back(r.row);
        for (uint32_t j = r.begin; j < r.end && (!by_place || j == r.begin); j += kPullSegment)
            seg.push_back({r.row, j, std::min(j + (uint32_t)kPullSegment, r.end), d > (uint32_t)kPullSegment ? 1u : 0u});
    }
    for (uint32_t place = kPullSegment; by_place && !longer.empty() && place < longer[0].end - longer[0].begin; place += kPullSegment)
        for (const ShortRow &r : longer) {
            if (r.end - r.begin <= place) break;
            seg.push_back({r.row, r.begin + place, std::min(r.begin + place + (uint32_t)kPullSegment, r.end), 1u});
        }
    const std::vector<uint32_t> table = segment_tables(longer, (uint32_t)std::max(kGiantRowMin, g->hub_min), rc);
    rc->n_seg = (int64_t)seg.size();
    rc->n_multi = (int64_t)multi.size();
    rc->n_long = (int64_t)longer.size();
    if (!longer.empty()) rc->longest = longer[0].end - longer[0].begin;
    // one block: what comes from the host in one copy, behind it the short rows
    std::vector<char> image;
    auto put = [&](const void *p, size_t bytes) {
        const size_t at = image.size();
        image.resize(at + (std::max<size_t>(bytes, 4) + 15) / 16 * 16);
        if (bytes) memcpy(image.data() + at, p, bytes);
        return at;
    };
    const size_t at_seg = put(seg.data(), seg.size() * sizeof(PullSegment)), at_table = put(table.data(), table.size() * 4),
                 at_multi = put(multi.data(), multi.size() * 4), at_rows = put(rows.data(), rows.size() * 4), at_tail = image.size();
    const size_t bytes = at_tail + (size_t)rc->n_tail * sizeof(ShortRow);
    if (on_host) put(tail.data(), tail.size() * sizeof(ShortRow));
    LKG_HIP(hipMalloc(&rc->block, std::max(bytes, image.size())));
    g->static_bytes += std::max(bytes, image.size());
    char *const base = static_cast<char *>(rc->block);
    rc->seg = reinterpret_cast<PullSegment *>(base + at_seg);
    set_segment_tables(rc, reinterpret_cast<uint32_t *>(base + at_table));
    rc->multi = reinterpret_cast<int32_t *>(base + at_multi);
    rc->longrows = reinterpret_cast<int32_t *>(base + at_rows);
    rc->tail = reinterpret_cast<ShortRow *>(base + at_tail);
    if (rc->n_tail && !on_host) LKG_HIP(hipMemcpyAsync(rc->tail, records, (size_t)rc->n_tail * sizeof(ShortRow), hipMemcpyDeviceToDevice, nullptr));
    LKG_HIP(hipMemcpy(base, image.data(), image.size(), hipMemcpyHostToDevice));
    return LOGOSKG_OK;
}

// The rows of distinct pairs with their work lists, where they are worth their room and there is some.
static logoskg_status pair_rows(logoskg_graph *g, const int32_t *in_sub, const uint16_t *in_rel, const int32_t *in_eid, Scratch &tmp) {
    constexpr size_t kNeverShort = (size_t)64 << 20;  // (a question to the runtime is 10 us)
    if (most_pair_bytes(g) > kNeverShort) {
        size_t free_bytes = 0, all_bytes = 0;
        if (hipMemGetInfo(&free_bytes, &all_bytes) != hipSuccess) (void)hipGetLastError();
        if (most_pair_bytes(g) > (free_bytes + scratch_bytes(&tmp)) / kPairRoom) return LOGOSKG_OK;
    }
    const size_t before = g->static_bytes;
    LKG_TRY(build_pairs_on_device(g, in_sub, in_rel, in_eid, tmp));
    const bool listed = !g->pairs.off || row_classes(g, g->pairs.off, true, tmp, &g->pairs.rows) == LOGOSKG_OK;
    g->pairs.bytes = g->static_bytes - before;
    if (!listed) {
        (void)hipGetLastError();  // (the graph works without them)
        drop_pairs(g);
    }
    return LOGOSKG_OK;
}

}  // namespace lkg

using namespace lkg;

extern "C" logoskg_status logoskg_build(const int32_t *subj, const int32_t *rel, const int32_t *obj,
                                        int64_t T, int32_t E, int32_t R,
                                        const logoskg_build_opts *opts, logoskg_graph **out) {
    if (!out) { set_error("out is NULL"); return LOGOSKG_EINVAL; }
    *out = nullptr;
    if (T < 0 || T >= (int64_t(1) << 31) || E <= 0 || R <= 0 || R > 65536) {
        set_error("sizes out of range: T=%lld E=%d R=%d", (long long)T, E, R);
        return LOGOSKG_EINVAL;
    }
    if (T > 0 && (!subj || !rel || !obj)) { set_error("triple arrays are NULL"); return LOGOSKG_EINVAL; }
    logoskg_build_opts o;
    memset(&o, 0, sizeof(o));
    if (opts) {
        if (opts->struct_size < 8 || opts->struct_size > sizeof(o)) {
            set_error("logoskg_build_opts.struct_size is %u", opts->struct_size);
            return LOGOSKG_EINVAL;
        }
        memcpy(&o, opts, opts->struct_size);
    }
    if (o.num_shards < 0 || o.num_shards > 127 || o.hub_min_degree < 0 || o.max_resident_shards < 0) {
        set_error("bad build options");
        return LOGOSKG_EINVAL;
    }
    if ((o.dev_alloc == nullptr) != (o.dev_free == nullptr)) {
        set_error("dev_alloc and dev_free must be given together");
        return LOGOSKG_EINVAL;
    }
    if (o.shard_dir && o.shard_dir[0] && o.num_shards <= 1) {
        set_error("shard_dir needs num_shards > 1");
        return LOGOSKG_EINVAL;
    }
    const bool device_build = o.num_shards <= 1 && !o.host_build;
    const bool device_sorts = !o.host_build;  // then the ids are checked on the device
    for (int64_t t = 0; !device_sorts && t < T; ++t) {
        if ((uint32_t)subj[t] >= (uint32_t)E || (uint32_t)obj[t] >= (uint32_t)E ||
            (uint32_t)rel[t] >= (uint32_t)R) {
            set_error("triple %lld = (%d, %d, %d) is out of range", (long long)t, subj[t], rel[t], obj[t]);
            return LOGOSKG_EINVAL;
        }
    }
    int ndev = 0;
    LKG_HIP(hipGetDeviceCount(&ndev));
    if (o.device < 0 || o.device >= ndev) { set_error("device %d not present", o.device); return LOGOSKG_EINVAL; }
    LKG_HIP(hipSetDevice(o.device));

    logoskg_graph *g = new (std::nothrow) logoskg_graph();
    if (!g) { set_error("out of host memory"); return LOGOSKG_ENOMEM; }
    g->device = o.device;
    g->E = E;
    g->R = R;
    g->T = T;
    g->Epad = ((int64_t)E + 63) / 64 * 64;
    g->hub_min = o.hub_min_degree > 0 ? std::max(o.hub_min_degree, kTailMaxDegree + 1) : kDefaultHubMin;
    g->num_shards = o.num_shards > 1 ? o.num_shards : 1;
    g->pool.set_spare([](void *x) { return give_up_pairs(static_cast<logoskg_graph *>(x)); }, g);
    if (o.dev_alloc) g->pool.set_allocator(o.dev_alloc, o.dev_free, o.alloc_ctx);

    logoskg_status st = LOGOSKG_OK;
    auto fail = [&](logoskg_status s) { logoskg_graph_free(g); return s; };
    try {
        std::unique_ptr<Scratch, void (*)(Scratch *)> scratch(nullptr, scratch_destroy);
        {
            Scratch *x = nullptr;
            if ((st = scratch_create(g, device_build, &x)) != LOGOSKG_OK) return fail(st);
            scratch.reset(x);
        }
        // work lists over the rows of OBJ (pull and predecessor kernels), and the rows of distinct pairs with theirs
        auto object_rows = [&]() -> logoskg_status {
            logoskg_status s = row_classes(g, g->in_off, false, *scratch, &g->in_rows);
            if (s == LOGOSKG_ENOMEM) {  // without the sorts' block, which is larger than what is left to do needs
                (void)hipGetLastError();
                scratch_release(scratch.get());
                s = row_classes(g, g->in_off, false, *scratch, &g->in_rows);
            }
            LKG_TRY(s);
            // (a build on the host takes no more of the device than its arrays; the sort of the pairs is 24 bytes per triple)
            return device_build ? pair_rows(g, g->in_sub, g->in_rel, g->in_eid, *scratch) : LOGOSKG_OK;
        };
        auto subject_row_counts = [&]() -> logoskg_status {
            unsigned int n[3];
            LKG_TRY(count_rows(g, g->out_off, *scratch, n));
            g->n_out_rows = n[0];
            g->n_out_hubs = n[2];
            return LOGOSKG_OK;
        };
        if (device_build) {
            if ((st = build_csr_on_device(g, subj, rel, obj, *scratch)) != LOGOSKG_OK) return fail(st);
            g->row_begin = g->out_off;
            if ((st = subject_row_counts()) != LOGOSKG_OK) return fail(st);
            if ((st = object_rows()) != LOGOSKG_OK) return fail(st);
        } else if (device_sorts) {
            // a sharded graph whose two sorts run on the device; the sorted arrays go to pinned host memory
            TripleSorter *sorter = nullptr;
            if ((st = sorter_create(g, subj, rel, obj, &sorter)) != LOGOSKG_OK) return fail(st);
            std::unique_ptr<TripleSorter, void (*)(TripleSorter *)> guard(sorter, sorter_destroy);
            std::vector<uint32_t> ooff;
            if ((st = sorter_offsets(sorter, false, &ooff)) != LOGOSKG_OK) return fail(st);
            if ((st = upload(&g->out_off, ooff, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
            if ((st = subject_row_counts()) != LOGOSKG_OK) return fail(st);
            if ((st = build_shards(g, subj, rel, obj, &o, ooff, sorter)) != LOGOSKG_OK) return fail(st);
            if (pairs_beside_shards(g, &o)) {  // (a cache of everything: its joined arrays are walked like a resident graph's)
                const int32_t *sub = nullptr, *eid = nullptr;
                const uint16_t *in_rel = nullptr;
                sorter_object_arrays(sorter, &sub, &in_rel, &eid);
                if ((st = pair_rows(g, sub, in_rel, eid, *scratch)) != LOGOSKG_OK) return fail(st);
            }
        } else {
        // out-degrees are needed by both the resident and the sharded form
        std::vector<uint32_t> ooff((size_t)E + 1, 0);
        for (int64_t t = 0; t < T; ++t) ooff[(size_t)subj[t] + 1]++;
        for (int32_t e = 0; e < E; ++e) ooff[(size_t)e + 1] += ooff[e];
        if ((st = upload(&g->out_off, ooff, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
        if ((st = subject_row_counts()) != LOGOSKG_OK) return fail(st);

        if (g->num_shards > 1) {
            if ((st = build_shards(g, subj, rel, obj, &o, ooff, nullptr)) != LOGOSKG_OK) return fail(st);
        } else {
            g->row_begin = g->out_off;
            {   // SUB: stable counting sort by subject
                std::vector<int32_t> oobj((size_t)T);
                std::vector<uint16_t> orel((size_t)T);
                std::vector<uint32_t> cur(ooff.begin(), ooff.end() - 1);
                for (int64_t t = 0; t < T; ++t) {
                    uint32_t p = cur[subj[t]]++;
                    oobj[p] = obj[t];
                    orel[p] = (uint16_t)rel[t];
                }
                if ((st = upload(&g->out_obj, oobj, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
                if ((st = upload(&g->out_rel, orel, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
            }
            {   // OBJ: stable counting sort by object, edge ids ascend inside a row
                std::vector<uint32_t> ioff((size_t)E + 1, 0);
                for (int64_t t = 0; t < T; ++t) ioff[(size_t)obj[t] + 1]++;
                for (int32_t e = 0; e < E; ++e) ioff[(size_t)e + 1] += ioff[e];
                std::vector<int32_t> isub((size_t)T), ieid((size_t)T);
                std::vector<uint16_t> irel((size_t)T);
                std::vector<uint32_t> cur(ioff.begin(), ioff.end() - 1);
                for (int64_t t = 0; t < T; ++t) {
                    uint32_t p = cur[obj[t]]++;
                    isub[p] = subj[t];
                    irel[p] = (uint16_t)rel[t];
                    ieid[p] = (int32_t)t;
                }
                if ((st = upload(&g->in_off, ioff, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
                if ((st = upload(&g->in_sub, isub, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
                if ((st = upload(&g->in_rel, irel, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
                if ((st = upload(&g->in_eid, ieid, &g->static_bytes)) != LOGOSKG_OK) return fail(st);
                if ((st = object_rows()) != LOGOSKG_OK) return fail(st);
            }
        }
        }
    } catch (const std::bad_alloc &) {
        set_error("out of host memory while sorting %lld triples", (long long)T);
        return fail(LOGOSKG_ENOMEM);
    }

    g->fr_seg_cap = (int64_t)E + T / kPushSegment + 64;  // every long row adds < deg/segment + 1 items
    constexpr size_t dev_ctr = C_TOTAL + kCensusWords * kCensusBlocks;
    const size_t ticket_bytes = (size_t)(g->Epad / (kTileEntities * kSuperTiles * kMegaSupers) + 2) * sizeof(unsigned int);
    auto rounded = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    const size_t of_ctr = rounded(dev_ctr * sizeof(unsigned long long) + ticket_bytes), of_tail = rounded((size_t)E * sizeof(int32_t)),
                 of_lists = of_ctr + of_tail + (size_t)g->fr_seg_cap * sizeof(RowSegment);
    char *lists = nullptr;
    if ((st = graph_alloc(g, (void **)&lists, of_lists)) != LOGOSKG_OK) return fail(st);
    g->static_bytes += of_lists;
    g->d_ctr = reinterpret_cast<unsigned long long *>(lists);
    g->fr_tail = reinterpret_cast<int32_t *>(lists + of_ctr);
    g->fr_seg = reinterpret_cast<RowSegment *>(lists + of_ctr + of_tail);
    g->count_tickets = reinterpret_cast<unsigned int *>(g->d_ctr + dev_ctr);
    if (hipMemset(g->count_tickets, 0, ticket_bytes) != hipSuccess || hipStreamSynchronize(nullptr) != hipSuccess) {
        set_error("hipMemset failed");
        return fail(LOGOSKG_EDEVICE);
    }
    constexpr size_t ctr_bytes = (C_TOTAL + 1 + 2 * kCensusSlot) * sizeof(unsigned long long), off_bytes = (LOGOSKG_MAX_QUERIES + 1) * sizeof(long long);
    static_assert(alignof(SmallReport) <= 8, "it lies behind 8-byte words");
    if (hipHostMalloc((void **)&g->h_ctr, ctr_bytes + off_bytes + sizeof(SmallReport), hipHostMallocDefault) != hipSuccess) {
        set_error("hipHostMalloc failed");
        return fail(LOGOSKG_ENOMEM);
    }
    g->h_census = g->h_ctr + C_TOTAL + 1;
    g->h_off = reinterpret_cast<long long *>(reinterpret_cast<char *>(g->h_ctr) + ctr_bytes);
    g->h_small = reinterpret_cast<SmallReport *>(reinterpret_cast<char *>(g->h_off) + off_bytes);
    for (int i = 0; i < 2; ++i) {
        if (!(g->side[i] = helper_stream(g->device, i)) ||
            hipEventCreateWithFlags(&g->ev_join[i], hipEventDisableTiming) != hipSuccess) {
            set_error("could not create the helper streams");
            return fail(LOGOSKG_EDEVICE);
        }
    }
    if (hipEventCreateWithFlags(&g->ev_fork, hipEventDisableTiming) != hipSuccess) {
        set_error("could not create events");
        return fail(LOGOSKG_EDEVICE);
    }
    *out = g;
    return LOGOSKG_OK;
}

extern "C" void logoskg_graph_free(logoskg_graph *g) {
    if (!g) return;
    (void)hipSetDevice(g->device);
    // nothing of this graph may still be queued when its events, streams and buffers go away
    // (a caller's stream can hold a wait on one of the events below)
    (void)hipDeviceSynchronize();
    free_shards(g);
    g->prof.release();
    for (int i = 0; i < 2; ++i) {
        if (g->side[i]) (void)hipStreamSynchronize(g->side[i]);
        if (g->ev_join[i]) (void)hipEventDestroy(g->ev_join[i]);
    }
    if (g->ev_fork) (void)hipEventDestroy(g->ev_fork);
    if (g->ev_rows) (void)hipEventDestroy(g->ev_rows);

    if (g->csr_block) {
        (void)hipFree(g->csr_block);
        g->out_off = g->in_off = nullptr;
        g->out_obj = g->out_eid = g->in_sub = g->in_eid = nullptr;
        g->out_rel = g->in_rel = nullptr;
    }
    void *ptrs[] = {g->out_off, g->out_obj, g->out_rel, g->in_off, g->in_sub, g->in_rel, g->in_eid,
                    g->in_rows.block, g->in_rows.block ? nullptr : (void *)g->in_rows.longrows,
                    g->d_ctr, g->long_index, g->row_pred, g->out_eid, g->plane_buf};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    drop_pairs(g);
    if (g->h_ctr) (void)hipHostFree(g->h_ctr);
    g->pool.trim();
    delete g;
}

extern "C" const char *logoskg_last_error(void) { return lkg::get_error(); }
extern "C" const char *logoskg_version(void) { return "logoskg-gfx950 0.1"; }

extern "C" logoskg_status logoskg_profile_enable(logoskg_graph *g, int32_t enable) {
    if (!g) { set_error("NULL graph"); return LOGOSKG_EINVAL; }
    g->prof.drain();
    g->prof.on = enable != 0;
    g->prof.counters = enable >= 2;
    return LOGOSKG_OK;
}

extern "C" logoskg_status logoskg_profile_read(logoskg_graph *g, logoskg_kernel_profile *out, int32_t capacity,
                                               int32_t *n_out) {
    if (!g || (capacity > 0 && !out)) { set_error("NULL argument"); return LOGOSKG_EINVAL; }
    (void)hipSetDevice(g->device);
    g->prof.drain();
    if (n_out) *n_out = KK_NUM;
    for (int i = 0; i < KK_NUM && i < capacity; ++i) {
        memset(&out[i], 0, sizeof(out[i]));
        strncpy(out[i].name, kKernelNames[i], sizeof(out[i].name) - 1);
        const Profiler::Acc &a = g->prof.acc[i];
        out[i].launches = a.launches;
        out[i].total_ms = a.total_ms;
        out[i].max_ms = a.max_ms;
        out[i].rows = a.units[0];
        out[i].edges = a.units[1];
        out[i].lines = a.units[2];
        out[i].items = a.units[3];
    }
    for (int i = 0; i < KK_NUM; ++i) g->prof.acc[i] = Profiler::Acc();
    return LOGOSKG_OK;
}
