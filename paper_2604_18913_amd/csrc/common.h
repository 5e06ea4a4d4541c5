// Internal declarations shared by the HIP translation units of liblogoskg.
// Nothing here is part of the public ABI (see include/logoskg.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <array>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <memory>
#include <string>
#include <unordered_map>
#include <vector>

#include "logoskg.h"

static_assert(sizeof(logoskg_build_opts) == 64 && sizeof(logoskg_graph_info) == 120,
              "the ctypes binding mirrors these layouts");

namespace lkg {

// ---------------------------------------------------------------- errors
void set_error(const char *fmt, ...);
const char *get_error();

#define LKG_HIP(call)                                                              \
    do {                                                                           \
        hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess) {                                                    \
            lkg::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),  \
                           __FILE__, __LINE__);                                    \
            return (e_ == hipErrorOutOfMemory) ? LOGOSKG_ENOMEM : LOGOSKG_EDEVICE; \
        }                                                                          \
    } while (0)

#define LKG_TRY(call)                         \
    do {                                      \
        logoskg_status s_ = (call);           \
        if (s_ != LOGOSKG_OK) return s_;      \
    } while (0)

// ---------------------------------------------------------------- device memory pool
// k-hop calls need several planes of hundreds of MB each; hipMalloc/hipFree of
// that size cost far more than the kernels, so freed blocks are kept and handed
// out again (exact-size match first, else the smallest block that is large
// enough and at most 2x the request).  A block released behind work that may
// still run (release_after) carries an event recorded on that work's stream: a
// later user on another stream waits for it, a user without a stream waits on
// the host.  Such a block can also be marked as cleared: the bytes that its user had asked for are zero (a block may be
// larger, and what lies behind them, also up to the next multiple of 256, is not), and only requests that
// these bytes hold are told so.
class DevPool {
public:
    logoskg_status alloc(void **out, size_t bytes) { return alloc(out, bytes, nullptr, false, nullptr); }
    logoskg_status alloc(void **out, size_t bytes, hipStream_t st, bool *zeroed = nullptr) {
        return alloc(out, bytes, st, true, zeroed);
    }
    void release(void *p);  // usable at once (the caller has waited for the block's last use)
    void release_after(void *const *ptrs, const bool *zeroed, int n, hipStream_t st);
    void trim();  // hipFree everything that is not handed out
    size_t bytes_held() const { return held_; }
    // the caller's allocator instead of hipMalloc / hipFree (set before the first alloc)
    void set_allocator(void *(*alloc_fn)(size_t, void *), void (*free_fn)(void *, void *), void *ctx) {
        alloc_fn_ = alloc_fn;
        free_fn_ = free_fn;
        ctx_ = ctx;
    }
    // what gives other memory back, true if there was any: asked when an allocation fails with nothing cached left
    void set_spare(bool (*give_up)(void *), void *ctx) {
        give_up_ = give_up;
        give_up_ctx_ = ctx;
    }
    ~DevPool();

private:
    struct After { hipEvent_t ev; hipStream_t stream; };
    struct Block { void *p; std::shared_ptr<After> after; size_t zeros; };  // zeros: so many bytes from its start are zero
    struct Live { size_t size, asked, zeros; };                             // of the block, of the request; zeros when handed out
    logoskg_status alloc(void **out, size_t bytes, hipStream_t st, bool have_stream, bool *zeroed);
    std::multimap<size_t, Block> free_;
    std::unordered_map<void *, Live> live_;
    std::vector<hipEvent_t> spare_events_;
    size_t held_ = 0;
    void *(*alloc_fn_)(size_t, void *) = nullptr;
    void (*free_fn_)(void *, void *) = nullptr;
    void *ctx_ = nullptr;
    bool (*give_up_)(void *) = nullptr;
    void *give_up_ctx_ = nullptr;
    bool raw_alloc(void **p, size_t bytes);
    void raw_free(void *p);
};

// ---------------------------------------------------------------- graph
constexpr int kLevelCounters = 5;
constexpr unsigned kCensusBlocks = 512;  // at most; kCensusWords each behind d_ctr's C_TOTAL
constexpr unsigned kCensusWords = 7;     // three sums, and up to four live words
constexpr int kTailMaxDegree = 32;      // rows up to this degree: one W-lane group per row
constexpr int kPullSegment = 1024;      // longer object rows are cut into segments of this many
                                        // entries, one wavefront each
constexpr int kPushSegment = 64;        // same for the subject rows of a push frontier
constexpr int kDefaultHubMin = 1024;    // object rows from this degree: block-per-row predecessor kernel
                                        // (shorter long rows: one wavefront per row)
constexpr int kDensePullPercent = 60;   // from this share of the triples leaving the frontier a hop is taken as dense
constexpr int kPredPushShare = 4;       // a level whose frontier holds at most T / this triples: long rows resolved from the subject side
constexpr int kGiantSegment = 8192;     // a giant row is walked by one 16-wave block per this many entries
constexpr int kGiantRowMin = 8192;      // hub rows from this size get a 16-wave block in the predecessor pass, smaller ones 4 waves
constexpr int kHubSegment = 2048;       // hub rows of narrow planes: a block of four wavefronts per this many entries
constexpr size_t kRowPredBytes = (size_t)8 << 30;  // most the row buffer of the predecessor pass may take
constexpr int kTileEntities = 64;       // entities per result tile (one wavefront of lanes)
constexpr int kSuperTiles = 16;         // tiles per super tile (1024 entities)
constexpr int kPredTiles = 4;           // tiles per block of the 16-word predecessor kernel
constexpr int kPredGroup = 4;           // lanes (= words) per entity in that kernel
constexpr int kMegaSupers = 64;         // super tiles per mega tile (65536 entities)

struct RowSegment {  // part [begin, min(begin + segment, row end)) of one CSR row
    int32_t row;
    uint32_t begin;
};

struct PullSegment {  // a segment [begin, end) of an object row; multi: the row has several segments
    int32_t row;
    uint32_t begin, end;
    uint32_t multi;
};

struct ShortRow {  // a CSR row with its bounds, so that a kernel needs no look-up in the offsets
    int32_t row;
    uint32_t begin, end;
};

// Small searches (small.hip): limits of what one block takes, and its report to the host.
constexpr int kSmallEdges = 2048;     // triples pushed per hop (and seeds)
constexpr int kSmallPairs = 1 << 15;  // (triple, query) pairs per hop
constexpr int kSmallEntities = 4096;  // reached entities (a power of two)
constexpr int kSmallHops = 16;
enum { kSmallDone = 0, kSmallGoOn = 1, kSmallBad = 2 };
struct SmallReport {
    int status, err, hops, n_all;
    int n_tail, n_seg;  // kSmallGoOn: rows of the frontier the general path goes on with
    int rows[kSmallHops + 1], reached[kSmallHops + 1];
    long long edges[kSmallHops + 1];
    long long off[65];
};

struct RowClasses {             // device work lists over the object rows, split by degree
    void *block = nullptr;      // holds all of them, or NULL (lists that are owned one by one)
    ShortRow *tail = nullptr;   // rows with 1 .. kTailMaxDegree entries, descending degree
    PullSegment *seg = nullptr;  // segments of the longer rows, longest rows first
    int32_t *multi = nullptr;   // rows cut into more than one segment
    int32_t *longrows = nullptr;  // rows with more than kTailMaxDegree entries, descending degree
                                  // (per streamed chunk when sharded); the first n_hub of them
                                  // have >= hub_min entries
    int64_t n_tail = 0, n_seg = 0, n_multi = 0, n_hub = 0, n_long = 0;
    uint32_t longest = 0;  // entries of the longest row if it has more than kTailMaxDegree (of a graph's in_rows)
    int64_t n_giant = 0;  // the first n_giant long rows have >= kGiantRowMin entries
    uint32_t *giant_seg_first = nullptr;  // [n_giant + 1] segments of kGiantSegment entries before every giant row
    int64_t n_giant_segs = 0;
    // (behind it) [n_giant_places + 1] the same segments by their place in the row, first ones first: before every place
    uint32_t *giant_place_first = nullptr;
    int64_t n_giant_places = 0;  // segments of the longest row
    uint32_t *hub_seg_first = nullptr;  // (behind it) [n_hub + 1] segments of kHubSegment entries before every hub row
    int64_t n_hub_segs = 0, n_split = 0, n_split_segs = 0;  // all; rows of several segments (the first ones), and theirs
};

// OBJ without its parallel triples: the rows' distinct subjects, for calls without whitelists, where a triple that repeats
// another's subject and object in a larger index adds nothing to a level and is never a predecessor.  Two orders of the
// same rows (off): `sub` / `eid` by triple index, for the predecessor pass; `pull_sub` by the in-degree of the subject,
// largest first (small graphs: by id), for pulled hops, which may take a row in any order and stop when nothing is missing:
// the subjects that most queries have reached come first.  Made by builds that sort on the device, where at most kPairShare
// percent of the triples are left and there is room (kPairRoom); off is NULL otherwise, also from when an allocation of the
// graph has found no memory but theirs (give_up_pairs).  (Distinct pairs of 30M triples of concepts 65 %, 3.4M 52 %, 300M
// hub-heavy ones 85 %.)  Worth 130 .. 330 us of a build of up to 0.8M triples (0.5 .. 2.5 ms), 2 ms of 7.5 with 3.4M: us of
// three hops with lists, 1 / 64 / 200 / 1,024 questions, without and with them:
//    80,000 triples   115 / 190 / 196 / 379    107 / 178 / 186 / 340       0.4M   115 / 201 / 178 / 416    114 / 202 / 183 / 373
//    0.2M             115 / 221 / 197 / 436    115 / 225 / 199 / 393       1.6M   135 / 227 / 243 / 506    133 / 211 / 228 / 497
//    0.2M hub-heavy   115 / 230 / 219 / 331    113 / 223 / 215 / 321       3.4M   161 / 287 / 358 / 694    157 / 266 / 323 / 693
// By the share that is left (1,024 questions, three hops with lists, without and with them; on 20M also under whitelists):
//    3.4M    92 %   870 /   888    88 %   864 /   885    80 %   852 /   860    65 %   831 /   822
//     20M    92 % 3,280 / 3,209    88 % 3,226 / 3,118    80 % 3,125 / 2,952    65 % 2,860 / 2,593    whitelists 80 % 2,230 / 2,200
constexpr int kPairShare = 90, kPairShareFew = 80;  // .. of graphs of fewer triples than kPairManyTriples
constexpr long long kPairManyTriples = 1 << 23;
constexpr int kPairRoom = 8;  // they take at most this part of the device memory that is free when they are made
struct PairRows {
    void *block = nullptr;  // holds the arrays
    size_t bytes = 0;       // of all that is held for them, counted in the graph's static_bytes
    uint32_t *off = nullptr;
    int32_t *pull_sub = nullptr, *sub = nullptr, *eid = nullptr;
    // every triple in pull_sub's order (rows as in_off has them), for pulled hops under whitelists: the first entries of all
    // rows are the same few subjects, and parallel triples ask for one line after the other
    int32_t *all_sub = nullptr;
    uint16_t *all_rel = nullptr;
    bool in_use = false;    // a call is about to launch what reads them
    bool wanted = false;    // .. and has done without memory that they hold: they go with the next search
    bool recorded = false;  // a recorded sequence reads them: they stay as long as the graph
    RowClasses rows;  // (segments by their place in the row: the first ones of all rows, the second ones, ..)
    int32_t *long_index = nullptr;  // as logoskg_graph::long_index
};

// ---------------------------------------------------------------- profiling
enum KernelKind {
    KK_CLEAR = 0, KK_SEED, KK_CENSUS, KK_LIVE, KK_PUSH_TAIL, KK_PUSH_SEG, KK_UPDATE, KK_PULL_TAIL,
    KK_PULL_SEG, KK_PULL_FINISH, KK_COUNT, KK_SCAN, KK_LISTS, KK_PRED, KK_PRED_HUB, KK_PRED_MID, KK_TRAVERSED,
    KK_PATHS, KK_SHARD_COPY, KK_TRIPLES, KK_PRED_WALK, KK_NUM
};
extern const char *const kKernelNames[KK_NUM];

// device counter slots (logoskg_graph::d_ctr); the statistics block holds four
// words per kernel class: rows, edges, lines, items
enum {
    C_NTAIL = 0, C_NSEG = 1, C_NROWS = 2, C_FEDGES = 3, C_NACTIVE = 4, C_ERR = 5,
    C_STATS = 8, C_TOTAL = C_STATS + 4 * KK_NUM  // the pinned host mirror holds one word more
};

// where a census of a narrow level leaves its counters in pinned memory: words C_NTAIL .. C_ERR, and one that says
// they are there
constexpr int kCensusDone = C_STATS, kCensusSlot = C_STATS + 8;

struct Profiler {
    bool on = false;        // bracket launches with events
    bool counters = false;  // also count rows / edges / lines inside the kernels
    struct Rec { int kind; hipEvent_t a, b; };
    struct Acc { int64_t launches = 0; double total_ms = 0, max_ms = 0; int64_t units[4] = {0, 0, 0, 0}; };
    std::vector<hipEvent_t> spare;
    std::vector<Rec> recs;
    Acc acc[KK_NUM];
    hipEvent_t cur_a = nullptr;
    int cur_kind = -1;
    void begin(int kind, hipStream_t st);
    void end(hipStream_t st);
    void drain();
    void release();
};

struct ProfScope {  // brackets the launches issued during its lifetime
    Profiler &p; hipStream_t st;
    ProfScope(Profiler &p_, int kind, hipStream_t st_) : p(p_), st(st_) { p.begin(kind, st); }
    ~ProfScope() { p.end(st); }
};

}  // namespace lkg

struct logoskg_graph {
    int device = 0;
    int32_t E = 0, R = 0;
    int64_t Epad = 0;  // E rounded up to a multiple of 64
    int64_t T = 0;
    int hub_min = lkg::kDefaultHubMin;
    int num_shards = 1;

    void *csr_block = nullptr;    // small resident graphs: holds the arrays of both CSRs
    // subject-sorted CSR (SUB): row s -> objects / relations of its triples
    uint32_t *out_off = nullptr;  // [E+1]
    uint32_t *row_begin = nullptr;    // [E] start of each subject's triples in the edge arrays
                                      // (== out_off when resident; shard-grouped order otherwise)
    uint8_t *shard_of_dev = nullptr;  // [Epad] device copy of the map P (255 = no shard)
    int32_t *out_obj = nullptr;   // [T]
    uint16_t *out_rel = nullptr;  // [T]
    // object-sorted CSR (OBJ): row v -> subjects / relations / edge ids of its triples
    uint32_t *in_off = nullptr;  // [E+1]
    int32_t *in_sub = nullptr;   // [T]
    uint16_t *in_rel = nullptr;  // [T]
    int32_t *in_eid = nullptr;   // [T]
    int32_t *out_eid = nullptr;  // [T] triple index of every entry of the subject-sorted CSR: what the
                                 // device build sorts by; else built on first use (ensure_out_eid)
    lkg::RowClasses in_rows;     // static row lists for the pull kernels
    lkg::PairRows pairs;         // the same rows without the parallel triples
    int64_t n_out_rows = 0, n_out_hubs = 0;

    // frontier work lists rebuilt every hop from the level's active bitmap (one block: d_ctr, fr_tail, fr_seg)
    int32_t *fr_tail = nullptr;          // [E] frontier rows of degree <= kTailMaxDegree
    lkg::RowSegment *fr_seg = nullptr;   // [fr_seg_cap] segments of the longer frontier rows
    int64_t fr_seg_cap = 0;
    unsigned long long *d_ctr = nullptr;  // device counters (see khop.hip)
    unsigned int *count_tickets = nullptr;  // (behind d_ctr) [mega tiles + 1] zero between two counts (result.hip)
    // pinned host memory, one block (three allocations: 0.44 ms for a graph of 50,000 triples, 0.41 with one):
    unsigned long long *h_ctr = nullptr;  // mirror of the counters
    long long *h_off = nullptr;           // [LOGOSKG_MAX_QUERIES + 1]: offsets of the last count
    unsigned long long *h_census = nullptr;  // [2][kCensusSlot]: counters of the levels of narrow_hops
    lkg::SmallReport *h_small = nullptr;  // written by k_small_search

    std::vector<int32_t> shard_of;  // host copy of the map P (empty when unsharded)
    std::vector<int64_t> shard_triples;
    void *shards = nullptr;  // lkg::ShardSet* when num_shards > 1

    // predecessor pass with 16-word planes: the kernels of the long object rows leave their
    // results in row_pred[row index][query] and the tile kernel moves them into the lists
    int32_t *long_index = nullptr;  // [E] position of a long row's entity in in_rows.longrows
    int32_t *row_pred = nullptr;    // [row_pred_rows][1024]
    int64_t row_pred_rows = 0;
    bool row_pred_tried = false;
    bool visited_asked = false;     // the last search's result was asked for its visited plane: the next one keeps it
    unsigned long long *plane_buf = nullptr;  // plane words of the bit-sliced predecessor pass (same first use)
    size_t plane_buf_bytes = 0;
    hipEvent_t ev_rows = nullptr;

    // the device's helper streams (default priority; shared by all graphs on the device) on which the
    // independent result kernels of a fetch can overlap (LOGOSKG_OVERLAP_FETCH=1)
    hipStream_t side[2] = {nullptr, nullptr};
    hipEvent_t ev_fork = nullptr, ev_join[2] = {nullptr, nullptr};

    lkg::DevPool pool;
    lkg::Profiler prof;
    size_t static_bytes = 0;
    size_t pinned_bytes = 0;
};

struct logoskg_result {
    logoskg_graph *g = nullptr;
    int Q = 0, k = 0, W = 0;
    int64_t Epad = 0;
    bool has_mask = false;
    bool has_counts = false;
    bool walk_exact = false;  // levels hold q^(h) of the plain iteration (no visited filter)
    unsigned long long *visited = nullptr;  // [Epad][W]; 16-word planes: the OR of the levels below vis_levels only
    // 16-word planes: hops do not keep visited unless keep_visited says so (they ask the levels, see Seen), fold_visited makes
    // it where it is read.  vis_dirty: the levels that may have left something in it (at least vis_levels).
    bool keep_visited = false;
    std::atomic<int> vis_levels{0}, vis_dirty{0};
    std::mutex vis_mutex;        // what makes visited behind the search: share_visited
    hipEvent_t vis_made = nullptr;  // visited is made behind the search, complete behind this (on whichever stream)
    int n_levels = 0;  // levels the search has got to; what lies behind is empty
    unsigned long long *levels = nullptr;   // [k+1][Epad][W]
    uint32_t *act = nullptr;      // [k+1][Epad/32]: entity has a non-zero line in that level
    unsigned long long *allow = nullptr;    // [R][W] relation -> queries that may follow it
    unsigned long long *live = nullptr;     // [k+1][16] queries whose level-h frontier has an out-edge, then
                                            // [k+1][kLevelCounters] counters of the levels (khop.hip)
    long long *seed_off = nullptr;  // [Q+1] and the batch's seeds behind it (k_seed's copy), for the path listing
    int32_t *seeds = nullptr;
    // result-list bookkeeping (count pass): for every query, the number of reached
    // entities below a tile, as three nested exclusive prefixes
    uint16_t *tile_base = nullptr;  // [ntiles][64W]  tiles (64 entities) inside their super tile
    uint32_t *super_base = nullptr; // [nsuper][64W]  super tiles (1024 entities) inside their mega tile
    uint32_t *mega_base = nullptr;  // [nmega][64W]   mega tiles (65536 entities)
    long long *d_reached_off = nullptr;  // [64W+1]
    // active entities (a bit in some level), ascending, and the place of each in that list; the
    // tiles of the count / list / predecessor kernels are cut from it (resident graphs)
    int32_t *tile_ent = nullptr;   // [Epad + 64], -1 behind the last id
    int32_t *cpos = nullptr;       // [Epad], defined for the listed entities
    uint32_t *act_chunk = nullptr; // per 2,048-entity chunk: listed entities in it (many chunks: before it); then *d_nact
    unsigned long long *d_nact = nullptr;
    long long n_active = -1;       // length of the list (known after the count pass)
    std::vector<int64_t> reached_off;  // host copy [Q+1]
    // a small search that ended in k_small_search: reached entities (ascending), offsets of the lists;
    // small_n < 0 for every other result
    long long *small_off = nullptr;
    int32_t *small_ent = nullptr;
    int small_n = -1, small_levels = 0;
    // the same bookkeeping for one level plane (logoskg_result_level_offsets)
    int level_counted = -1;
    uint16_t *lvl_tile_base = nullptr;
    uint32_t *lvl_super_base = nullptr, *lvl_mega_base = nullptr;
    long long *d_level_off = nullptr;
    std::vector<int64_t> level_off;
    // active triples of one hop for one query range (logoskg_result_triples_offsets)
    int trip_h = -1, trip_q0 = 0, trip_q1 = 0;
    int64_t trip_n = 0;            // entries of level trip_h - 1 over the range
    int64_t trip_total = 0;        // length of the concatenation of their rows of SUB
    int32_t *trip_ent = nullptr;   // [trip_n] those entities, query-major
    long long *trip_off = nullptr; // [trip_n + 1] where every entry's row starts in that concatenation
    long long *trip_chunk_entry = nullptr;  // [chunks + 1] entry behind the first position of every 256-position chunk
    long long *trip_chunk_first = nullptr;  // [chunks + 1] with a whitelist: allowed triples before the chunk
    std::vector<int64_t> trip_off_host;  // [trip_q1 - trip_q0 + 1]
    // chain-count tables of one (query, length) (logoskg_result_walks_count)
    int walk_q = -1, walk_d = -1;
    int64_t walk_total = 0;
    unsigned long long *walk_cnt = nullptr;   // [walk_d + 1][Epad] chains that end in the entity after h triples
    unsigned long long *walk_cum = nullptr;   // [walk_d][T] per hop: running sums inside the rows of OBJ
    unsigned long long *walk_pref = nullptr;  // [E + 1] chains that end in a smaller entity
    std::vector<logoskg_hop_stats> stats;
    mutable hipStream_t last_stream = nullptr;  // stream of the latest call that used the result
    bool complete = false;  // logoskg_khop ran to its end: every non-zero line of the planes has its bit in act
};

namespace lkg {

// device-side helpers -------------------------------------------------------
__device__ __forceinline__ int lane() { return (int)__lane_id(); }

// True when any lane of the caller's aligned W-lane group has `p` set.  Every
// lane of the group must be active at the call.
template <int W>
__device__ __forceinline__ bool group_any(bool p) {
    if constexpr (W == 1) {
        return p;
    } else {
        unsigned long long b = __ballot(p);
        int g0 = lane() & ~(W - 1);
        return ((b >> g0) & ((1ull << W) - 1ull)) != 0ull;
    }
}

__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }

__device__ __forceinline__ unsigned long long shfl64(unsigned long long v, int src) {
    int lo = __shfl((int)(unsigned)(v & 0xffffffffull), src);
    int hi = __shfl((int)(unsigned)(v >> 32), src);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

__device__ __forceinline__ unsigned long long shfl_xor64(unsigned long long v, int m) {
    int lo = __shfl_xor((int)(unsigned)(v & 0xffffffffull), m);
    int hi = __shfl_xor((int)(unsigned)(v >> 32), m);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

__device__ __forceinline__ unsigned long long shfl_up64(unsigned long long v, int d) {
    int lo = __shfl_up((int)(unsigned)(v & 0xffffffffull), d);
    int hi = __shfl_up((int)(unsigned)(v >> 32), d);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

// exclusive prefix sum over the lanes of a wavefront; `total` receives the sum
__device__ __forceinline__ int wave_excl_scan(int v, int &total) {
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int y = __shfl_up(x, d);
        if (lane() >= d) x += y;
    }
    total = __shfl(x, 63);
    return x - v;
}

__device__ __forceinline__ long long wave_sum(long long v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += (long long)shfl_xor64((unsigned long long)v, m);
    return v;
}

// 64x64 bit-matrix transpose across a wavefront: on entry lane r holds row r
// (bit c = M[r][c]); on return lane c holds column c (bit r = M[r][c]).  Six
// butterfly steps; in step j the off-diagonal j x j blocks of every 2j x 2j block
// change places.
__device__ __forceinline__ unsigned long long transpose64(unsigned long long x) {
    const unsigned long long lowmask[6] = {0x00000000FFFFFFFFull, 0x0000FFFF0000FFFFull, 0x00FF00FF00FF00FFull,
                                           0x0F0F0F0F0F0F0F0Full, 0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        const int j = 32 >> s;
        const unsigned long long m = lowmask[s];
        unsigned long long y = shfl_xor64(x, j);
        if (lane() & j) x = ((y >> j) & m) | (x & ~m);
        else x = (x & m) | ((y & m) << j);
    }
    return x;
}

// bits of word w (0..W-1) that belong to queries < Q
__device__ __forceinline__ unsigned long long query_bits(int Q, int w) {
    int lo = w * 64;
    if (Q >= lo + 64) return ~0ull;
    if (Q <= lo) return 0ull;
    return (1ull << (Q - lo)) - 1ull;
}

// Where a kernel on 16-word planes finds what the queries have reached so far: a line of `base` where the entity is active in
// one of the first `gate` levels (0: everywhere; base NULL: nowhere), and of the levels first .. last - 1 where it is
// active there.  Pulled hops that kept the visited plane read and wrote a line of it per object row, for rows that most
// hops reach once: four of the ten lines that such a row moved in a search of three hops with the counts and the clearing
// behind it.
struct Seen {
    const unsigned long long *base, *levels;
    const uint32_t *act;
    long long plane, actw;
    int gate, first, last;
    // more than half of the object rows are active in the last level: its lines (zero elsewhere) are read without asking (three
    // hops on hub-heavy 20M 1,482 -> 1,441 us, four 2,090 -> 2,029, 30M triples 839 -> 829, 3.4M the same)
    bool sure;
    bool keep;  // base is the plane that the hop keeps: it holds all levels, and its line is written where something is reached
};

__device__ __forceinline__ bool active_in(const Seen &s, int level, int e) {
    return (s.act[(size_t)level * s.actw + (e >> 5)] >> (e & 31)) & 1u;
}

constexpr int kSeenGate = 3;  // at most so many levels gate the base

__device__ __forceinline__ bool active_in_base(const Seen &s, int e) {
    bool on = s.gate == 0;
#pragma unroll
    for (int l = 0; l < kSeenGate; ++l) on |= l < s.gate && active_in(s, l, e);
    return on;
}

// A launch holds at most UINT32_MAX threads.  Items whose kernels take several lanes each go in ranges, launch(first, n), of
// per_block items to a block of 256 threads; nearly always there is one.
constexpr long long kMaxBlocks = (long long)UINT32_MAX / 256;

template <typename Launch>
inline void launch_ranges(long long n, long long per_block, Launch launch, long long max_blocks = kMaxBlocks) {
    for (long long first = 0, most = max_blocks * per_block; first < n; first += most) launch(first, n - first < most ? n - first : most);
}

inline int words_for_queries(int Q) { return Q <= 64 ? 1 : (Q <= 256 ? 4 : 16); }

// The segments of the lanes' subject rows (n of them from edge lo on; 0: none) to out[at ..].  Called by a whole wavefront, which
// writes the many segments of a hub row together: listed by one lane, those of 200,000 edges were 40 us.
__device__ __forceinline__ void write_segments(RowSegment *out, unsigned long long at, unsigned n, int32_t row, uint32_t lo) {
    constexpr unsigned kAlone = 4;
    if (n <= kAlone)
        for (unsigned x = 0; x < n; ++x) out[at + x] = RowSegment{row, lo + x * (uint32_t)kPushSegment};
    for (unsigned long long m = __ballot(n > kAlone); m; m &= m - 1) {
        const int from = __ffsll((long long)m) - 1;
        const unsigned long long to = shfl64(at, from);
        const unsigned all = (unsigned)__shfl((int)n, from);
        const int32_t r = __shfl(row, from);
        const uint32_t first = (uint32_t)__shfl((int)lo, from);
        for (unsigned x = (unsigned)lane(); x < all; x += 64) out[to + x] = RowSegment{r, first + x * (uint32_t)kPushSegment};
    }
}

// arguments of the list / predecessor kernels (result.hip)
struct FillArgs {
    int32_t E, R;
    int Q, k, q0, q1, hub_min;
    long long entries;  // of all lists asked for
    long long ntiles;
    const int32_t *tile_ent;  // the tiles' entities (list of active entities) or NULL: tile i = ids 64 i ..
    const int32_t *cpos;      // entity -> place in tile_ent (garbage for entities not in the list), or NULL
    long long n_listed;       // length of tile_ent's list
    unsigned long long *plane_buf;  // bit-sliced plane words between k_pred_walk and k_pred_emit, or NULL
    size_t plane_buf_bytes;
    int sparse;             // 16-word planes: mostly empty words (k_emit_sparse)
    int emit_eid_cap, emit_line_cap;  // most that k_pred_emit puts in LDS (edge ids / lines)
    uint32_t push_levels;   // bit h: level h of the long rows is resolved from the subject side (k_pred_push), the row
                            // kernels leave it out; host_graph / host_result are what the host code needs for that
    void *host_graph, *host_result;
    uint32_t dense_levels;  // bit h: nearly every triple leaves level h - 1, so the predecessor kernels gather the
                            // line of every entry of a row at level h without asking for its frontier bit first
    void *ev_rows;                    // host side: event between the block-per-row kernel and the list writer
    long long tile_begin, tile_count;  // tiles this predecessor launch covers
    long long plane;   // words per plane
    long long actw;    // uint32 words per active bitmap
    const unsigned long long *visited, *levels, *allow;
    // the level planes as the kernels of a page read them: `levels` itself, or the page's words of every line packed
    // (k_page_planes).  Word w of entity e in level h: plv[h * pplane + e * pstride + w - pfirst]
    const unsigned long long *plv;
    long long pplane;
    int pstride, pfirst;
    const uint32_t *act;
    const uint16_t *tile_base;
    const uint32_t *super_base, *mega_base;
    const long long *reached_off;
    const uint32_t *in_off;
    const int32_t *in_sub, *in_eid;
    const uint16_t *in_rel;
    const int32_t *rows;  // long object rows of this predecessor launch
    long long row_base;   // position of rows[0] in the graph's list of long rows
    const int32_t *long_index;  // entity -> position in that list (long rows only)
    int32_t *row_pred;    // [rows of the launch][1024] results of the row kernels, or NULL: they
                          // write the lists themselves
    int32_t *entity;
    uint8_t *hop;
    int32_t *pred;
    unsigned long long *stats_pred, *stats_hub, *stats_mid;  // rows / edges / lines counters or NULL
    int fuse_lists;  // the tile kernel also writes the entity and hop lists
    long long n_giant_rows;  // hub rows of the launch that get a 16-wave block per segment (the first ones)
    const uint32_t *giant_seg_first;  // [n_giant_rows + 1]
    long long n_giant_segs;
    const uint32_t *giant_place_first;  // [n_giant_places + 1], or NULL (rows that come range by range)
    long long n_giant_places;
    // the hub rows' segments for k_fetch_narrow (hub_seg_first NULL: rows that come range by range)
    const uint32_t *hub_seg_first;
    long long n_hub_rows, n_hub_segs, n_split_rows, n_split_segs;
    int32_t *seg_pred;  // [n_split_segs][64 W]
};

struct Scratch;  // a build's device temporaries (build_device.hip)
logoskg_status scratch_create(logoskg_graph *g, bool resident, Scratch **out);
void scratch_destroy(Scratch *s);
void scratch_release(Scratch *s);  // gives its memory back
size_t scratch_bytes(const Scratch *s);  // .. that it holds in one block
// build.hip: the rows of distinct pairs go, where nothing needs them any more that has been launched or recorded: true if so
bool give_up_pairs(logoskg_graph *g);
size_t most_pair_bytes(const logoskg_graph *g);  // of the arrays, the work lists and the index
// hipMalloc, with the memory of the distinct pairs where there is no other
logoskg_status graph_alloc(logoskg_graph *g, void **p, size_t bytes);
logoskg_status build_csr_on_device(logoskg_graph *g, const int32_t *subj, const int32_t *rel, const int32_t *obj, Scratch &tmp);
// rows of a CSR on the device: with an entry, of more than kTailMaxDegree, of at least hub_min
logoskg_status count_rows_on_device(const uint32_t *d_off, int32_t E, int hub_min, Scratch &tmp, unsigned int (&n)[3]);
logoskg_status classify_on_device(const uint32_t *d_off, int32_t E, int hub_min, Scratch &tmp, RowClasses *rc, ShortRow **records, std::vector<ShortRow> *longer);
// g->pairs' arrays (not its work lists) from the object-sorted ones; pairs.off stays NULL where they are not kept
// (of the object-sorted triples on the device, rows by g->in_off)
logoskg_status build_pairs_on_device(logoskg_graph *g, const int32_t *in_sub, const uint16_t *in_rel, const int32_t *in_eid, Scratch &tmp);
Seen seen_levels(const logoskg_result *r, int upto);
// khop.hip: visited becomes the OR of the levels below `upto` where it does not hold them yet (a captured launch leaves that open)
logoskg_status fold_visited(logoskg_result *r, int upto, hipStream_t st);
// the same for all levels behind the search, for a call on any stream and thread: work on st that follows finds the plane complete
logoskg_status share_visited(logoskg_result *r, hipStream_t st);
bool visited_by_search(const logoskg_result *r);  // .. and whether it is so without
bool captured(hipStream_t st);  // result.hip
struct TripleSorter;  // the triple list on the device during a sharded build (build_device.hip)
logoskg_status sorter_create(logoskg_graph *g, const int32_t *subj, const int32_t *rel, const int32_t *obj,
                             TripleSorter **out);
void sorter_destroy(TripleSorter *s);
logoskg_status sorter_offsets(TripleSorter *s, bool by_object, std::vector<uint32_t> *off);
logoskg_status sorter_subject_order(TripleSorter *s, const uint32_t *d_row_begin, int32_t *h_obj, uint16_t *h_rel);
logoskg_status sorter_object_order(TripleSorter *s, int32_t *h_sub, uint16_t *h_rel, int32_t *h_eid);
void sorter_object_arrays(const TripleSorter *s, const int32_t **sub, const uint16_t **rel, const int32_t **eid);  // behind it, on the device
bool pairs_beside_shards(const logoskg_graph *g, const logoskg_build_opts *opts);  // shards.hip: room for them by the caller's limits
logoskg_status ensure_out_eid(logoskg_graph *g, hipStream_t st);
// small.hip: *next_hop = the hop the general path goes on with (k + 1: none), the frontier's counters in g->h_ctr
logoskg_status small_search(logoskg_graph *g, logoskg_result *r, const logoskg_query_batch *b, bool want_counts,
                            bool force_push, int *next_hop, hipStream_t st);
logoskg_status small_fetch(logoskg_result *r, int q0, int q1, int32_t *entity, uint8_t *hop, int32_t *pred,
                           hipStream_t st);
// Tables of the segments that the predecessor pass cuts long rows (longest first) into, one behind the other, with their
// counts; where they lie on the device; into the arguments of a fetch
std::vector<uint32_t> segment_tables(const std::vector<ShortRow> &longer, uint32_t giant_min, RowClasses *rows);
void set_segment_tables(RowClasses *rows, uint32_t *table);
void set_row_segments(FillArgs *a, const RowClasses &rows);
void drop_walk_tables(logoskg_result *r);
void launch_lists(Profiler &prof, const FillArgs &a, int W, hipStream_t st);
void launch_pred(Profiler &prof, const FillArgs &a, int W, long long n_hub_rows, long long n_other_rows, bool mask,
                 hipStream_t st_tiles, hipStream_t st_rows);
logoskg_status sharded_pred(logoskg_graph *g, FillArgs *a, int W, bool mask, hipStream_t st);
long long max_chunk_rows(const logoskg_graph *g);
const RowClasses *joined_rows(const logoskg_graph *g);
// (prof_kind: the kernel class the launch is timed under)
logoskg_status census_lists(logoskg_graph *g, logoskg_result *r, int h, unsigned long long *ctr, hipStream_t st,
                            int prof_kind = KK_CENSUS);
void launch_push_lists(logoskg_graph *g, logoskg_result *r, int h, const unsigned long long *hc,
                       const int32_t *obj, const uint16_t *rel, bool update, const int32_t *list_tail,
                       const lkg::RowSegment *list_seg, const unsigned long long *ctr, hipStream_t st);
void shard_info(const logoskg_graph *g, logoskg_graph_info *o);
bool shard_out_arrays(const logoskg_graph *g, const int32_t **obj, const uint16_t **rel);
bool shard_in_arrays(const logoskg_graph *g, const int32_t **sub, const uint16_t **rel, const int32_t **eid);
void launch_pull_range(logoskg_graph *g, logoskg_result *r, int h, const RowClasses &rc, const int32_t *in_sub,
                       const uint16_t *in_rel, const unsigned long long *hc, bool want_stats, bool first,
                       hipStream_t st);
logoskg_status run_sharded_hop(logoskg_graph *g, logoskg_result *r, int h, bool pull, bool want_stats,
                               const unsigned long long *hc, hipStream_t st, logoskg_hop_stats *hs);
void free_shards(logoskg_graph *g);
// build.hip: per-device helper streams shared by all graphs (which = 0, 1: fetch side work; 2: shard copies)
hipStream_t helper_stream(int device, int which);
logoskg_status build_shards(logoskg_graph *g, const int32_t *subj, const int32_t *rel,
                            const int32_t *obj, const logoskg_build_opts *opts, const std::vector<uint32_t> &ooff,
                            TripleSorter *sorter);

}  // namespace lkg
