"""Kernels whose wavefronts hand data over in LDS, run on the CPU (wavefronts.h) with the wavefronts of a
block one after the other between two barriers, first to last and last to first: the results may not depend
on it."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_18913_amd", "csrc")


def text(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def between(src, first, last):
    at = src.index(first)
    return src[at:src.index(last, at)]


def definition(src, head):
    """From `head` (the start of a definition) to its closing brace."""
    at = src.index(head)
    i = src.index("{", at)
    depth = 0
    while True:
        depth += {"{": 1, "}": -1}.get(src[i], 0)
        i += 1
        if depth == 0:
            return src[at:i] + (";" if src[i] == ";" else "") + "\n"


def run(tmp_path, code):
    code = re.sub(r"asm volatile\([^;]*\);", "", code)
    cpp = tmp_path / "kernel.cpp"
    cpp.write_text('#include "wavefronts.h"\n' + code)
    exe = tmp_path / "kernel"
    p = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-I", HERE, "-o", str(exe), str(cpp)],
                       capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr[-4000:]
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr


def device_helpers():
    common = text("common.h")
    return between(common, "__device__ __forceinline__ int lane()", "inline int words_for_queries")


LISTS_MAIN = """
template <int W, int NB, int TILES> int check(const std::vector<int> &waves, bool listed) {
    constexpr int Qp = 64 * W;
    const int E = 2500, k = 3, Q = W == 1 ? 50 : 230, Epad = (E + 63) / 64 * 64;
    unsigned long long rng = 7 + W;
    auto next = [&]() { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33); };
    std::vector<unsigned long long> levels((size_t)(k + 1) * Epad * W), visited((size_t)Epad * W);
    std::vector<int> ent;
    for (int e = 0; e < E; ++e) {
        if (listed && next() % 3 == 0) continue;
        ent.push_back(e);
        for (int q = 0; q < Q; ++q)
            if (next() % 4 == 0) {
                levels[((size_t)(next() % (k + 1)) * Epad + e) * W + q / 64] |= 1ull << (q & 63);
                visited[(size_t)e * W + q / 64] |= 1ull << (q & 63);
            }
    }
    const int n = (int)ent.size(), tiles = (n + 63) / 64, supers = (tiles + 15) / 16;
    ent.resize(n + 64, -1);
    std::vector<uint16_t> tile_base((size_t)tiles * Qp);
    std::vector<uint32_t> super_base((size_t)supers * Qp), mega_base(Qp);
    std::vector<long long> off(Qp + 1);
    std::vector<int> want_ent, want_hop;
    for (int q = 0; q < Qp; ++q) {
        off[q] = (long long)want_ent.size();
        for (int i = 0; i < n; ++i) {
            const long long before = (long long)want_ent.size() - off[q];
            if (i % 1024 == 0) super_base[(size_t)(i / 1024) * Qp + q] = (uint32_t)before;
            if (i % 64 == 0) tile_base[(size_t)(i / 64) * Qp + q] = (uint16_t)(before - super_base[(size_t)(i / 1024) * Qp + q]);
            if (!((visited[(size_t)ent[i] * W + q / 64] >> (q & 63)) & 1)) continue;
            int h = 0;
            while (!((levels[((size_t)h * Epad + ent[i]) * W + q / 64] >> (q & 63)) & 1)) ++h;
            want_ent.push_back(ent[i]);
            want_hop.push_back(h);
        }
    }
    off[Qp] = (long long)want_ent.size();
    std::vector<int32_t> entity(want_ent.size(), -7);
    std::vector<uint8_t> hop(want_ent.size(), 99);
    FillArgs a;
    memset((void *)&a, 0, sizeof(a));
    a.E = E; a.Q = Q; a.k = k; a.q0 = 0; a.q1 = Q;
    a.ntiles = tiles; a.tile_ent = listed ? ent.data() : nullptr;
    a.plane = (long long)Epad * W; a.visited = visited.data(); a.levels = levels.data();
    a.tile_base = tile_base.data(); a.super_base = super_base.data(); a.mega_base = mega_base.data();
    a.reached_off = off.data(); a.entity = entity.data(); a.hop = hop.data();
    run_grid((unsigned)((tiles + TILES - 1) / TILES), 64 * W, waves, [&] { k_lists<W, NB, TILES>(a); });
    int bad = 0;
    for (size_t i = 0; i < want_ent.size(); ++i) bad += entity[i] != want_ent[i] || (NB && hop[i] != want_hop[i]);
    printf("%d words, %d hop bits, %d tiles, list %d: %d of %zu entries wrong\\n", W, NB, TILES, listed, bad, want_ent.size());
    return bad;
}

int main() {
    int bad = 0;
    for (bool listed : {false, true}) {
        bad += check<1, 0, 4>({0}, listed) + check<1, 2, 1>({0}, listed);
        for (const std::vector<int> &waves : {std::vector<int>{0, 1, 2, 3}, std::vector<int>{3, 2, 1, 0}})
            bad += check<4, 0, 16>(waves, listed) + check<4, 2, 16>(waves, listed) + check<4, 2, 4>(waves, listed) +
                   check<4, 0, 1>(waves, listed);
    }
    return bad != 0;
}
"""


def test_lists_of_narrow_planes(tmp_path):
    common, result = text("common.h"), text("result.hip")
    run(tmp_path, "\n".join([
        between(common, "constexpr int kTileEntities", "struct RowSegment"),
        device_helpers(),
        definition(common, "struct FillArgs {"),
        definition(result, "__device__ __forceinline__ long long tile_entity("),
        "template <int W>\n" + definition(result, "__device__ __forceinline__ unsigned long long stage_word("),
        definition(result, "__device__ __forceinline__ unsigned long long range_bits("),
        definition(result, "__device__ __forceinline__ long long super_start("),
        "template <int W, int NB, int TILES>\n" + definition(result, "__global__ void __launch_bounds__(64 * W) k_lists("),
        LISTS_MAIN]))


SMALL_MAIN = """
// n_seeds seeds with `fan` triples each into objects of their own: the search takes one hop
static int check(const std::vector<int> &waves, int n_seeds, int fan, bool whole) {
    const int edges = n_seeds * fan, E = n_seeds + edges;
    std::vector<uint32_t> off(E + 1, edges);
    std::vector<int32_t> obj(edges), seeds(n_seeds), kept(n_seeds), ent(kSmallEntities, -1);
    std::vector<uint16_t> rel(edges);
    for (int i = 0; i < n_seeds; ++i) {
        seeds[i] = i;
        off[i] = (uint32_t)(i * fan);
    }
    for (int j = 0; j < edges; ++j) obj[j] = E - 1 - j;
    const int actw = (E + 63) / 64 * 2;
    std::vector<unsigned long long> visited(E + 64), levels(2 * (size_t)(E + 64));
    std::vector<uint32_t> act(2 * actw);
    long long seed_off[2] = {0, n_seeds}, kept_off[2], list_off[65];
    SmallReport rep;
    memset((void *)&rep, 0xee, sizeof(rep));
    SmallArgs a;
    memset((void *)&a, 0, sizeof(a));
    a.Q = 1; a.hops = 1; a.want_counts = 1; a.force_push = 1;
    a.E = E; a.T = edges; a.num_seeds = n_seeds; a.plane = E + 64; a.actw = actw;
    a.seed_off = seed_off; a.seeds = seeds.data(); a.out_off = off.data(); a.out_obj = obj.data(); a.out_rel = rel.data();
    a.visited = visited.data(); a.levels = levels.data(); a.act = act.data();
    a.kept_off = kept_off; a.kept_seeds = kept.data(); a.ent = ent.data(); a.off = list_off; a.rep = &rep;
    run_grid(1, kSmallThreads, waves, [&] { k_small_search(a); });
    int bad = 0;
    if (whole) {
        bad = rep.status != kSmallDone || rep.hops != 1 || rep.n_all != E || rep.off[64] != E || rep.reached[1] != edges;
        for (int e = 0; e < E; ++e)
            bad += ent[e] != e || visited[e] != 1 || levels[e] != (e < n_seeds) || levels[(size_t)a.plane + e] != (e >= n_seeds);
    } else {  // handed over before the hop, nothing of which may have been taken
        bad = rep.status != kSmallGoOn || rep.hops != 0 || rep.n_all != n_seeds || rep.edges[0] != edges || rep.rows[0] != n_seeds;
        for (int e = 0; e < E; ++e) bad += visited[e] != (e < n_seeds) || levels[(size_t)a.plane + e] != 0;
    }
    printf("%d seeds, %d triples: status %d, %d entities, %d wrong\\n", n_seeds, edges, rep.status, rep.n_all, bad);
    return bad;
}

int main() {
    std::vector<int> forward(kSmallThreads / 64), backward;
    std::iota(forward.begin(), forward.end(), 0);
    backward.assign(forward.rbegin(), forward.rend());
    int bad = 0;
    for (const auto &waves : {forward, backward})
        bad += check(waves, 2048, 1, true) + check(waves, 683, 3, false) + check(waves, 682, 3, true) + check(waves, 1, 2048, true);
    return bad != 0;
}
"""


def test_a_small_search_at_the_limit_of_its_list(tmp_path):
    # 2,048 seeds and 2,048 triples: the hop fills the list of 4,096 reached entities exactly
    common, small = text("common.h"), text("small.hip")
    run(tmp_path, "\n".join([
        between(common, "constexpr int kTailMaxDegree", "struct RowSegment"),
        between(common, "constexpr int kSmallEdges", "struct RowClasses"),
        device_helpers(),
        between(small, "constexpr int kSmallThreads", "// One block per fetched query"),
        SMALL_MAIN]))


PATHS_MAIN = """
struct Graph {
    int E, k, R;
    std::vector<uint32_t> in_off, out_off;
    std::vector<int32_t> in_sub, in_eid, out_obj, out_eid, seeds;
    std::vector<uint16_t> in_rel, out_rel;
    std::vector<std::vector<int>> level;  // [k + 1][E] of the one query
    std::vector<bool> keep;
    // every shortest path, ordered by the triples read from the target
    void search(int v, int h, std::vector<int> &path, std::vector<std::vector<int>> &all, size_t most) const {
        if (all.size() >= most) return;
        if (h == 0) {
            all.push_back(std::vector<int>(path.rbegin(), path.rend()));
            return;
        }
        for (uint32_t j = in_off[v]; j < in_off[v + 1]; ++j)
            if (keep[in_rel[j]] && level[h - 1][in_sub[j]]) {
                path.push_back(in_eid[j]);
                search(in_sub[j], h - 1, path, all, most);
                path.pop_back();
            }
    }
};

// k > 8: a band of entities, and the levels of the walks of exactly h triples
static Graph make(unsigned seed, bool masked, int k) {
    unsigned long long rng = seed;
    auto next = [&]() { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33); };
    Graph g;
    g.E = 900;
    g.k = k;
    g.R = 5;
    std::vector<std::array<int, 3>> t;
    const int rows[] = {1, 127, 128, 129, 130, 300, 1025, 2500};  // objects 0 .. 7, and short rows behind them
    for (int o = 0; o < g.E; ++o)
        for (int i = o < 8 ? rows[o] : (int)(next() % 6); i > 0; --i)
            t.push_back({(int)(k > 8 && o >= 8 ? (o + g.E - 1 - next() % 3) % g.E : next() % g.E), (int)(next() % g.R), o});
    for (size_t i = t.size(); i > 1; --i) std::swap(t[i - 1], t[next() % i]);
    const size_t T = t.size();
    auto csr = [&](int key, std::vector<uint32_t> &off, std::vector<int32_t> &other, std::vector<uint16_t> &rel, std::vector<int32_t> &eid) {
        off.assign(g.E + 1, 0);
        other.resize(T); rel.resize(T); eid.resize(T);
        for (auto &x : t) off[x[key] + 1]++;
        for (int e = 0; e < g.E; ++e) off[e + 1] += off[e];
        auto cur = off;
        for (size_t i = 0; i < T; ++i) {
            const uint32_t p = cur[t[i][key]]++;
            other[p] = t[i][2 - key]; rel[p] = (uint16_t)t[i][1]; eid[p] = (int32_t)i;
        }
    };
    csr(2, g.in_off, g.in_sub, g.in_rel, g.in_eid);
    csr(0, g.out_off, g.out_obj, g.out_rel, g.out_eid);
    for (int r = 0; r < g.R; ++r) g.keep.push_back(!masked || r % 2 == 0);
    g.seeds = {(int)(next() % g.E), 9, 9, 700};
    g.level.assign(g.k + 1, std::vector<int>(g.E));
    std::vector<int> seen(g.E);
    for (int s : g.seeds) g.level[0][s] = seen[s] = 1;
    for (int h = 1; h <= g.k; ++h) {
        for (auto &x : t)
            if (g.level[h - 1][x[0]] && g.keep[x[1]] && (k > 8 || !seen[x[2]])) g.level[h][x[2]] = 1;
        for (int e = 0; e < g.E; ++e) seen[e] |= g.level[h][e];
    }
    return g;
}

template <int NW> int check(unsigned seed, bool masked, bool seeds_side, int max_paths, const std::vector<int> &waves, int k = 5) {
    const Graph g = make(seed, masked, k);
    const int q = 3, Epad = (g.E + 63) / 64 * 64, actw = Epad / 32;
    std::vector<unsigned long long> levels((size_t)(g.k + 1) * Epad), allow(g.R);
    std::vector<uint32_t> act((size_t)(g.k + 1) * actw);
    for (int h = 0; h <= g.k; ++h)
        for (int e = 0; e < g.E; ++e)
            if (g.level[h][e]) {
                levels[(size_t)h * Epad + e] = 1ull << q;
                act[(size_t)h * actw + e / 32] |= 1u << (e % 32);
            }
    for (int r = 0; r < g.R; ++r) allow[r] = g.keep[r] ? 1ull << q : 0;
    const long long n = (long long)g.seeds.size(), seed_off[] = {0, 0, 0, 0, n};
    std::vector<int32_t> query, target, length;
    for (int e = 0; e < g.E; e += e < 12 ? 1 : 19) {
        query.push_back(q);
        target.push_back(e);
        length.push_back(e % (g.k + 1));
    }
    const int pairs = (int)target.size();
    std::vector<int32_t> count(pairs, -7), edges((size_t)pairs * max_paths * g.k, -7);
    PathArgs a;
    memset((void *)&a, 0, sizeof(a));
    a.Q = 4; a.k = g.k; a.W = 1; a.E = g.E; a.R = g.R; a.plane = Epad; a.actw = actw;
    a.levels = levels.data(); a.act = act.data(); a.allow = masked ? allow.data() : nullptr;
    a.in_off = g.in_off.data(); a.in_sub = g.in_sub.data(); a.in_rel = g.in_rel.data(); a.in_eid = g.in_eid.data();
    a.seed_off = seed_off; a.seeds = g.seeds.data(); a.out_off = g.out_off.data(); a.out_obj = g.out_obj.data();
    a.out_rel = g.out_rel.data(); a.out_eid = seeds_side ? g.out_eid.data() : nullptr;
    a.query_idx = query.data(); a.target = target.data(); a.length = k > 8 ? length.data() : nullptr; a.max_paths = max_paths;
    a.path_count = count.data(); a.path_edges = edges.data();
    run_grid(pairs, 64 * NW, waves, [&] { k_paths<NW>(a); });
    int bad = 0, total = 0, longest = 0;
    for (int i = 0; i < pairs; ++i) {
        int d = 0;
        if (k > 8) d = g.level[length[i]][target[i]] ? length[i] : g.k + 1;
        else while (d <= g.k && !g.level[d][target[i]]) ++d;
        std::vector<std::vector<int>> all;
        std::vector<int> path;
        if (d <= g.k) g.search(target[i], d, path, all, max_paths);
        bad += count[i] != (int)all.size();
        total += (int)all.size();
        if (!all.empty()) longest = std::max(longest, d);
        for (int p = 0; p < max_paths; ++p)
            for (int x = 0; x < g.k; ++x) {
                const int want = p < (int)all.size() && x < (int)all[p].size() ? all[p][x] : -1;
                bad += edges[((size_t)i * max_paths + p) * g.k + x] != want;
            }
    }
    printf("%d wavefronts, masked %d, seeds' side %d, %d paths: %d found, of up to %d triples, %d wrong\\n", NW, masked, seeds_side, max_paths, total, longest, bad);
    return bad;
}

int main() {
    int bad = 0;
    for (bool masked : {false, true})
        for (bool seeds_side : {false, true})
            for (int most : {16, 2}) {
                bad += check<1>(5, masked, seeds_side, most, {0}) + check<4>(6, masked, seeds_side, most, {1, 2, 0, 3}, 40);
                for (const std::vector<int> &waves : {std::vector<int>{0, 1, 2, 3}, std::vector<int>{3, 2, 1, 0}, std::vector<int>{2, 0, 3, 1}})
                    bad += check<4>(5 + most, masked, seeds_side, most, waves);
            }
    return bad != 0;
}
"""


def test_path_listing_between_one_wavefront_and_the_block(tmp_path):
    # rows around the length up to which one wavefront goes on alone, and long ones on all levels
    common, paths = text("common.h"), text("paths.hip")
    run(tmp_path, "\n".join([
        "#include <array>\n#define LOGOSKG_MAX_K 254",
        device_helpers(),
        between(paths, "struct PathArgs {", "// NW wavefronts (one block)"),
        "template <int NW>\n" + definition(paths, "__global__ void __launch_bounds__(64 * NW) k_paths("),
        PATHS_MAIN]))


WALKS_MAIN = """
int main() {
    int bad = 0;
    for (unsigned share : {100u, 60u, 5u})  // of the entities that are in the level
        for (const std::vector<int> &waves : {std::vector<int>{0, 1, 2, 3}, std::vector<int>{3, 2, 1, 0}, std::vector<int>{1, 3, 0, 2}}) {
            unsigned long long rng = share;
            auto next = [&]() { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33); };
            // giant rows of two and three segments, then longer ones by descending degree, then short ones
            std::vector<int> degree = {2 * kGiantSegment + 5, kGiantSegment + 1};
            for (int i = 0; i < 41; ++i) degree.push_back(1600 - 39 * i);
            for (int i = 0; i < 300; ++i) degree.push_back((int)(next() % 33));
            const int E = (int)degree.size(), n_giant = 2, n_long = 41;
            std::vector<int32_t> place(E), rows;
            std::iota(place.begin(), place.end(), 0);
            for (int i = E; i > 1; --i) std::swap(place[i - 1], place[next() % i]);
            std::vector<uint32_t> off(E + 1);
            for (int i = 0; i < E; ++i) off[place[i] + 1] = degree[i];
            for (int e = 0; e < E; ++e) off[e + 1] += off[e];
            for (int i = 0; i < n_giant + n_long; ++i) rows.push_back(place[i]);
            const uint32_t T = off[E];
            std::vector<int32_t> sub(T);
            std::vector<uint16_t> rel(T);
            std::vector<unsigned long long> prev(E), level(2 * E), allow(4), cum(T, 77), cnt(E), totals(5, 77);
            for (auto &s : sub) s = (int32_t)(next() % E);
            for (auto &r : rel) r = (uint16_t)(next() % 4);
            for (auto &c : prev) c = next() % 1000;
            for (int e = 0; e < E; ++e) level[E + e] = next() % 100 < share ? 4 : 3;
            allow = {4, 0, 7, 4};
            std::vector<uint32_t> first = {0, 3, 5};
            const unsigned long_blocks = share == 60 ? 5 : share == 5 ? n_long : 30;  // rows per block: 9, 1, 2
            unsigned overflow = 0;
            run_grid(5 + long_blocks + (E + 255) / 256, 256, waves, [&] {
                k_walk_count<true>(rows.data(), first.data(), n_giant, 5, n_long, long_blocks, E, 1, 0, 4ull, level.data() + E,
                                   allow.data(), off.data(), sub.data(), rel.data(), prev.data(), cnt.data(), cum.data(),
                                   totals.data(), &overflow);
            });
            run_grid(5, 256, waves, [&] {
                k_walk_join_giant(rows.data(), first.data(), n_giant, 1, 0, 4ull, level.data(), E, 1, off.data(), totals.data(), T,
                                  cum.data(), &overflow);
            });
            int wrong = overflow != 0;
            for (int e = 0; e < E; ++e) {
                unsigned long long sum = 0;
                const bool in = level[E + e] & 4;
                for (uint32_t j = off[e]; j < off[e + 1]; ++j) {
                    wrong += cum[j] != (in ? sum : 77);
                    if (rel[j] != 1) sum += prev[sub[j]];
                }
                wrong += cnt[e] != (in ? sum : 0);
            }
            printf("%u %% in the level: %d wrong\\n", share, wrong);
            bad += wrong;
        }
    return bad != 0;
}
"""


def test_chain_counts_of_every_class_of_rows(tmp_path):
    common, walks = text("common.h"), text("walks.hip")
    run(tmp_path, "\n".join([
        between(common, "constexpr int kTailMaxDegree", "struct RowSegment"),
        device_helpers(),
        between(walks, "constexpr unsigned long long kWalkCountLimit", "// pref[0] = 0 and the running sum over"),
        WALKS_MAIN]))
