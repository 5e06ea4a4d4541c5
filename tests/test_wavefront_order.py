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
        bad += check<1, 0, 4>({0}, listed) + check<1, 2, 4>({0}, listed);
        for (const std::vector<int> &waves : {std::vector<int>{0, 1, 2, 3}, std::vector<int>{3, 2, 1, 0}})
            bad += check<4, 0, 16>(waves, listed) + check<4, 2, 16>(waves, listed) + check<4, 2, 4>(waves, listed);
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
