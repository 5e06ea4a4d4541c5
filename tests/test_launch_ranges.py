"""Short rows go to launches of fewer than 2^32 threads.  On the CPU: the ranges themselves, and the push kernel (its text run
by wavefronts.h) over ranges of a frontier list.  On the GPU: a pulled hop over more short rows than one launch takes."""
import numpy as np
import pytest

from helpers import progress
from test_wavefront_order import between, definition, device_helpers, run, text


def ranges():
    common = text("common.h")
    return between(common, "constexpr long long kMaxBlocks", "inline int words_for_queries")


def test_ranges_cover_all_rows_and_fit_a_launch(tmp_path):
    run(tmp_path, ranges() + """
int main() {
    int bad = 0;
    for (int lanes : {1, 4, 8, 16}) {
        const long long per_block = 256 / lanes, most = kMaxBlocks * per_block;
        for (long long n : {0ll, 1ll, per_block, most - 1, most, most + 1, (1ll << 29) - 1, 1ll << 29, (1ll << 31) - 1, 2 * most + 5}) {
            long long next = 0;
            launch_ranges(n, per_block, [&](long long first, long long m) {
                bad += first != next || m < 1 || (m + per_block - 1) / per_block * 256 > (long long)UINT32_MAX;
                next = first + m;
            });
            bad += next != n;
        }
    }
    return bad != 0;
}
""")


PUSH_MAIN = """
template <int W, bool MASK> int check(long long max_blocks) {
    const int E = 400, R = 5;
    unsigned long long rng = 3 + W;
    auto next = [&]() { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33); };
    std::vector<uint32_t> off(E + 1), begin(E);
    std::vector<int32_t> obj, rows;
    std::vector<uint16_t> rel;
    std::vector<unsigned long long> prev((size_t)E * W), known(prev.size()), cur(prev.size()), want(prev.size()), allow((size_t)R * W);
    for (auto &x : allow) x = (unsigned long long)next() << 32 | next();
    std::vector<uint32_t> act((E + 31) / 32 + 1), want_act(act);
    for (int e = 0; e < E; ++e) {
        begin[e] = off[e] = (uint32_t)obj.size();
        for (int d = next() % 33; d > 0; --d) obj.push_back(next() % E), rel.push_back(next() % R);
        const int words = next() % 3 == 0 ? W : 1 + next() % 2;
        for (int i = 0; i < words; ++i) prev[(size_t)e * W + next() % W] |= 1ull << (next() & 63);
        known[(size_t)e * W + next() % W] = (unsigned long long)next() << 32 | next();
        if (obj.size() > begin[e]) rows.push_back(e);
    }
    off[E] = (uint32_t)obj.size();
    for (int e : rows)
        for (uint32_t j = off[e]; j < off[e + 1]; ++j)
            for (int w = 0; w < W; ++w) {
                const unsigned long long m = prev[(size_t)e * W + w] & (MASK ? allow[(size_t)rel[j] * W + w] : ~0ull) & ~known[(size_t)obj[j] * W + w];
                want[(size_t)obj[j] * W + w] |= m;
                if (m) want_act[obj[j] >> 5] |= 1u << (obj[j] & 31);
            }
    unsigned long long ctr[8] = {};
    ctr[C_NTAIL] = rows.size();
    constexpr int G = push_tail_lanes<W>();
    int launches = 0;
    launch_ranges((long long)rows.size(), 256 / G, [&](long long first, long long n) {
        ++launches;
        run_grid((unsigned)((n * G + 255) / 256), 256, {0, 1, 2, 3}, [&] {
            k_push_tail<W, MASK>(rows.data(), first, ctr, off.data(), begin.data(), obj.data(), rel.data(), allow.data(), prev.data(), known.data(),
                                 cur.data(), act.data());
        });
    }, max_blocks);
    const int bad = (cur != want) + (act != want_act) + ((launches > 1) != (max_blocks < 100));
    printf("%d words, mask %d, at most %lld blocks: %d launches, %d wrong\\n", W, MASK, max_blocks, launches, bad);
    return bad;
}

int main() {
    int bad = 0;
    for (long long most : {1ll, 3ll, kMaxBlocks})
        bad += check<1, false>(most) + check<4, true>(most) + check<16, false>(most) + check<16, true>(most);
    return bad != 0;
}
"""


def test_pushed_rows_in_ranges(tmp_path):
    khop = text("khop.hip")
    lanes64 = ("static inline unsigned long long __shfl(unsigned long long v, int from) { return fibers::exchange(v).seen[from & 63]; }\n"
               "static inline int __popc(unsigned x) { return __builtin_popcount(x); }\nstatic inline int __ffs(int x) { return __builtin_ffs(x); }\n"
               "enum { C_NTAIL = 0 };\n")
    run(tmp_path, "".join([lanes64, device_helpers(),
                           between(khop, "__device__ __forceinline__ void mark_active(", "// One wavefront per segment (64"), PUSH_MAIN]))


@pytest.mark.gpu
def test_pulled_rows_past_one_launch():
    """Subject 0 has a triple to each of 2^29 + 70 entities: as many short object rows, with eight lanes each."""
    import torch
    import paper_2604_18913_amd as lkg
    E = (1 << 29) + 70
    zero = np.zeros(E, dtype=np.int32)
    progress("triples")
    g = lkg.Graph(zero, zero, np.arange(E, dtype=np.int32), E, 1)
    progress("graph")
    res = g.khop(np.array([0, 1], np.int64), np.array([0], np.int32), 1, direction="pull")
    progress("search")
    assert res.offsets()[1] == E
    entity, hop, pred = res.fetch()
    assert bool((entity == torch.arange(E, dtype=torch.int32, device="cuda")).all())
    assert hop[0] == 0 and pred[0] == -1 and bool((hop[1:] == 1).all()) and bool((pred[1:] == entity[1:]).all())
    progress("lists")
    res.close()
    g.close()
