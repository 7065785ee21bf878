"""Pruned searches of more than 256 chunks, where k_search_batch takes its rows as straight-line code (a block per chunk),
against the search of the full row set, which takes other kernels: every key set, whole chunks and a remainder, buffers that nothing, little
and everything fits, energies and bandwidths of every kind; and a batch of problems whose chunks together are that many."""
import pytest

pytestmark = pytest.mark.gpu

HW = dict(pe_rows=24, pe_cols=9, n_arrays=1, rf_bytes=200, gb_bytes=30000, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0)
SHAPES = [dict(I=96, K=60, L=96, J=60),                      # 20736 tilings, 324 chunks
          dict(I=4096, K=60, L=4096, J=72)]                  # 24336: 381 chunks, the last of 16 tilings


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("hw", [dict(), dict(gb_bytes=1 << 40, e_dram=171.3), dict(gb_bytes=24), dict(gb_bytes=4), dict(dram_bw=60.0, gb_bw=100.0, n_arrays=3, e_gb=5.7)])
def test_straight_line_rows(shape, hw):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c, h = M.chain(dict(batch=2, word_bytes=2, tiling_mode=1, c_softmax=10, **shape)), M.hw(dict(HW, **hw))
    for keys in ([0], [1], [2], [3], [0, 1]):
        got, codes = M.mmee_chain_search_many([(c, h, o) for o in keys], M.SEARCH_PRUNED)
        want, want_codes = M.mmee_chain_search_many([(c, h, o) for o in keys], M.SEARCH_EXHAUSTIVE)
        assert codes == want_codes == [M.ENOFEASIBLE if h.gb_bytes < 6 else M.OK] * len(keys), keys      # (the smallest mapping takes three words)
        for g, w in zip(got, want):
            assert bytes(g.best) + bytes(g.cost) == bytes(w.best) + bytes(w.cost), keys


def test_a_batch_of_small_problems():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    points = []
    for k in range(24):                                      # 24 shapes of 6 to 25 chunks: too little shared for k_search_pruned
        c = M.chain(dict(batch=1 + k % 3, I=12 * (k + 4), K=20, L=24 + 12 * (k % 5), J=12, word_bytes=2, tiling_mode=1, c_softmax=10))
        points.append((c, M.hw(dict(HW, gb_bytes=2000 + 700 * k)), k % 4))
    got, codes = M.mmee_chain_search_many(points, M.SEARCH_PRUNED)
    for (c, h, o), g, code in zip(points, got, codes):
        want, want_codes = M.mmee_chain_search_many([(c, h, o)], M.SEARCH_EXHAUSTIVE)
        assert code == want_codes[0] and (code or bytes(g.best) + bytes(g.cost) == bytes(want[0].best) + bytes(want[0].cost))
