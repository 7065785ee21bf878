"""Pruned searches of one problem where k_search_batch's blocks and items begin and end, against the exhaustive search of the same
problem, which takes another kernel: a part of a chunk, whole chunks and one more; the last size whose chunks two blocks share and the
next; as many chunks as there are blocks, and some blocks with two.  Buffers that nothing, little and everything fits, and
energies of zero, where every candidate costs the same and the lowest index decides.  Each search twice in a row, and
without allocation in between: the blocks' count is left as it was found."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

HW = dict(pe_rows=24, pe_cols=9, n_arrays=1, rf_bytes=200, gb_bytes=30000, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0)


# tilings: 1, 36, 64 (a chunk), 81, 8100 (127 chunks, the last of 36), 8192 (128), 8640 (135), 16384 (256), 32768 (512), 33280 (520)
@pytest.mark.parametrize("I, K, L, J", [(1, 1, 1, 1), (4, 8, 4, 1), (8, 8, 2, 2), (36, 1, 36, 1), (36, 48, 48, 36), (120, 24, 24, 24), (60, 60, 60, 16),
                                        (120, 24, 120, 24), (120, 120, 120, 24), (120, 120, 4096, 48)])
@pytest.mark.parametrize("hw", [dict(), dict(gb_bytes=1 << 40, e_dram=171.3), dict(gb_bytes=24), dict(gb_bytes=8), dict(gb_bytes=4), dict(gb_bytes=0),
                                dict(e_dram=0.0, e_gb=0.0, e_rf=0.0, e_mac=0.0, dram_bw=0.0, gb_bw=0.0)])
def test_one_problem(I, K, L, J, hw):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c, h = M.chain(dict(batch=2, I=I, K=K, L=L, J=J, word_bytes=2, tiling_mode=1, c_softmax=10)), M.hw(dict(HW, **hw))
    for keys in ([0], [1], [2], [3], [0, 1]):
        want, codes = M.mmee_chain_search_many([(c, h, o) for o in keys], M.SEARCH_EXHAUSTIVE)
        for _ in range(2):
            got, got_codes = M.mmee_chain_search_many([(c, h, o) for o in keys], M.SEARCH_PRUNED)
            assert got_codes == codes == [M.ENOFEASIBLE if h.gb_bytes < 6 else M.OK] * len(keys), keys      # (the smallest mapping takes three words)
            for g, w in zip(got, want):
                assert bytes(g.best) + bytes(g.cost) == bytes(w.best) + bytes(w.cost), keys


def test_calls_without_allocation_in_turn_with_others():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    buf = torch.zeros(C.sizeof(M.Result), dtype=torch.uint8, device="cuda")
    for turn in range(3):
        for seq, gb in ((1, 1 << 20), (64, 4096), (512, 32768), (2048, 1 << 20)):
            w = dict(B=1, H=2, N=seq, d=64, word_bytes=2, tiling_mode=1, c_softmax=10)
            h = dict(HW, gb_bytes=gb)
            for o in range(4):
                M.mmee_search_noalloc(w, h, o, M.SEARCH_PRUNED, buf.data_ptr())
                torch.cuda.synchronize()
                got, want = M.Result.from_buffer_copy(buf.cpu().numpy().tobytes()), M.mmee_search_ex(w, h, o, M.SEARCH_PRUNED)
                assert bytes(got.best) + bytes(got.cost) == bytes(want.best) + bytes(want.cost), (turn, seq, gb, o)
