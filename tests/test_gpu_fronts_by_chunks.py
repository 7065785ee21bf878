"""The fronts over the kept rows (k_front_points, k_front_merge) against the walk over the full row set, which takes
other kernels and must find the same points: fewer tilings than a chunk, whole chunks and remainders, one merge list
and several, problems beyond what the chunked path takes, capacities nothing fits, room for fewer points than there are.
The library counts the fronts it walks: every problem of at most 512 chunks of 64 tilings is to take the chunked path,
also where there are many points.  The counts are of points that are on the front of their wave, block or list, before the launch's
staircase drops what other blocks cover; which of the kernels' ways the largest take is test_gpu_front_ways's."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

HW = dict(pe_rows=5, pe_cols=8, n_arrays=1, rf_bytes=64, gb_bytes=20000, e_dram=171.3, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=3.0, gb_bw=20.0)


@pytest.mark.parametrize("shape,hw,walked", [
    (dict(batch=1, I=2, K=3, L=2, J=3), dict(gb_bytes=30), False),              # 16 tilings
    (dict(batch=3, I=8, K=8, L=8, J=1), dict(), False),                         # 64
    (dict(batch=1, I=36, K=16, L=36, J=4), dict(dram_bw=1.0), False),           # 9 * 5 * 9 * 3 = 1215: 19 chunks
    (dict(batch=2, I=720, K=12, L=360, J=6), dict(gb_bytes=4000), False),       # 30 * 6 * 24 * 4 = 17280: 270 chunks, 75 points in a wave
    (dict(batch=1, I=720, K=24, L=720, J=30), dict(dram_bw=60.0), True),        # 30 * 8 * 30 * 8 = 57600: walked
    (dict(batch=1, I=36, K=16, L=36, J=4), dict(gb_bytes=4), False),            # nothing fits
    (dict(batch=1, I=1173, K=128, L=1173, J=128, tiling_mode=0), dict(), False),    # 64 tilings, 66 points in a wave
    (dict(batch=1, I=600, K=64, L=600, J=64), dict(), False),                   # 28224 tilings, 99 points in a block
    (dict(batch=1, I=720720, K=1, L=1, J=1), dict(), False),                    # 240 tilings, 67 points in a wave, 2 in all
    (dict(batch=1, I=20160, K=1009, L=1680, J=1), dict(), False),               # 6720 tilings, 1069 points in a block's waves
    (dict(batch=1, I=1009, K=55440, L=36, J=36), dict(), False),                # 19440 tilings, 6917 points in all lists
])
def test_same_points_as_the_full_row_set(shape, hw, walked):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    walks = M._lib.mmee_front_walks
    walks.restype = ctypes.c_uint64
    c, h = dict(dict(word_bytes=2, tiling_mode=1, c_softmax=10), **shape), dict(HW, **hw)
    for front in (M.mmee_chain_pareto, M.mmee_chain_front_bs_da):
        before = walks()
        code, got = front(c, h, M.SEARCH_PRUNED)
        assert walks() - before == int(walked), front
        want_code, want = front(c, h, M.SEARCH_EXHAUSTIVE)
        assert walks() - before == int(walked) + 1
        assert code == want_code and len(got) == len(want), (front, code, want_code, len(got), len(want))
        assert [bytes(r.best) + bytes(r.cost) for r in got] == [bytes(r.best) + bytes(r.cost) for r in want]
        # counted per point, as a walk over the kept rows would
        per_pass = (86 + 74 + 110) * (want[0].space // 540000) * (9 if front is M.mmee_chain_pareto else 1) if want else 0
        assert all(r.evaluated == per_pass * (len(got) + 1) for r in got)
        print(front.__name__, len(got), flush=True)
        if len(want) > 1:
            code, few = front(c, h, M.SEARCH_PRUNED, capacity=len(want) - 1)
            assert code == M.EOVERFLOW and [bytes(r.best) for r in few] == [bytes(r.best) for r in want[:-1]]
