"""Calls in which one problem's energies, regrouped on trust, have to be summed once more in order: the device times of the
problems that the repetition leaves alone are those of their own launches, and nothing is left for the next call."""
import pytest

pytestmark = pytest.mark.gpu

# 102400 tilings, fractional energies: one launch of k_search_batch takes some 30 us
LARGE = dict(B=1, H=24, N=3000, d=80, word_bytes=2, tiling_mode=1, c_softmax=10)
LARGE_HW = dict(pe_rows=24, pe_cols=9, n_arrays=3, rf_bytes=200, gb_bytes=300000, e_dram=171.3, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=60.0, gb_bw=200.0)
# 225 tilings, whole energies so large that the optimum lies beyond 2^52: proven in order only
SMALL = dict(B=1, H=1, N=16, d=4, word_bytes=2, tiling_mode=1, c_softmax=10)
SMALL_HW = dict(pe_rows=4, pe_cols=4, n_arrays=1, rf_bytes=64, gb_bytes=4096, e_dram=1e13, e_gb=1e13, e_rf=1e13, e_mac=1e13, dram_bw=64.0, gb_bw=256.0)


@pytest.fixture(scope="module")
def M():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as mod
    return mod


@pytest.mark.parametrize("small_keys", [[0, 2], [0]])        # a pass of its own; in the batch with the large one
@pytest.mark.parametrize("large_first", [True, False])
@pytest.mark.parametrize("before", ["nothing", "a long call"])
def test_times_of_what_was_not_repeated(M, small_keys, large_first, before):
    large, small = [(LARGE, LARGE_HW, 0)], [(SMALL, SMALL_HW, o) for o in small_keys]
    points = large + small if large_first else small + large
    M.mmee_shutdown()
    if before == "a long call":                              # an older call's times in every slot, milliseconds
        M.mmee_search_many([(dict(LARGE, H=h), LARGE_HW, 0) for h in (24, 12, 6)], M.SEARCH_EXHAUSTIVE)
    results, codes = M.mmee_search_many(points, M.SEARCH_PRUNED)
    assert not any(codes)
    again = M.mmee_search_ex(LARGE, LARGE_HW, 0)             # (an error left by the call before would be reported here)
    lone = min(M.mmee_search_ex(LARGE, LARGE_HW, 0).kernel_seconds for _ in range(5))
    for (w, h, o), r in zip(points, results):
        want = M.mmee_search_ex(w, h, o, M.SEARCH_ORDERED_SUM)
        assert bytes(r.best) + bytes(r.cost) == bytes(want.best) + bytes(want.cost), (w, o)
        assert 0 < r.kernel_seconds <= r.seconds
        if w is LARGE:
            assert 0.5 * lone < r.kernel_seconds < 20 * lone, (r.kernel_seconds, lone)
            assert bytes(r.best) == bytes(again.best)
        else:
            assert r.cost.energy_pj >= 2.0 ** 52
