"""Fronts over the kept rows where the staircase that drops covered candidates is coarse, clamped or left over: latencies
far above and below the estimate its steps start from (no DRAM time, a slow bus, one array cell), buffer sizes in one
step, ties across blocks; both kinds of front in turn on changing problems, so that a staircase or counter that a call left
behind would cover points of the next.  Against the walk over the full row set, which takes other kernels."""
import random

import pytest

pytestmark = pytest.mark.gpu

HW = dict(pe_rows=5, pe_cols=8, n_arrays=1, rf_bytes=64, gb_bytes=20000, e_dram=171.3, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=3.0, gb_bw=20.0)


def test_same_points_in_any_order_of_calls():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    problems = []
    for shape in (dict(batch=1, I=1, K=1, L=1, J=1), dict(batch=7, I=64, K=16, L=64, J=16), dict(batch=1, I=97, K=60, L=1, J=101),
                  dict(batch=2, I=48, K=30, L=36, J=20)):
        for hw in (dict(), dict(dram_bw=0.0), dict(dram_bw=1e-6), dict(gb_bw=1e-5), dict(gb_bw=0.0, dram_bw=0.0, pe_rows=1, pe_cols=1),
                   dict(pe_rows=512, pe_cols=512, dram_bw=1e9, gb_bw=1e9), dict(e_dram=0.0, e_gb=0.0, e_rf=0.0, e_mac=0.0), dict(gb_bytes=8)):
            problems.append((dict(dict(word_bytes=2, tiling_mode=1, c_softmax=10), **shape), dict(HW, **hw)))
    want = {}
    for n, (c, h) in enumerate(problems):
        for front in (M.mmee_chain_pareto, M.mmee_chain_front_bs_da):
            code, points = front(c, h, M.SEARCH_EXHAUSTIVE)
            want[n, front] = code, [bytes(r.best) + bytes(r.cost) for r in points]
    calls = list(want) * 2
    random.Random(3).shuffle(calls)
    for n, front in calls:
        code, points = front(*problems[n], M.SEARCH_PRUNED)
        assert (code, [bytes(r.best) + bytes(r.cost) for r in points]) == want[n, front], (problems[n], front.__name__)
