"""Exhaustive searches at the capacities where rows start and stop to fit: the dense kernel compares a row's (A, B) part
with what its (D, E) part and C leave of the buffer, and passes over rows that no tiling of a wave fits.  Capacities
are buffer sizes that occur (a row exactly fills the buffer), one word less, the smallest and the largest there are, one
tiling's worth and none.  Against the oracle's enumeration of the whole space: index, energy and latency bit-exact."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

# 81 tilings: a full chunk of 64 and a ragged one
W = dict(B=1, H=2, N=36, d=1, word_bytes=2, tiling_mode=1, c_softmax=10)
H = dict(pe_rows=4, pe_cols=3, n_arrays=1, rf_bytes=24, gb_bytes=0, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0,
         dram_bw=64.0, gb_bw=256.0)


@pytest.mark.parametrize("change", [dict(), dict(dram_bw=60.0), dict(e_dram=171.3), dict(e_gb=5.7, dram_bw=3.7)])
def test_capacities_that_rows_fill_exactly(change):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    h = dict(H, **change)
    sizes = M.mmee_eval_batch(W, dict(h, gb_bytes=1 << 40), 0, M.mmee_space_size(W, h) // 18)["bs_words"]
    sizes = sorted({int(v) for v in sizes} - {0})
    some = sizes[:3] + sizes[len(sizes) // 2:len(sizes) // 2 + 2] + sizes[-2:]
    for words in sorted({0, 1 << 60} | set(some) | {v - 1 for v in some}):
        hc = dict(h, gb_bytes=2 * words)
        rc, idx, cost, _, _ = O.search_all(O.workload(W), O.hw(hc))
        for keys in ([0], [1], [2], [3], [0, 1], [0, 3]):
            if rc:
                for o in keys:
                    assert M.mmee_search_ex(W, hc, o, M.SEARCH_EXHAUSTIVE, allow_infeasible=True)[0] == M.ENOFEASIBLE, (words, o)
                continue
            for o, got in zip(keys, M.mmee_search_multi(W, hc, keys, M.SEARCH_EXHAUSTIVE)):
                assert got.best.idx == idx[o], (words, keys, o)
                assert got.cost.energy_pj == cost[o].energy_pj and got.cost.latency_cycles == cost[o].latency_cycles
