"""Exhaustive searches under every way the dense kernel adds a candidate's energy up, against the
oracle's enumeration of the whole space: whole-number energies with a DRAM bandwidth or array count
that is no power of two (regrouped sum), a whole buffer energy next to fractional ones (fused
first sum), a fractional buffer energy (summed in order), and a whole buffer energy too large for its
product to be exact (in order again).  Index, energy and latency bit-exact."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

W = dict(B=1, H=3, N=24, d=10, word_bytes=2, tiling_mode=1, c_softmax=10)
H = dict(pe_rows=4, pe_cols=3, n_arrays=1, rf_bytes=24, gb_bytes=900, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0,
         dram_bw=64.0, gb_bw=256.0)


@pytest.mark.parametrize("change", [
    dict(dram_bw=60.0), dict(n_arrays=3), dict(dram_bw=0.0, n_arrays=3),
    dict(e_dram=137.25), dict(e_dram=137.25, dram_bw=60.0), dict(e_rf=0.3, e_mac=0.7, n_arrays=3),
    dict(e_gb=5.7, e_dram=137.3), dict(e_gb=5.7, dram_bw=60.0), dict(e_gb=0.0, e_dram=0.1),
    dict(e_gb=2.0 ** 40, e_rf=0.1), dict(gb_bytes=60, e_dram=137.25), dict(gb_bytes=8),
])
def test_exhaustive_energy_against_the_oracle(change):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    h = dict(H, **change)
    ow, oh = O.workload(W), O.hw(h)
    for objective in (M.OBJ_ENERGY, M.OBJ_LATENCY_THEN_ENERGY):
        rc, idx, cost, _, _ = O.search(ow, oh, objective)
        code, got = M.mmee_search_ex(W, h, objective, M.SEARCH_EXHAUSTIVE, allow_infeasible=True)
        assert (code == 0) == (rc == 0), (change, objective)
        if rc == 0:
            assert got.best.idx == idx, (change, objective)
            assert got.cost.energy_pj == cost.energy_pj and got.cost.latency_cycles == cost.latency_cycles
        print(change, objective, "ok", flush=True)


@pytest.mark.parametrize("change", [dict(), dict(dram_bw=60.0), dict(n_arrays=3, e_dram=137.25), dict(e_gb=5.7, dram_bw=3.7)])
def test_exhaustive_key_sets_against_the_oracle(change):
    """Every set of keys: the passes the dense kernel makes of it return each key's own optimum."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    w, h = dict(W, N=18, d=4), dict(H, gb_bytes=300, **change)
    rc, idx, cost, _, _ = O.search_all(O.workload(w), O.hw(h))
    assert rc == 0
    for mask in range(1, 16):
        keys = [o for o in range(4) if mask >> o & 1]
        for o, got in zip(keys, M.mmee_search_multi(w, h, keys, M.SEARCH_EXHAUSTIVE)):
            assert got.best.idx == idx[o], (change, keys, o)
            assert got.cost.energy_pj == cost[o].energy_pj and got.cost.latency_cycles == cost[o].latency_cycles
