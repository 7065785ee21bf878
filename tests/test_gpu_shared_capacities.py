"""Shared pruned searches (k_search_pruned) at the numbers of distinct capacities where its row loop changes width and where a
round of capacities ends, against one call per problem, which takes another kernel."""
import random

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_caps", [2, 3, 6, 7, 10, 11, 32, 33])
def test_widths_of_the_row_loop(n_caps):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    rng = random.Random(n_caps)
    w = dict(B=1, H=3, N=60, d=24, word_bytes=2, tiling_mode=1, c_softmax=10)
    caps = rng.sample(range(60, 30000), n_caps)
    points = []
    for k in range(max(n_caps, 24)):
        h = dict(pe_rows=rng.choice([1, 3, 8, 16]), pe_cols=rng.choice([2, 7, 32]), n_arrays=rng.choice([1, 2, 3]), rf_bytes=rng.choice([8, 64, 96]),
                 gb_bytes=2 * caps[k % n_caps], e_dram=rng.uniform(100, 300), e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=rng.choice([64.0, 60.0]),
                 gb_bw=rng.choice([256.0, 100.0]))
        points += [(w, h, o) for o in (0, 1, 3)]             # a key set only this kernel shares
    results, codes = M.mmee_search_many(points, M.SEARCH_PRUNED)
    for (w, h, o), r, code in zip(points, results, codes):
        want_code, want = M.mmee_search_ex(w, h, o, M.SEARCH_PRUNED, allow_infeasible=True)
        assert code == want_code, (h, o)
        if not code:
            assert bytes(r.cost) == bytes(want.cost) and bytes(r.best) == bytes(want.best), (h, o)
