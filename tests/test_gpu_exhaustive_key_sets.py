"""Exhaustive searches for several keys in one call, either side of the sizes at which the kernel changes, against
one call per key (which takes the dense kernel at every size): every key set, power-of-two and other bandwidths and
array counts, energies that regroup, that let the first sum be fused and that do neither."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 1), (2, 1, 4, 1), (8, 1, 8, 1), (4, 2, 4, 4), (8, 4, 8, 4), (8, 8, 8, 8), (256, 2, 256, 2), (16, 8, 16, 8),
          (128, 4, 128, 4), (32, 16, 32, 16), (16, 16, 16, 128), (64, 16, 64, 16), (256, 8, 256, 8), (128, 32, 128, 32), (128, 64, 128, 64),
          (128, 128, 128, 128), (512, 64, 512, 64), (4096, 64, 4096, 64)]
HW = dict(pe_rows=16, pe_cols=7, n_arrays=1, rf_bytes=256, gb_bytes=20000, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0)
KINDS = [dict(), dict(e_dram=171.3), dict(e_dram=171.3, e_gb=5.7), dict(dram_bw=60.0, n_arrays=3), dict(e_dram=171.3, e_gb=5.7, dram_bw=60.0)]


@pytest.mark.parametrize("kind", range(len(KINDS)))
def test_several_keys_find_what_each_finds_alone(kind):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    h = dict(HW, **KINDS[kind])
    for I, K, L, J in SHAPES:
        c = dict(batch=3, I=I, K=K, L=L, J=J, word_bytes=2, tiling_mode=0, c_softmax=10)
        alone = [M.mmee_chain_search_multi(c, h, [o], M.SEARCH_EXHAUSTIVE)[0] for o in range(4)]
        for mask in range(1, 16):
            keys = [o for o in range(4) if mask >> o & 1]
            got = M.mmee_chain_search_multi(c, h, keys, M.SEARCH_EXHAUSTIVE)
            for o, r in zip(keys, got):
                assert bytes(r.best) + bytes(r.cost) == bytes(alone[o].best) + bytes(alone[o].cost), (I, K, L, J, mask, o)
                assert r.evaluated == alone[o].evaluated
