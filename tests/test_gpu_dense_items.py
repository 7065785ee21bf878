"""Exhaustive searches where the dense kernel's chunks and items begin and end: one tiling less than a chunk, exactly chunks, one
more; fewer tasks than blocks and several items a block; candidate numbers beyond 2^31 and 2^32; extents in every order of
length, since a chunk's tilings are neighbours in an order of their own.  Against the oracle's enumeration of the
whole space, or, where that is long, against the pruned search: index, energy and latency bit-exact."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

H = dict(pe_rows=4, pe_cols=3, n_arrays=1, rf_bytes=24, gb_bytes=4000, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0)


# tilings: 1, 36, 64, 81 (a chunk and 17), 128 (two), 192, 225, 192
@pytest.mark.parametrize("I, K, L, J, mode", [(1, 1, 1, 1, 0), (4, 8, 4, 1, 0), (8, 8, 2, 2, 0), (36, 1, 36, 1, 1), (8, 8, 8, 2, 0), (2, 128, 32, 2, 0),
                                              (16, 4, 16, 4, 0), (12, 6, 2, 6, 1)])
@pytest.mark.parametrize("gb", [4, 300, 4000, 1 << 40])       # 4: two words, which no mapping fits
def test_chunks_against_the_oracle(I, K, L, J, mode, gb):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c = dict(batch=2, I=I, K=K, L=L, J=J, word_bytes=2, tiling_mode=mode, c_softmax=10)
    h = dict(H, gb_bytes=gb)
    rc, idx, cost, _, _ = O.search_all(O.workload(c), O.hw(h))
    for keys in ([0], [1], [2], [3], [0, 1], [1, 3]):
        if rc:
            results, codes = M.mmee_chain_search_many([(c, h, o) for o in keys], M.SEARCH_EXHAUSTIVE)
            assert rc == M.ENOFEASIBLE and codes == [rc] * len(keys), keys
            assert all(r.cost.valid == 0 and r.best.idx == 2**64 - 1 and r.cost.energy_pj == r.cost.latency_cycles == float("inf") for r in results), keys
            continue
        for o, got in zip(keys, M.mmee_chain_search_multi(c, h, keys, M.SEARCH_EXHAUSTIVE)):
            assert got.best.idx == idx[o], (keys, o)
            assert got.cost.energy_pj == cost[o].energy_pj and got.cost.latency_cycles == cost[o].latency_cycles


# 4900 and 10692 tilings: 2.6e9 and 5.8e9 candidates; long extents first, last and in the middle
@pytest.mark.parametrize("I, K, L, J, mode", [(512, 64, 512, 64, 1), (2048, 768, 3072, 768, 0), (64, 512, 64, 512, 1), (768, 3072, 768, 2048, 0)])
def test_long_searches_against_the_pruned_ones(I, K, L, J, mode):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c = dict(batch=1, I=I, K=K, L=L, J=J, word_bytes=2, tiling_mode=mode, c_softmax=10)
    for gb in (64 << 10, 1 << 40):
        for o in range(4):
            a, b = (M.mmee_chain_search_multi(c, dict(H, gb_bytes=gb), [o], f)[0] for f in (M.SEARCH_EXHAUSTIVE, M.SEARCH_PRUNED))
            assert bytes(a.best) + bytes(a.cost) == bytes(b.best) + bytes(b.cost), (gb, o)


# 30, 32, 36, 441, 448 and 450 tilings: both sides of the lines below which several keys are one pass of k_search
@pytest.mark.parametrize("I, K, L, J", [(16, 4, 2, 1), (8, 2, 8, 1), (4, 8, 4, 1), (64, 64, 36, 1), (64, 24, 24, 1), (16, 16, 12, 4)])
@pytest.mark.parametrize("hw", [dict(gb_bytes=1 << 40), dict(gb_bytes=200), dict(gb_bytes=1 << 40, dram_bw=60.0, gb_bw=100.0), dict(gb_bytes=1 << 40, e_dram=171.3, e_gb=5.7)])
def test_several_keys_against_each_alone(I, K, L, J, hw):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c, h = dict(batch=2, I=I, K=K, L=L, J=J, word_bytes=2, tiling_mode=1, c_softmax=10), dict(H, **hw)
    alone = [M.mmee_chain_search_multi(c, h, [o], M.SEARCH_EXHAUSTIVE)[0] for o in range(4)]
    for mask in range(1, 16):
        keys = [o for o in range(4) if mask >> o & 1]
        for o, got in zip(keys, M.mmee_chain_search_multi(c, h, keys, M.SEARCH_EXHAUSTIVE)):
            assert bytes(got.best) + bytes(got.cost) == bytes(alone[o].best) + bytes(alone[o].cost), (keys, o)
            assert 0 < got.kernel_seconds < got.seconds, (keys, o)


def test_a_search_longer_than_the_host_looks_for():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    c = dict(batch=1, I=360, K=360, L=360, J=360, word_bytes=2, tiling_mode=1, c_softmax=10)     # 331 776 tilings, 1.8e11 candidates
    h = dict(H, gb_bytes=1 << 40, e_dram=171.3, e_gb=5.7)
    for a, b in zip(*(M.mmee_chain_search_multi(c, h, [0, 1, 2, 3], f) for f in (M.SEARCH_EXHAUSTIVE, M.SEARCH_PRUNED))):
        assert bytes(a.best) + bytes(a.cost) == bytes(b.best) + bytes(b.cost)
        assert 0 < a.kernel_seconds < a.seconds


def test_a_large_search_takes_no_memory_per_tiling():
    """102 400 tilings: the tables of the searches that keep them in memory are 2 KiB a tiling."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    small, large = (dict(batch=1, I=n, K=80, L=n, J=80, word_bytes=2, tiling_mode=1, c_softmax=10) for n in (1, 3000))
    M.mmee_shutdown()
    M.mmee_chain_search_multi(small, H, [0], M.SEARCH_EXHAUSTIVE)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    M.mmee_chain_search_multi(large, dict(H, gb_bytes=64 << 10), [0], M.SEARCH_EXHAUSTIVE)
    assert free - torch.cuda.mem_get_info()[0] < 32 << 20
