"""Many accelerators on few shapes in one call (k_search_pruned: shared row side, capacities in rounds of
sixteen, groups of at most 64 problems) against one call per problem, which takes another kernel.  Every key set;
fewer tilings than a chunk, whole chunks and a remainder; one capacity for all, more capacities than a round,
more problems than a group; capacities nothing fits; bandwidths, array counts and energies of every kind."""
import random

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as mod
    return mod


SHAPES = [dict(N=2, d=3, tiling_mode=1), dict(N=60, d=10, tiling_mode=1), dict(N=64, d=32, tiling_mode=0), dict(N=36, d=75, tiling_mode=1)]


def accelerators(rng, n, caps):
    return [dict(pe_rows=rng.choice([1, 3, 8, 16]), pe_cols=rng.choice([2, 7, 8, 32]), n_arrays=rng.choice([1, 1, 2, 3]),
                 rf_bytes=rng.choice([8, 64, 96]), gb_bytes=caps[k % len(caps)], e_dram=rng.choice([200.0, rng.uniform(100, 300), 0.0]),
                 e_gb=rng.choice([6.0, 5.7]), e_rf=rng.choice([1.0, 0.0]), e_mac=1.0, dram_bw=rng.choice([64.0, 60.0, 0.0]),
                 gb_bw=rng.choice([256.0, 100.0, 0.0])) for k in range(n)]


@pytest.mark.parametrize("n,n_caps", [(8, 1), (9, 5), (17, 16), (40, 17), (64, 64), (70, 70)])
def test_same_results_as_one_call_per_problem(M, n, n_caps):
    rng = random.Random(1000 * n + n_caps)
    caps = [4] + [rng.randrange(100, 60000) for _ in range(n_caps - 1)] if n_caps > 1 else [4000]
    points = []
    for shape in rng.sample(SHAPES, 2):
        w = dict(B=1, H=rng.choice([1, 3]), word_bytes=2, c_softmax=10, **shape)
        for k, h in enumerate(accelerators(rng, n, caps)):
            mask = (k % 15) + 1
            points += [(w, h, o) for o in range(4) if mask >> o & 1]
    results, codes = M.mmee_search_many(points, M.SEARCH_PRUNED)
    infeasible = 0
    for (w, h, o), r, code in zip(points, results, codes):
        want_code, want = M.mmee_search_ex(w, h, o, M.SEARCH_PRUNED, allow_infeasible=True)
        assert code == want_code, (w, h, o)
        infeasible += code != 0
        if code:
            assert r.cost.valid == 0
            continue
        assert r.best.idx == want.best.idx, (w, h, o)
        assert bytes(r.cost) == bytes(want.cost) and bytes(r.best) == bytes(want.best), (w, h, o)
        assert r.evaluated == want.evaluated and r.space == want.space
    if n_caps > 1:
        assert 0 < infeasible < len(points)
    # once more: nothing of a call is left for the next
    again, codes2 = M.mmee_search_many(points, M.SEARCH_PRUNED)
    assert list(codes2) == list(codes) and [r.best.idx for r in again] == [r.best.idx for r in results]


@pytest.mark.parametrize("n", [1, 255, 257, 4096, 4097])
def test_decode_of_short_and_long_lists(M, n):
    """Lists up to 4096 indices are read and written in pinned host memory, longer ones on the device."""
    import oracle as O
    w, h = dict(B=1, H=2, N=60, d=10, word_bytes=2, tiling_mode=1, c_softmax=10), accelerators(random.Random(n), 1, [4000])[0]
    space = M.mmee_space_size(w, h)
    idx = [random.Random(n + k).randrange(space) for k in range(n)]
    got = M.mmee_decode(w, h, idx)
    assert [m.idx for m in got] == idx
    for k in sorted({0, n // 2, n - 1, min(n - 1, 255), min(n - 1, 256)}):
        want, _, _ = O.evaluate(O.workload(w), O.hw(h), idx[k])
        for fld in ("xG", "xD", "order", "level"):
            assert list(getattr(got[k], fld)) == list(getattr(want, fld)), (n, k, fld)
        assert (got[k].recompute, got[k].stat1, got[k].stat2, got[k].fused) == (want.recompute, want.stat1, want.stat2, want.fused)


def test_records_of_a_shape_take_room_for_its_own_problems(M):
    """One shape of sixty-four problems beside one of many tilings and four problems: what the call keeps on the device
    goes by each shape's own number of problems (4 MB of records here; 62 MB if all were sized for the largest)."""
    import torch
    rng = random.Random(3)
    small = dict(batch=1, I=8, K=2, L=8, J=2, word_bytes=2, tiling_mode=0, c_softmax=0)
    large = dict(batch=1, I=5040, K=720, L=360, J=48, word_bytes=2, tiling_mode=1, c_softmax=0)      # 60 * 30 * 24 * 10 = 432000 tilings
    sizes = [(small, 64), (dict(small, batch=2), 64), (large, 4)]
    points = [(c, h, 0) for c, n in sizes for h in accelerators(rng, n, [4000, 40000])]
    M.mmee_shutdown()
    M.mmee_chain_search_many(points[:2], M.SEARCH_PRUNED)        # the offline stage and the small buffers
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    results, codes = M.mmee_chain_search_many(points, M.SEARCH_PRUNED)
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken < 48 << 20, taken
    for (c, h, o), r, code in zip(points, results, codes):
        assert code == 0
        want = M.mmee_chain_search_multi(c, h, [o], M.SEARCH_PRUNED)[0]
        assert bytes(r.cost) == bytes(want.cost) and r.best.idx == want.best.idx


def test_shapes_of_many_problems_share_beside_single_ones(M):
    """Sixty-four problems on one shape of 324 chunks beside forty shapes with one problem each: the call takes the former through
    the kernel that shares the row side and the latter through the batched one, each with the device time of its launches."""
    rng = random.Random(11)
    shape = dict(batch=1, I=2048, K=2048, L=2048, J=2048, word_bytes=2, tiling_mode=0, c_softmax=0)
    h = accelerators(rng, 64, [20000, 60000, 500000])
    many = [(shape, dict(k, gb_bytes=k["gb_bytes"] + 2 * n), o) for n, k in enumerate(h) for o in (0, 1)]
    single = [(dict(shape, K=64 * (2 * q + 1)), accelerators(rng, 1, [100000])[0], 0) for q in range(40)]
    points = many + single
    results, codes = M.mmee_chain_search_many(points, M.SEARCH_PRUNED)
    assert not any(codes)
    times = [{r.kernel_seconds for r in results[a:b]} for a, b in ((0, len(many)), (len(many), len(points)))]
    assert all(len(t) == 1 for t in times) and times[0] != times[1]
    for (c, h, o), r in zip(points, results):
        want = M.mmee_chain_search_multi(c, h, [o], M.SEARCH_PRUNED)[0]
        assert bytes(r.cost) == bytes(want.cost) and bytes(r.best) == bytes(want.best) and r.evaluated == want.evaluated, (c, h, o)


def test_order_of_the_problems_does_not_matter(M):
    """Waves drop what a lower published value beats, so which positions are recovered hangs on who publishes first:
    the same problems in other orders (other places in their group, other waves), and the same call again and again, with
    accelerators whose optima many tilings reach."""
    rng = random.Random(23)
    points = []
    for c in (dict(batch=2, I=512, K=64, L=512, J=64, word_bytes=2, tiling_mode=0, c_softmax=10),
              dict(batch=1, I=360, K=48, L=360, J=48, word_bytes=2, tiling_mode=1, c_softmax=10)):
        for n, h in enumerate(accelerators(rng, 40, [20000, 50000, 400000])):
            h = dict(h, gb_bytes=h["gb_bytes"] + 64 * n, **(dict(dram_bw=0.0, gb_bw=0.0) if n % 4 == 0 else {}))
            points += [(c, h, o) for o in ((0, 1), (2,), (3, 1), (0, 1, 2, 3))[n % 4]]
    want, codes = M.mmee_chain_search_many(points, M.SEARCH_PRUNED)
    assert not any(codes)
    single = [M.mmee_chain_search_multi(c, h, [o], M.SEARCH_PRUNED)[0] for c, h, o in points]
    assert [bytes(r.best) + bytes(r.cost) for r in want] == [bytes(r.best) + bytes(r.cost) for r in single]
    for turn in range(8):
        order = list(range(len(points)))
        if turn >= 4:
            rng.shuffle(order)
        got, _ = M.mmee_chain_search_many([points[k] for k in order], M.SEARCH_PRUNED)
        assert all(bytes(r.best) + bytes(r.cost) == bytes(want[k].best) + bytes(want[k].cost) for k, r in zip(order, got)), turn
