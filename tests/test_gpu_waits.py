"""Short calls wait for a word in pinned memory that their last kernel writes, and fall back to the stream when it is long in
coming: work of the caller's ahead of them on the stream, calls of several threads, every key set; records and device
times are those of the call itself."""
import threading

import pytest

pytestmark = pytest.mark.gpu

W = dict(B=1, H=4, N=96, d=40, word_bytes=2, tiling_mode=1, c_softmax=10)
H = dict(pe_rows=8, pe_cols=8, n_arrays=1, rf_bytes=64, gb_bytes=20000, e_dram=200.0, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=64.0, gb_bw=256.0)
KEYS = ([0], [1], [2], [3], [0, 1])


def records(M, h=H):
    return [[bytes(r.best) + bytes(r.cost) for r in M.mmee_search_multi(W, h, keys)] for keys in KEYS] + \
        [[bytes(r.best) + bytes(r.cost) for r in front(W, h)[1]] for front in (M.mmee_pareto, M.mmee_front_bs_da)]


def test_work_ahead_on_the_stream():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    want = records(M)
    stream = torch.cuda.Stream()
    M._lib.mmee_set_stream(stream.cuda_stream)
    try:
        for k, keys in enumerate(KEYS):
            with torch.cuda.stream(stream):
                torch.cuda._sleep(120_000_000)               # some 50 ms, longer than the word is looked for
            got = M.mmee_search_multi(W, H, keys)
            assert [bytes(r.best) + bytes(r.cost) for r in got] == want[k]
            assert 0 < got[0].kernel_seconds < 0.02 < got[0].seconds
        for k, front in enumerate((M.mmee_pareto, M.mmee_front_bs_da)):
            with torch.cuda.stream(stream):
                torch.cuda._sleep(120_000_000)
            points = front(W, H)[1]
            assert [bytes(r.best) + bytes(r.cost) for r in points] == want[len(KEYS) + k]
            assert 0 < points[0].kernel_seconds < 0.02 < points[0].seconds
    finally:
        M._lib.mmee_set_stream(None)


def test_several_threads():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    hws = [dict(H, gb_bytes=8000 + 4000 * k) for k in range(4)]
    want = [records(M, h) for h in hws]
    got = [None] * len(hws)

    def work(k):
        got[k] = [records(M, hws[k]) for _ in range(20)]

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(hws))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(len(hws)):
        assert all(g == want[k] for g in got[k])
