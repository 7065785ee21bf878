"""The buffer-size / DRAM-access front where its parts run out of room: a block's points sorted instead of settled pair by
pair (more than 512), the merge's list in several turns (more than 4096), its points sorted at the end (more than 1024) or before
(more than 2048); and, with less room for a block's points than there is, a block's waves one after the other, and the walk where that
does not help.  Against the walk over the full row set.

That a shape takes these ways is certain whatever the blocks know of one another: a candidate dropped for what another block
published is covered by a point that stays in the launch, and so is all that it would have covered, so with less known a wave's
front only grows.  The counts here hold with every block knowing the complete staircase (counted on the CPU from the kept rows)."""
import ctypes
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HW = dict(pe_rows=5, pe_cols=8, n_arrays=1, rf_bytes=64, gb_bytes=20000, e_dram=171.3, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=3.0, gb_bw=20.0)
OUTGROWN, POOL_SORTED, WAVE_BY_WAVE, TURNS, SORTED, SORTED_EARLY = (1 << k for k in range(6))


@pytest.mark.parametrize("shape,ways,not_ways", [
    ((36, 16, 36, 4), 0, 63),                                                   # 758 points in all lists at most
    ((20160, 1009, 1680, 1), SORTED, OUTGROWN | SORTED_EARLY),                  # 1550 points left
    ((110880, 332640, 1, 1), POOL_SORTED, OUTGROWN | SORTED_EARLY),             # 580 points in a block, 610 left
    ((332640, 20160, 997, 1), POOL_SORTED | TURNS | SORTED_EARLY, OUTGROWN),    # 634 in a block, a list of 22281, 11594 left
])
def test_ways_of_a_large_front(shape, ways, not_ways):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2604_03446_amd as M
    way, walks = M._lib.mmee_front_way, M._lib.mmee_front_walks
    way.restype, walks.restype = ctypes.c_uint32, ctypes.c_uint64
    c = dict(zip("IKLJ", shape), batch=1, word_bytes=2, tiling_mode=1, c_softmax=10)
    want_code, want = M.mmee_chain_front_bs_da(c, HW, M.SEARCH_EXHAUSTIVE, capacity=4096)
    for _ in range(3):                                       # (what the blocks know of one another is another each time)
        before = walks()
        code, got = M.mmee_chain_front_bs_da(c, HW, M.SEARCH_PRUNED, capacity=4096)
        assert walks() == before
        print(shape, len(got), bin(way()), flush=True)
        assert way() & ways == ways and not way() & not_ways, bin(way())
        assert code == want_code and [bytes(r.best) + bytes(r.cost) for r in got] == [bytes(r.best) + bytes(r.cost) for r in want]


SMALL_POOL = r"""
import ctypes, sys
sys.path.insert(0, %r)
import torch
import paper_2604_03446_amd as M
way, walks = M._lib.mmee_front_way, M._lib.mmee_front_walks
way.restype, walks.restype = ctypes.c_uint32, ctypes.c_uint64
hw = dict(pe_rows=5, pe_cols=8, n_arrays=1, rf_bytes=64, gb_bytes=20000, e_dram=171.3, e_gb=6.0, e_rf=1.0, e_mac=1.0, dram_bw=3.0, gb_bw=20.0)
for shape, mode in (((36, 16, 36, 4), 1), ((1173, 128, 1173, 128), 0), ((20160, 1009, 1680, 1), 1)):
    c = dict(zip("IKLJ", shape), batch=1, word_bytes=2, tiling_mode=mode, c_softmax=10)
    for front in (M.mmee_chain_front_bs_da, M.mmee_chain_pareto):
        want = front(c, hw, M.SEARCH_EXHAUSTIVE, capacity=1024)
        before = walks()
        got = front(c, hw, M.SEARCH_PRUNED, capacity=1024)
        assert got[0] == want[0] and [bytes(r.best) + bytes(r.cost) for r in got[1]] == [bytes(r.best) + bytes(r.cost) for r in want[1]], (shape, front)
        assert (walks() - before == 1) == bool(way() & 1), (shape, front)
        print("WAY", front.__name__, shape[0], way(), flush=True)
"""


@pytest.mark.parametrize("pool", [1, 32, 64])
def test_less_room_than_there_is(pool):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, "-c", SMALL_POOL % root], capture_output=True, text=True, timeout=100, env=dict(os.environ, MMEE_FRONT_POOL=str(pool)))
    assert p.returncode == 0, p.stderr[-2000:]
    print(p.stdout)
    way = {tuple(ln.split()[1:3]): int(ln.split()[3]) for ln in p.stdout.splitlines() if ln.startswith("WAY")}
    assert len(way) == 6
    if pool == 1:                                            # no room for the first point
        assert all(w & OUTGROWN for w in way.values())
    if pool == 32:                                           # at least 34 points and places asked for in vain in a block of 36 x 16 x 36 x 4
        assert way["mmee_chain_front_bs_da", "36"] & WAVE_BY_WAVE
    if pool == 64:                                           # at least 67 in a block of 1173 x 128 x 1173 x 128
        assert way["mmee_chain_front_bs_da", "1173"] & WAVE_BY_WAVE
