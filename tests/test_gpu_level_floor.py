"""What the level floor counts, read off one at a time with unit costs: barriers
and barrier-free levels of thin-run windows, hand-overs between the windows of a
spread run, launches."""
import numpy as np
import pytest
import torch

import gen
import oracle
from tests.gpu_util import dev, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")

FIELDS = ("thin_level_ns", "thin_wave_level_ns", "launch_ns", "graph_node_ns", "grid_barrier_ns", "flag_hop_ns")


def _chain_of_levels(widths):
    """Level l has widths[l] rows; a row reads the first row of the level before."""
    first = np.concatenate([[0], np.cumsum(widths)])
    rp, col, val = [0], [], []
    for l, w in enumerate(widths):
        for r in range(first[l], first[l + 1]):
            if l:
                col.append(first[l - 1])
                val.append(-0.5)
            col.append(r)
            val.append(2.0)
            rp.append(len(col))
    return gen.Csr(int(first[-1]), np.array(rp, np.int32), np.array(col, np.int32), np.array(val))


def _counts(h, nrhs, **kw):
    out = {}
    for f in FIELDS:
        costs = dict.fromkeys(FIELDS, 0.0)
        costs[f] = 1.0
        out[f] = round(h.level_floor(costs, sp.ORIGINAL, nrhs, **kw) * 1e3, 6)
    return out


@pytest.mark.parametrize("widths,barriers", [
    ([1] * 40, 0),                       # one wave throughout
    ([100] + [1] * 50, 1),               # after the wide level only
    ([100] + [1] * 50 + [100] + [1] * 50, 3),
    ([1, 65, 64, 1, 1, 70], 4),          # around each level of more than 64 rows
    ([600] + [1] * 5 + [600], 7),        # more rows than threads: a barrier per level
])
def test_barriers_of_a_window(widths, barriers):
    h = sp.Handle()
    h.analyze(*dev(_chain_of_levels(widths)))
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=512)
    n = _counts(h, 1)
    assert (n["thin_level_ns"], n["thin_wave_level_ns"]) == (barriers, len(widths) - barriers)
    assert (n["launch_ns"], n["flag_hop_ns"]) == (3, 0)  # gather, one window, scatter
    assert _counts(h, 1, rows=True)["launch_ns"] == 1


def test_columns_count_as_items():
    h = sp.Handle()
    h.analyze(*dev(_chain_of_levels([1, 33, 1, 1])))
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=512)
    assert _counts(h, 1)["thin_level_ns"] == 0
    assert _counts(h, 2)["thin_level_ns"] == 2  # 66 items, and the level before
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=512, thin_cols=1)
    assert _counts(h, 2)["thin_level_ns"] == 0


def test_hand_overs_of_a_spread_run():
    m = _chain_of_levels([1500] * 10)  # more than one window's rows
    h = sp.Handle()
    h.analyze(*dev(m))
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=1024)
    one, two = _counts(h, 1), _counts(h, 2)
    assert one["flag_hop_ns"] >= 3 and two["flag_hop_ns"] >= one["flag_hop_ns"]
    assert one["launch_ns"] == 3  # the gather of one column marks x
    assert two["launch_ns"] == 4
    assert _counts(h, 2, rows=True)["launch_ns"] == 2
    assert _counts(h, 2, graph=True)["graph_node_ns"] == 4
    assert one["thin_level_ns"] + one["thin_wave_level_ns"] == 10


@pytest.mark.parametrize("nrhs,width,tail,windows", [(1, 2, 63, 1), (1, 2, 64, 2), (1, 60, 20, 1), (1, 65, 20, 1),
                                                     (4, 2, 127, 1), (4, 2, 128, 2), (4, 17, 40, 1)])
def test_a_long_narrow_tail_has_windows_of_its_own(nrhs, width, tail, windows):
    """Levels of at most 64 items that follow wider ones are one wave's work in
    windows of their own if they are 64 or more (128 with several columns)."""
    m = _chain_of_levels([100] * 4 + [width] * tail)
    h = sp.Handle()
    h.analyze(*dev(m))
    b_np = gen.rhs(m, nrhs)
    b = to_dev(b_np)
    h.set_schedule(sp.ORIGINAL, mode=1)
    ref = h.solve(b)
    assert oracle.relerr(ref.cpu().numpy(), oracle.solve(m, b_np)) <= 1e-10
    for wg in (256, 512, 1024):
        h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=wg)
        assert _counts(h, nrhs)["flag_hop_ns"] == windows - 1
        assert torch.equal(h.solve(b), ref)
    h.set_schedule(sp.ORIGINAL, mode=3)
    assert torch.equal(h.solve(b), ref)
    h.check()
