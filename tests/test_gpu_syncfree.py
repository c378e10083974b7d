"""The two forms of the synchronisation-free executor (schedule mode 3): LDS
windows where levels are narrow, a wait per row elsewhere. Each case says on the
host which form it takes, the launch profile confirms it, and both forms give the
oracle's solution and the bits of the wide-level launches (every row of at most
512 off-diagonals sums its products in ascending position and divides once)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from tests.gpu_util import dev, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")

TOL = 1e-10
LINE = 1600  # off-diagonals a level on average


def _layered(widths, seed, draws=4):
    """Levels of the given widths; a row reads up to `draws` rows of the level before."""
    rng = np.random.default_rng(seed)
    first = np.concatenate([[0], np.cumsum(widths)])
    n = int(first[-1])
    key = [np.arange(n) * n + np.arange(n)]
    for l in range(1, len(widths)):
        rows = np.arange(first[l], first[l + 1])
        key += [rows * n + rng.integers(first[l - 1], first[l], rows.size) for _ in range(draws)]
    key = np.unique(np.concatenate(key))
    r, c = key // n, key % n
    val = rng.uniform(-1, 1, key.size) / (draws + 1)
    val[r == c] = 1.0 + rng.random(n)
    return gen.Csr(n, np.searchsorted(r, np.arange(n + 1)).astype(np.int32), c.astype(np.int32), val)


CASES = {
    # too many off-diagonals a level
    "dense_levels": lambda: _layered([1000] * 30, 1),
    "random_wide": lambda: gen.window_random(30000, 12, 20000, 6),
    # a level of 8,000 rows fits no window
    "wide_first": lambda: _layered([8000] + [40, 3, 70] * 60, 2),
    # below the line, narrow levels: windows
    "narrow": lambda: _layered([30, 5, 60] * 100, 3),
}


def _row_by_row(m):
    lv = oracle.levels(m)
    widths = np.diff(lv.level_ptr)
    return (m.nnz - m.n) > LINE * widths.size or widths.max() > 6783


def _form(h, run):
    h.profile_start()
    run()
    p = h.profile_stop()
    return {k: v["launches"] for k, v in p.items()}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("nrhs", [1, 2, 9])
def test_forms(case, nrhs):
    m = CASES[case]()
    assert _row_by_row(m) == (case != "narrow")
    h = sp.Handle()
    h.analyze(*dev(m))
    b_np = gen.rhs(m, nrhs)
    b = to_dev(b_np)
    h.set_schedule(sp.ORIGINAL, mode=1)
    ref = h.solve(b)
    assert oracle.relerr(ref.cpu().numpy(), oracle.solve(m, b_np)) <= TOL
    for grid in (0, 1, 3, 128, 2048):
        h.set_schedule(sp.ORIGINAL, mode=3, wide_grid=grid)
        assert torch.equal(h.solve(b), ref), grid
    h.check()
    n = _form(h, lambda: h.solve(b))
    assert (n["wide_level"], n["thin_run"]) == ((0, 1) if case == "narrow" else (1, 0))
    # by rows, without allocation, and graph replays with new right-hand sides between them
    if nrhs > 1:
        assert torch.equal(h.solve_rows(b.t().contiguous()).t(), ref)
    h.prepare(sp.ORIGINAL, nrhs)
    x = torch.empty_like(b)
    assert torch.equal(h.solve(b, x=x, noalloc=True), ref)
    src = b.clone()
    with torch.cuda.stream(torch.cuda.Stream()):
        g = h.graph_create(src, x)
        for scale in (1.0, -2.0, 1.0):
            src.copy_(b * scale)
            h.graph_launch(g)
            torch.cuda.synchronize()
            assert torch.equal(x, ref * scale)
    h.check()


def test_rewritten_row_by_row():
    m = gen.window_random(30000, 12, 20000, 6)
    h = sp.Handle()
    h.analyze(*dev(m))
    st = h.rewrite(sp.THIN_ROWS, 32, 4.0, 0)
    assert st["rows_rewritten"] > 0 and st["nnz_Lp"] - m.n > LINE * st["nlev_after"]
    for nrhs in (1, 3):
        b = gen.rhs(m, nrhs)
        h.set_schedule(sp.REWRITTEN, mode=3, wide_grid=256)
        x = h.solve(to_dev(b) if nrhs > 1 else to_dev(b[0]), sp.REWRITTEN)
        h.check()
        assert oracle.relerr(x.cpu().numpy().reshape(nrhs, -1), oracle.solve(m, b)) <= TOL


@pytest.mark.parametrize("nrhs,windows", [(1, True), (2, True), (8, False), (16, False), (32, False)])
def test_several_columns_need_more_levels_a_window(nrhs, windows):
    """A mesh-like matrix below the line whose windows hold 12 levels: windows
    for one or two columns, a wait per row for more (32 columns took 1,153 us in
    windows against 678)."""
    m = gen.torso2_like(1, 60000)
    assert not _row_by_row(m)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    h.set_schedule(sp.ORIGINAL, mode=1)
    ref = h.solve(b)
    h.set_schedule(sp.ORIGINAL, mode=3, wide_grid=256)
    assert torch.equal(h.solve(b), ref)
    n = _form(h, lambda: h.solve(b))
    h.check()
    assert (n["wide_level"], n["thin_run"]) == ((0, 1) if windows else (1, 0))


@pytest.mark.parametrize("nrhs,windows", [(2, True), (8, True), (32, False)])
def test_windows_that_read_little_from_outside(nrhs, windows):
    """Six levels of 256 rows a window, which read only the level before them:
    about 210 outside dependencies a level, so windows pay for 8 columns (431 us
    against 1,082 on 400 levels)."""
    m = _layered([256] * 120, 4, 5)
    assert not _row_by_row(m)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    h.set_schedule(sp.ORIGINAL, mode=1)
    ref = h.solve(b)
    h.set_schedule(sp.ORIGINAL, mode=3)
    assert torch.equal(h.solve(b), ref)
    n = _form(h, lambda: h.solve(b))
    h.check()
    assert (n["wide_level"], n["thin_run"]) == ((0, 1) if windows else (1, 0))


@pytest.mark.parametrize("nrhs", [1, 4])
@pytest.mark.parametrize("width,windows", [(2400, True), (4200, False)])
def test_levels_that_fill_a_window_alone(width, windows, nrhs):
    """Most rows in levels of 4,200 rows are solved row by row, also below the
    line (one column: 780 us in windows against 465 at 6,500 rows); the levels
    between them are narrow."""
    m = _layered(([width] + [2] * 60) * 6, 8, 2)
    assert not _row_by_row(m)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    h.set_schedule(sp.ORIGINAL, mode=1)
    ref = h.solve(b)
    h.set_schedule(sp.ORIGINAL, mode=3)
    assert torch.equal(h.solve(b), ref)
    n = _form(h, lambda: h.solve(b))
    h.check()
    assert (n["wide_level"], n["thin_run"]) == ((0, 1) if windows else (1, 0))


def _solve_ns(h, b):
    x = torch.empty_like(b)
    for _ in range(3):
        h.solve(b, x=x)
    t = []
    for _ in range(7):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        h.solve(b, x=x)
        e1.record()
        torch.cuda.synchronize()
        t.append(e0.elapsed_time(e1) * 1e6)
    return float(np.median(t))


@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("mk", [lambda: gen.window_random(30000, 5, 64, 5), lambda: gen.bidiagonal(20000, 3),
                                lambda: _layered([1000] * 60, 1)])
def test_finish_times_are_the_executors(mk, nrhs):
    """The last level finishes about when a mode-3 solve does, in either form (a
    narrow matrix takes 0.6 ms in windows and 3.9 ms row by row). The stamps
    cost something and a solve has two transposes and a fill besides, so the
    last finish may be from 0.4 to 2 solve times."""
    m = mk()
    h = sp.Handle()
    nlev = h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    h.set_schedule(sp.ORIGINAL, mode=3)
    solve = _solve_ns(h, b)
    best = np.inf
    for _ in range(3):
        t = h.level_finish_times(b).cpu().numpy()
        h.check()
        assert t.shape == (nlev,) and np.all(np.isfinite(t)) and np.all(t >= 0) and t[0] < t[-1]
        best = min(best, float(t.max()))
    assert 0.4 * solve <= best <= 2.0 * solve, (best, solve)


def test_finish_times_leave_the_plan():
    """Graphs captured before (window tables and images of another schedule) and
    the next solves are not touched."""
    m = gen.window_random(9000, 5, 64, 5)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, 2))
    x = torch.empty_like(b)
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=256)
    ref = h.solve(b).clone()
    h.prepare(sp.ORIGINAL, 2)
    with torch.cuda.stream(torch.cuda.Stream()):
        g = h.graph_create(b, x)
        for _ in range(3):
            h.level_finish_times(b)
            x.zero_()
            h.graph_launch(g)
            torch.cuda.synchronize()
            assert torch.equal(x, ref)
            assert torch.equal(h.solve(b, noalloc=True, x=torch.empty_like(b)), ref)
    h.check()
