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
