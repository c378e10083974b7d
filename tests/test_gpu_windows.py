"""LDS windows of the thin runs: every width class of the inline records (2, 6
and 10 dependencies a row, overflow records beyond, windows of one level), one
wave and several, one column and several, against the oracle and, bit for bit,
against the wide-level launches (every executor sums a row's products in
ascending position and divides once)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from tests.gpu_util import dev, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")

TOL = 1e-10


def _solve(h, b, nrhs, **sched):
    h.set_schedule(sp.ORIGINAL, **sched)
    x = h.solve(b)
    h.check()
    return x


@pytest.mark.parametrize("draws", [1, 2, 3, 6, 7, 10, 13])
@pytest.mark.parametrize("n,window", [(1, 64), (2, 64), (65, 4), (1000, 64), (4099, 700), (9001, 3000)])
def test_widths(draws, n, window):
    m = gen.window_random(n, 17 * draws + n, window, draws)
    h = sp.Handle()
    h.analyze(*dev(m))
    for nrhs in (1, 3):
        b = gen.rhs(m, nrhs)
        ref = oracle.solve(m, b)
        wide = _solve(h, to_dev(b), nrhs, mode=1)
        assert oracle.relerr(wide.cpu().numpy(), ref) <= TOL
        for wg in (256, 512, 1024):
            assert torch.equal(_solve(h, to_dev(b), nrhs, mode=2, wg_threads=wg), wide), (nrhs, wg)
        assert torch.equal(_solve(h, to_dev(b), nrhs, mode=2, wg_threads=1024, thin_cols=1), wide)
        assert torch.equal(_solve(h, to_dev(b), nrhs, mode=3), wide)


def test_long_rows_keep_their_order():
    # rows beyond the sorted length, with levels that do not follow the columns
    rng = np.random.default_rng(5)
    n = 1400
    a = np.zeros((n, n))
    for i in range(1, n):
        a[i, rng.integers(0, i, size=2)] = rng.uniform(-1, 1, size=2)
    for i in (700, 1399):
        a[i, rng.permutation(i)[:650]] = rng.uniform(-1, 1, size=650)
    a[np.arange(n), np.arange(n)] = 1.0 + np.abs(a).sum(1)
    m = gen.from_dense_lower(a)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = gen.rhs(m, 1)
    ref = oracle.solve(m, b)
    for mode in (0, 1, 2, 3):
        assert oracle.relerr(_solve(h, to_dev(b), 1, mode=mode).cpu().numpy(), ref) <= TOL, mode


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_division_at_the_ends_of_the_range(mode):
    # diagonals whose reciprocal leaves the normal range are divided in full
    d = np.array([2.0 ** -1060, -2.0 ** -1010, 2.0 ** 1015, 3.0, -7.0, 2.0 ** -1000, 2.0 ** 1000, 1e-300])
    b = np.array([2.0 ** -1050, 2.0 ** -1020, 2.0 ** 1010, 1.0, 0.0, 3.0 * 2.0 ** -990, 2.0 ** 990, 5e-299])
    m = gen.from_dense_lower(np.diag(d))
    h = sp.Handle()
    h.analyze(*dev(m))
    x = _solve(h, to_dev(b), 1, mode=mode).cpu().numpy()
    assert np.array_equal(x, b / d)


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("levels", [1, 2])
def test_division_of_small_numbers(mode, levels):
    """Dividends near and below the normal range, zeros of both signs and
    quotients at the ends of the range under ordinary and extreme diagonals,
    alone in a window of one level and behind a dependency of weight 0: the
    quotients are those of one IEEE division, bit for bit."""
    rng = np.random.default_rng(11)
    e = np.concatenate([rng.integers(-1074, -890, 1500), rng.integers(960, 1023, 300), rng.integers(-40, 40, 300)])
    b = np.ldexp(rng.uniform(1, 2, e.size), e) * rng.choice([-1.0, 1.0], e.size)
    d = np.ldexp(rng.uniform(1, 2, e.size), rng.integers(-45, 45, e.size)) * rng.choice([-1.0, 1.0], e.size)
    ends = [(a, q) for a in (0.0, -0.0, 2.0 ** -1074, 2.0 ** -1022, 2.0 ** -900, 2.0 ** -901, 1.0, 9 * 2.0 ** -1074)
            for q in (2.0, -3.0, 6.0, 2.0 ** 119, 2.0 ** 120, 3.0 * 2.0 ** 119, 2.0 ** 1000, 2.0 ** -1000)]
    b = np.concatenate([b, [a for a, _ in ends], [float.fromhex("0x1.e2169b426629cp-1019")]])
    d = np.concatenate([d, [q for _, q in ends], [float.fromhex("0x1.6ee71b15cff4bp+0")]])
    with np.errstate(over="ignore", under="ignore"):
        keep = np.isfinite(b / d)
        b, d = b[keep], d[keep]
        n = b.size
        if levels == 1:
            m = gen.from_dense_lower(np.diag(d))
            want = b / d
        else:  # row n + i reads row i with weight 0
            rp = np.concatenate([np.arange(n), n + 2 * np.arange(n + 1)]).astype(np.int32)
            col = np.concatenate([np.arange(n), np.stack([np.arange(n), n + np.arange(n)], 1).reshape(-1)])
            val = np.concatenate([d, np.stack([np.zeros(n), d], 1).reshape(-1)])
            m = gen.Csr(2 * n, rp, col.astype(np.int32), val)
            x = b / d
            want = np.concatenate([x, (b - 0.0 * x) / d])
            b = np.concatenate([b, b])
    h = sp.Handle()
    h.analyze(*dev(m))
    x = _solve(h, to_dev(b), 1, mode=mode).cpu().numpy()
    bad = np.nonzero(x.view(np.int64) != want.view(np.int64))[0]
    assert bad.size == 0, (bad.size, b[bad[0]].hex(), d[bad[0] % n].hex(), x[bad[0]].hex(), want[bad[0]].hex())


@pytest.mark.parametrize("mode", [1, 2, 3])
def test_infinities_stay_infinities(mode):
    m = gen.from_dense_lower(np.array([[0.5, 0, 0], [0, 2.0, 0], [1.0, 0, 4.0]]))
    h = sp.Handle()
    h.analyze(*dev(m))
    h.set_schedule(sp.ORIGINAL, mode=mode)
    x = h.solve(to_dev(np.array([1.7e308, np.inf, 1.0]))).cpu().numpy()
    assert x[0] == np.inf and x[1] == np.inf and x[2] == -np.inf
    with pytest.raises(sp.SptrsvError):
        h.check()


@pytest.mark.parametrize("nrhs,thin_cols", [(1, 0), (2, 0), (3, 1), (8, 1), (9, 1), (17, 1), (6, 2)])
def test_spread_windows_repeat(nrhs, thin_cols):
    """Runs of many windows spread over workgroups: column groups below, at and
    above the number of XCDs; repeated, by rows and in graph replays with new
    right-hand sides in between (stale values of the solve before must not pass
    for finished ones)."""
    m = gen.stencil2d_chain(70, 900, 3)
    h = sp.Handle()
    h.analyze(*dev(m))
    h.set_schedule(sp.ORIGINAL, mode=1)
    b1, b2 = to_dev(gen.rhs(m, nrhs)), to_dev(gen.rhs(m, nrhs)[:, ::-1])
    ref1, ref2 = h.solve(b1).clone(), h.solve(b2).clone()
    h.set_schedule(sp.ORIGINAL, mode=2, wg_threads=256, thin_cols=thin_cols)
    for _ in range(3):
        assert torch.equal(h.solve(b1), ref1)
        assert torch.equal(h.solve(b2), ref2)
        if nrhs > 1:
            assert torch.equal(h.solve_rows(b1.t().contiguous()).t(), ref1)
            assert torch.equal(h.solve_rows(b2.t().contiguous()).t(), ref2)
    b, x = b1.clone(), torch.empty_like(b1)
    with torch.cuda.stream(torch.cuda.Stream()):
        g = h.graph_create(b, x)
        for src, ref in ((b1, ref1), (b2, ref2), (b1, ref1)):
            b.copy_(src)
            h.graph_launch(g)
            torch.cuda.synchronize()
            assert torch.equal(x, ref)
    h.check()


@pytest.mark.parametrize("draws,window", [(3, 40), (5, 64), (9, 500), (12, 4000)])
@pytest.mark.parametrize("nrhs", [1, 2, 9])
def test_sync_free_in_windows_and_row_by_row(draws, window, nrhs):
    """Mode 3 below and above the line between its two forms gives the bits of
    the wide-level launches, by columns, by rows and without allocation."""
    m = gen.window_random(30000, draws, window, draws)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    ref = _solve(h, b, nrhs, mode=1)
    for grid in (0, 1, 128, 2048):
        assert torch.equal(_solve(h, b, nrhs, mode=3, wide_grid=grid), ref)
    h.prepare(sp.ORIGINAL, nrhs)
    x = torch.empty_like(b)
    assert torch.equal(h.solve(b, x=x, noalloc=True), ref)
    if nrhs > 1:
        assert torch.equal(h.solve_rows(b.t().contiguous()).t(), ref)
    h.check()


@pytest.mark.parametrize("nrhs", [5, 24, 40, 63, 65, 130])
@pytest.mark.parametrize("wg", [256, 512, 1024])
def test_columns_of_a_row_in_two_waves(nrhs, wg):
    """All columns in one workgroup: a row's items straddle waves, and a level's
    last row is repeated by lanes that must not write it."""
    m = gen.window_random(3001, nrhs, 24, 3)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, nrhs))
    ref = _solve(h, b, nrhs, mode=1)
    for _ in range(4):
        assert torch.equal(_solve(h, b, nrhs, mode=2, wg_threads=wg), ref)


@pytest.mark.parametrize("nrhs,width,wide", [(1, 5000, False), (1, 5200, True), (2, 4000, False), (2, 4175, True),
                                             (8, 1800, False), (8, 1900, True)])
def test_widest_levels_of_a_thin_run(nrhs, width, wide):
    """A thin run takes levels up to 24 bytes of LDS a row beside x, wider ones
    are launches: 26 levels of 4,175 rows, two columns, 225 us against 902 in
    windows of their own."""
    rng = np.random.default_rng(width)
    i = np.arange(width, 3 * width)
    r = np.concatenate([np.arange(3 * width), i])
    c = np.concatenate([np.arange(3 * width), i - i % width - width + rng.integers(0, width, i.size)])
    val = np.concatenate([1.0 + rng.random(3 * width), rng.uniform(-1, 1, i.size)])
    o = np.lexsort((c, r))
    m = gen.Csr(3 * width, np.searchsorted(r[o], np.arange(3 * width + 1)).astype(np.int32), c[o].astype(np.int32),
                val[o])
    h = sp.Handle()
    h.analyze(*dev(m))
    b_np = gen.rhs(m, nrhs)
    b = to_dev(b_np)
    ref = _solve(h, b, nrhs, mode=1)
    assert oracle.relerr(ref.cpu().numpy(), oracle.solve(m, b_np)) <= TOL
    assert torch.equal(_solve(h, b, nrhs, mode=2), ref)
    h.profile_start()
    h.solve(b)
    n = {k: v["launches"] for k, v in h.profile_stop().items()}
    assert (n["wide_level"], n["thin_run"]) == ((3, 0) if wide else (0, 1))
