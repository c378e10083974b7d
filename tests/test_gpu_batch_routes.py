"""Routes of a batched solve: one column a group when there are few tasks, groups
of four otherwise, and matrices that leave the persistent queue because their
levels are wide. Every route gives the oracle's solution and the bits of the
per-matrix solves."""
import numpy as np
import pytest
import torch

import gen
import oracle
from tests.gpu_util import dev, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")

TOL = 1e-10


def _layered(width, levels, seed, draws=4):
    """`levels` levels of `width` rows, each row reading up to `draws` rows of the level before."""
    rng = np.random.default_rng(seed)
    n = width * levels
    rows = np.arange(width, n)
    cols = [(rows // width - 1) * width + rng.integers(0, width, rows.size) for _ in range(draws)]
    key = np.unique(np.concatenate([rows * n + c for c in cols] + [np.arange(n) * n + np.arange(n)]))
    r, c = key // n, key % n
    val = rng.uniform(-1, 1, key.size) / (draws + 1)
    val[r == c] = 1.0 + rng.random(n)
    return gen.Csr(n, np.searchsorted(r, np.arange(n + 1)).astype(np.int32), c.astype(np.int32), val)


def _batch(mats):
    h = sp.Handle()
    h.batch_analyze([m.n for m in mats], to_dev(np.concatenate([m.row_ptr for m in mats]).astype(np.int32)),
                    to_dev(np.concatenate([m.col for m in mats]).astype(np.int32)),
                    to_dev(np.concatenate([m.val for m in mats])))
    return h


def _check(mats, nrhs, **sched):
    h = _batch(mats)
    if sched:
        h.set_schedule(sp.BATCH, mode=2, **sched)
    b = np.concatenate([gen.rhs(m, nrhs).reshape(-1) for m in mats])
    bd = to_dev(b)
    x, x2, x3 = (torch.zeros_like(bd) for _ in range(3))
    h.batch_solve(bd, x, nrhs)
    h.batch_solve(bd, x2, nrhs, looped=True)
    h.batch_solve(bd, x3, nrhs)
    h.check()
    assert torch.equal(x, x2) and torch.equal(x, x3)
    xs, off = x.cpu().numpy(), 0
    for m in mats:
        bm = b[off * nrhs:(off + m.n) * nrhs].reshape(nrhs, m.n)
        assert oracle.relerr(xs[off * nrhs:(off + m.n) * nrhs].reshape(nrhs, m.n), oracle.solve(m, bm)) <= TOL
        off += m.n


@pytest.mark.parametrize("nrhs", [1, 3, 4, 5, 16])
@pytest.mark.parametrize("widths", [(3000,), (600, 20), (7000, 300, 5), (1700,) * 6, (3400, 3400, 8, 8, 8)])
def test_wide_levels(widths, nrhs):
    _check([_layered(w, 12, 7 * i + w) for i, w in enumerate(widths)], nrhs)


@pytest.mark.parametrize("nrhs", [4, 5, 7, 13, 17])
@pytest.mark.parametrize("wg", [256, 512, 1024])
def test_groups_of_four(nrhs, wg):
    """More columns of matrices than CUs: the last group overlaps where four does
    not divide."""
    mats = [gen.window_random(60 + 7 * i, i, 16, 4) for i in range(66)] + [_layered(900, 4, 1)]
    _check(mats, nrhs, wg_threads=wg)


def _ms(f, reps=5):
    for _ in range(3):
        f()
    t = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        f()
        e1.record()
        torch.cuda.synchronize()
        t.append(e0.elapsed_time(e1))
    return float(np.median(t))


@pytest.mark.parametrize("others", [0, 300])
def test_a_matrix_of_wide_levels_uses_the_device(others):
    """40 levels of 3,000 rows take about 0.17 ms as launches and 2 ms in one
    workgroup per group of four columns: a batch that holds such a matrix may
    not take 4 times as long as the matrix and the rest solved apart."""
    nrhs = 4
    wide, small = _layered(3000, 40, 1), [_layered(8, 50, i) for i in range(others)]
    h = sp.Handle()
    h.analyze(*dev(wide))
    h.set_schedule(sp.ORIGINAL, mode=1)
    b = to_dev(gen.rhs(wide, nrhs))
    x = torch.empty_like(b)
    apart = _ms(lambda: h.solve(b, x=x))

    def batch_ms(mats):
        hb = _batch(mats)
        bb = to_dev(np.concatenate([gen.rhs(m, nrhs).reshape(-1) for m in mats]))
        xb = torch.empty_like(bb)
        t = _ms(lambda: hb.batch_solve(bb, xb, nrhs))
        hb.check()
        return t

    if small:
        apart += batch_ms(small)
    assert batch_ms([wide] + small) <= 4 * apart
