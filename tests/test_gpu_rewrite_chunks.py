"""The decision scan of the rewriting takes its candidates eight at a time from
as many levels as that needs, and counts the rows a new target keeps 64 at a
time: levels just below, at and above those sizes, against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from tests.gpu_util import dev
from tests.test_gpu_rewrite import compare

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")

SIZES = {
    "ones": [1] * 40,
    "around_a_chunk": [3, 7, 1, 8, 1, 9, 1, 1, 16, 17, 2, 7, 8, 9, 15],
    "around_a_wave": [5, 63, 1, 64, 2, 65, 1, 128, 129, 1],
    "one_of_one": [1],
}


def _leveled(sizes, seed):
    """Row in level k > 0: one entry of level k - 1, another of any level before."""
    rng = np.random.default_rng(seed)
    n = sum(sizes)
    a = np.zeros((n, n))
    at = 0
    for k, size in enumerate(sizes):
        for i in range(at, at + size):
            if k:
                a[i, rng.integers(at - sizes[k - 1], at)] = rng.uniform(0.1, 1.0)
                a[i, rng.integers(0, at)] = rng.uniform(0.1, 1.0)
        at += size
    a[np.arange(n), np.arange(n)] = 1.0 + np.abs(a).sum(1)
    return gen.from_dense_lower(a)


# a matrix of one level is answered without a scan and reports no target step,
# where the oracle counts its only level as one
ONE = pytest.param("one_of_one", marks=pytest.mark.xfail(strict=True, reason="target_steps of one level: 0 here, 1 in the oracle"))


@pytest.mark.parametrize("sizes", [k for k in SIZES if k != "one_of_one"] + [ONE])
@pytest.mark.parametrize("opt", [(0, 4, 0.0, 0), (0, 12, 4.0, 0), (0, 70, 2.0, 3), (1, 0.0, 0.0, 0), (1, 60.0, 3.0, 0)])
def test_levels_around_the_chunk(sizes, opt):
    m = _leveled(SIZES[sizes], len(SIZES[sizes]))
    lv = oracle.levels(m)
    h = sp.Handle()
    h.analyze(*dev(m))
    st = h.rewrite(*opt)
    compare(m, h, st, oracle.rewrite(m, *opt, None, lv), lv, nrhs=(1,))
