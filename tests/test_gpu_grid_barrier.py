"""The device-wide barrier of the persistent wide run, at grids below, at and
above its number of release words and the size of an arrival group; solves
repeat on the barrier block that the one before left, eagerly and in a graph,
and agree bit for bit with a launch per level."""
import pytest
import torch

import gen
from tests.gpu_util import dev, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_2206_05843_amd")


@pytest.mark.parametrize("grid", [1, 2, 3, 4, 5, 31, 32, 33, 64, 65, 1280, 4096])
def test_persistent_run_repeats(grid):
    m = gen.window_random(6000, 11, 900, 4)
    h = sp.Handle()
    h.analyze(*dev(m))
    b = to_dev(gen.rhs(m, 3))
    h.set_schedule(mode=1)
    ref = h.solve(b)
    h.set_schedule(mode=1, wide_grid=grid, wide_threads=64)
    for _ in range(4):
        assert torch.equal(h.solve(b), ref)
        h.check()
    x = torch.empty_like(ref)
    with torch.cuda.stream(torch.cuda.Stream()):
        g = h.graph_create(b, x)
        for _ in range(3):
            x.fill_(float("nan"))
            h.graph_launch(g)
            torch.cuda.synchronize()
            assert torch.equal(x, ref)
            assert torch.equal(h.solve(b), ref)
    h.check()
