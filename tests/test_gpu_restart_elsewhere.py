"""A context taken to a body somewhere else (mpm_invalidate): the grid blocks that the last
step stamped for the old body are not allocated again beside the new one's, so that a pool
that fits each body is enough.  In every form of the step, on lattices that sort in one
launch and in several.  Against the FP64 oracle."""
import numpy as np
import pytest

from gpu_util import GpuRun
from test_gpu_crowded_block import FORMS, _bodies, _oracle, _match

pytestmark = pytest.mark.gpu


def _halves(n_cells):
    out = []
    for half in range(2):
        sc = _bodies(n_cells)
        n = sc.n // 2
        for name in ("x", "v", "B", "F", "mat"):
            setattr(sc, name, getattr(sc, name)[half * n:(half + 1) * n].copy())
        out.append(sc)
    return out


def _grid_blocks(sc):
    """Blocks within one block of a block that holds particles, inside the lattice."""
    b = np.unique(np.floor(sc.x.astype(np.float64) / sc.dx + 0.25).astype(np.int64) >> 2, axis=0)
    offs = np.stack(np.meshgrid(*[[-1, 0, 1]] * 3, indexing="ij"), -1).reshape(-1, 3)
    near = np.unique((b[:, None] + offs[None]).reshape(-1, 3), axis=0)
    top = np.array([c // 4 for c in sc.n_cells])
    return int(((near >= 0) & (near <= top)).all(axis=1).sum())


@pytest.mark.parametrize("n_cells", [(32, 32, 32), (64, 92, 124)])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_pool_that_fits_each_body(form, n_cells):
    first, second = _halves(n_cells)
    a, b = _grid_blocks(first), _grid_blocks(second)
    room = max(a, b) + 12   # particles may enter a few more blocks in these steps
    assert room < a + b
    run = GpuRun(first, max_blocks=room, **FORMS[form])
    ck, p = run.ck, run.parts
    assert run.steps(first.dt, 3)["status"] == 0
    for sc in (second, first):
        p.load(sc.x, sc.v, sc.B, sc.F)
        ck.check(ck.mpm_invalidate(run.ctx.h))
        got = run.steps(sc.dt, 3)
        assert got["status"] == 0
        _match(got, _oracle(form, sc, 3), "%s, from elsewhere" % form)
        s, stats = ck.mpm_get_stats(run.ctx.h, run.stream)
        assert s == 0 and stats.n_grid_blocks <= room
    run.close()
