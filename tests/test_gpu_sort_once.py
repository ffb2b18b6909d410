"""Lattices of up to 12,288 virtual blocks sort in one launch between the steps of a
context.  After mpm_invalidate a step takes the separate launches instead: in deterministic
mode both must give the same bits, for particles that change cells and blocks on every step,
with a sort of keys alone in between."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun

pytestmark = pytest.mark.gpu


def _scene(n_cells):
    sc = scenes.random_blob(31, n_cells=n_cells, lo_cells=(3.3, 4.6, 3.1), ext_cells=(9, 6, 8), F_scale=0.02, dt=1e-4, dx=1.0 / 64,
                            v_scale=0.3)
    # up to a third of a cell per step along each axis
    sc.v += (0.25 * sc.dx / sc.dt * np.array([1.0, -0.3, 0.7])).astype(np.float32)
    return sc


@pytest.mark.parametrize("n_cells", [(24, 24, 24), (32, 32, 32), (60, 64, 72), (62, 92, 124), (62, 92, 128)])
def test_one_launch_equals_separate_launches(n_cells):
    import torch
    sc = _scene(n_cells)
    once, apart = GpuRun(sc, deterministic=True), GpuRun(sc, deterministic=True)
    keys = torch.empty(sc.n, dtype=torch.int32, device="cuda")
    for k in range(8):
        a = once.steps(sc.dt, 1 + k % 2)
        for _ in range(1 + k % 2):
            apart.ck.check(apart.ck.mpm_invalidate(apart.ctx.h))
            b = apart.steps(sc.dt, 1)
        if k == 4:   # keys alone: the next step of either context takes the separate launches
            once.ck.check(once.ck.mpm_sort_keys(once.ctx.h, once.parts.c, keys.data_ptr(), None, once.stream))
        assert a["status"] == 0 and b["status"] == 0
        for name in ("x", "v", "B", "F"):
            assert np.array_equal(a[name], b[name]), (k, name)
    assert np.array_equal(once.parts.read()["id"], apart.parts.read()["id"])
    once.close()
    apart.close()

