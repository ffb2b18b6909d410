"""G2P shares a particle block among 4, 2 or 1 workgroups by the number of particle
blocks (lines at 384 and 1,280 blocks), and inside mpm_step forms the grid update as it
gathers a block's velocities (a separate form for tiles that touch the sticky walls).
Ragged bodies on either side of the lines, resting on the floor's wall band and under
gravity, against the FP64 checker's own steps."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state, oracle_step

pytestmark = pytest.mark.gpu


def _ragged(ext, n_cells, model, seed=11):
    """A body of `ext` cells on the floor band with a third of its particles missing, one
    block holding only a few and one holding more than a pass of 512 can take."""
    sc = scenes.random_blob(seed, n_cells=n_cells, lo_cells=(3.25, 2.25, 3.5), ext_cells=ext, model=model,
                            gravity=(0.0, -9.8, 0.0), bc_band=2, dt=1e-4, E=3.5e4, rho=1600.0, v_scale=0.3,
                            B_scale=0.3, F_scale=0.01)
    rng = np.random.default_rng(seed)
    keep = rng.random(sc.n) < 0.67
    block = np.floor(sc.x.astype(np.float64) / sc.dx + 0.25).astype(np.int64) >> 2
    thin = (block == block[0]).all(axis=1)
    keep &= ~thin
    keep[np.flatnonzero(thin)[:3]] = True
    for name in ("x", "v", "B", "F", "mat"):
        setattr(sc, name, getattr(sc, name)[keep])
    # crowd a block in the middle: 900 more particles at random places inside it
    mid = (np.floor(sc.x[sc.n // 2].astype(np.float64) / sc.dx + 0.25).astype(np.int64) >> 2)
    lo = np.maximum(4 * mid - 0.24, 2.1)   # inside the block and above the floor band
    x = ((lo + (4 * mid + 3.74 - lo) * rng.random((900, 3))) * sc.dx).astype(np.float32)
    pick = rng.integers(0, sc.n, 900)
    for name in ("v", "B", "F", "mat"):
        a = getattr(sc, name)
        setattr(sc, name, np.concatenate([a, a[pick]]))
    sc.x = np.concatenate([sc.x, x])
    return sc


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("ext,n_cells,lo,hi", [((4, 3, 5), (16, 16, 16), 1, 384), ((23, 22, 21), (64, 64, 64), 300, 384),
                                               ((30, 29, 28), (64, 64, 64), 385, 1280),
                                               ((44, 43, 45), (64, 64, 64), 1281, 4000)])
def test_split_blocks_match_checker(ext, n_cells, lo, hi, deterministic):
    sc = _ragged(ext, n_cells, scenes.DRUCKER_PRAGER if ext[0] % 2 else scenes.FIXED_COROTATED)
    run = GpuRun(sc, deterministic=deterministic)
    got = run.steps(sc.dt, 3)
    assert got["status"] == 0
    s, stats = run.ck.mpm_get_stats(run.ctx.h, run.stream)
    assert s == 0 and lo <= stats.n_particle_blocks <= hi
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F))
    for _ in range(3):
        _, g = oracle_step(sc, st, sc.dt)
    m, vt = run.grids()   # the last step leaves its updated grid
    assert nerr(m, g["m"]) <= TOL
    assert nerr(m[..., None].astype(np.float64) * vt, g["m"][..., None] * g["v"]) <= TOL
    for name in ("x", "v", "F"):
        e = nerr(got[name], getattr(st, name))
        log("%d blocks: %s %.2e" % (stats.n_particle_blocks, name, e))
        assert e <= TOL, name
    run.close()
