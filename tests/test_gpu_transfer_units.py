"""APIC, PIC and quadratic P2G sums in units of their own block: a light, slow, soft body
beside a heavy, fast, stiff one, whose contributions to the grid are 5e8 times larger.
Every quantity of each body is normalised by that body's own largest value.  The units are
2^-39 of the largest contribution of a pass over at most 512 of the block's particles, so
that they add less than 1e-8 to a node of the light body; the tolerance is that of the FP32
step."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state
from test_gpu_transfer_blocks import KINDS, _oracle_step

pytestmark = pytest.mark.gpu


def _pair():
    kw = dict(n_cells=(32, 32, 32), model=scenes.FIXED_COROTATED, dt=1e-5, dx=1.0 / 32, B_scale=0.0)
    light = scenes.random_blob(71, lo_cells=(4.3, 5.2, 4.6), ext_cells=(6, 5, 7), rho=1.0, E=10.0, v_scale=1e-3, F_scale=1e-3,
                               **kw)
    heavy = scenes.random_blob(72, lo_cells=(20.3, 19.4, 18.6), ext_cells=(5, 6, 5), rho=1e4, E=1e7, v_scale=50.0,
                               F_scale=0.01, **kw)
    n = light.n
    light.materials += heavy.materials
    light.mat[:] = 0
    heavy.mat[:] = 1
    for name in ("x", "v", "B", "F", "mat"):
        setattr(light, name, np.concatenate([getattr(light, name), getattr(heavy, name)]))
    return light, n


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("steps", [1, 3])
def test_each_body_in_its_own_units(kind, steps):
    sc, n = _pair()
    run = GpuRun(sc, **KINDS[kind])
    got = run.steps(sc.dt, steps)
    assert got["status"] == 0
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F, mat=sc.mat))
    for _ in range(steps):
        g = _oracle_step(kind, sc, st, sc.dt)
    m, vt = run.grids()
    if kind == "quadratic":
        m, vt = m[0], vt[0]
    H = st.F - np.eye(3)
    for body, part, half in (("light", slice(0, n), slice(0, 16)), ("heavy", slice(n, None), slice(16, None))):
        errs = dict(m=nerr(m[..., half, :, :], g["m"][..., half, :, :]),
                    p=nerr((m[..., None].astype(np.float64) * vt)[..., half, :, :, :],
                           (g["m"][..., None] * g["v"])[..., half, :, :, :]),
                    v=nerr(got["v"][part], st.v[part]), H=nerr(got["H"][part], H[part]))
        log("%s %d steps, %s body: %s" % (kind, steps, body, " ".join("%s=%.2e" % e for e in errs.items())))
        for k, e in errs.items():
            assert e <= TOL, (body, k)
    run.close()


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("n", [200, 300, 513, 1500, 2048])
def test_unit_grows_within_a_block(kind, n):
    """One block, whose particles in the upper halves of the cells along z (the later rounds of a pass) move 1e6 times
    faster: the sums of the first rounds are taken over into the larger unit."""
    sc = scenes.random_blob(73, n_cells=(16, 16, 16), model=scenes.FIXED_COROTATED, dt=1e-5, E=1e4, B_scale=0.0, F_scale=1e-3)
    rng = np.random.default_rng(n)
    X = 4.0 + 3.7 * rng.random((n, 3))
    sc.x = (X * sc.dx).astype(np.float32)
    up = ((X[:, 2] + 0.25) % 1.0) >= 0.5
    sc.v = (np.where(up, 10.0, 1e-5)[:, None] * (1.0 + rng.random((n, 3)))).astype(np.float32)
    sc.B = np.zeros((n, 3, 3), np.float32)
    sc.F = (np.eye(3)[None] + 1e-3 * rng.standard_normal((n, 3, 3))).astype(np.float32)
    sc.mat = np.zeros(n, np.uint8)
    run = GpuRun(sc, **KINDS[kind])
    got = run.phase_step(sc.dt)
    assert got["status"] == 0
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F))
    g = _oracle_step(kind, sc, st, sc.dt)
    q = 0 if kind == "quadratic" else slice(None)
    errs = dict(m=nerr(got["m"][q], g["m"]), p=nerr(got["p"][q], g["p"]), v=nerr(got["v"], st.v), F=nerr(got["F"], st.F))
    log("%s %d particles: %s" % (kind, n, " ".join("%s=%.2e" % e for e in errs.items())))
    for k, e in errs.items():
        assert e <= TOL, k
    run.close()
