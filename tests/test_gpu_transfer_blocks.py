"""The APIC, PIC and quadratic kernels on the block loops that the MLS kernels run: kept
block orders and neighbourhoods from step to step, G2P's sharing of blocks at its lines
(384 and 1,280 blocks) with the grid update folded into the gather, and the step-global
P2G unit with its float-atomic path above the bound.  Each against the FP64 oracle's same
transfer."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state
from test_gpu_split import _ragged

pytestmark = pytest.mark.gpu

KINDS = {"apic": dict(transfer=1), "pic": dict(transfer=2), "quadratic": dict(quadratic=True)}


def _oracle_step(kind, sc, st, dt):
    if kind == "quadratic":
        status, _, g = oracle.step_quadratic(oracle.scene_config(sc), oracle.scene_materials(sc), st, dt, grids=True)
    else:
        status, _, g = oracle.step(oracle.scene_config(sc, KINDS[kind]["transfer"]), oracle.scene_materials(sc), st, dt,
                                   grids=True)
    assert status == 0
    return g


def _compare(kind, tag, got, m, st, g):
    em = nerr(m[0] if kind == "quadratic" else m, g["m"])
    errs = {k: nerr(got[k], getattr(st, k)) for k in ("x", "v", "F")}
    log("%s %s: grid m %.2e %s" % (kind, tag, em, " ".join("%s=%.2e" % kv for kv in errs.items())))
    assert em <= TOL
    for k, e in errs.items():
        assert e <= TOL, k


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("ext,n_cells,lo,hi", [((4, 3, 5), (16, 16, 16), 1, 384), ((30, 29, 28), (64, 64, 64), 385, 1280),
                                               ((44, 43, 45), (64, 64, 64), 1281, 4000)])
def test_step_sequence_matches_oracle(kind, ext, n_cells, lo, hi):
    """Three steps in one call (orders kept, update folded), then three more: the second
    call starts from the first one's state and kept orders."""
    sc = _ragged(ext, n_cells, scenes.DRUCKER_PRAGER if ext[0] % 2 else scenes.FIXED_COROTATED)
    run = GpuRun(sc, **KINDS[kind])
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F))
    for call in range(2 if hi <= 384 else 1):
        got = run.steps(sc.dt, 3)
        assert got["status"] == 0
        s, stats = run.ck.mpm_get_stats(run.ctx.h, run.stream)
        assert s == 0 and lo <= stats.n_particle_blocks <= hi
        for _ in range(3):
            g = _oracle_step(kind, sc, st, sc.dt)
        _compare(kind, "%d blocks, call %d" % (stats.n_particle_blocks, call), got, run.grids()[0], st, g)
    run.close()


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("scale", [1.0, 200.0])
def test_p2g_above_the_bound(kind, scale):
    """Velocities of some particles scaled in place after a step formed the bound: at 200
    those particles go around the tile, straight into the pool."""
    import torch
    sc = scenes.random_blob(7, model=scenes.FIXED_COROTATED, n_cells=(16, 16, 16), lo_cells=(5.0, 5.5, 4.5),
                            ext_cells=(5, 4, 6), F_scale=0.03, E=1e5, v_scale=0.5)
    run = GpuRun(sc, **KINDS[kind])
    dt = 1e-4
    assert run.steps(dt, 1)["status"] == 0
    cur = run.parts.current
    pick = torch.arange(0, run.parts.n, 37, device="cuda")
    run.parts.state[cur, 3:6, pick] *= scale
    torch.cuda.synchronize()
    before = run.parts.read_by_id()
    got = run.phase_step(dt)
    assert got["status"] == 0
    st = oracle_state(before)
    g = _oracle_step(kind, sc, st, dt)
    q = 0 if kind == "quadratic" else slice(None)
    assert nerr(got["p"][q], g["p"]) <= TOL
    _compare(kind, "in-place velocity x%g" % scale, got, got["m"], st, g)
    run.close()
