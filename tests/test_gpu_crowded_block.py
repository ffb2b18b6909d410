"""A block holding more particles than its capacity (2,048) among ordinary ones, over several
steps of one call: its range of sorted positions is never ordered, and the keys at those
positions are left over from before the sort.  The call reports MPM_E_CAPACITY, no kernel
follows an order that was not formed, and the context (or the job beside it) goes on
exactly.  Against the FP64 oracle."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state, oracle_step
from test_gpu_transfer_blocks import KINDS, _oracle_step

pytestmark = pytest.mark.gpu

CROWD = 2100
FORMS = dict(KINDS, mls={}, deterministic=dict(deterministic=True), fused=dict(fused=True))


def _bodies(n_cells):
    """Two small bodies, in the first and the last blocks of the grid."""
    kw = dict(n_cells=n_cells, ext_cells=(5, 4, 6), model=scenes.FIXED_COROTATED, gravity=(0.0, -9.8, 0.0), bc_band=2,
              dt=1e-4, E=3.5e4, v_scale=0.3, B_scale=0.3, F_scale=0.01, dx=1.0 / 64)
    sc = scenes.random_blob(41, lo_cells=(3.25, 3.5, 3.25), **kw)
    end = scenes.random_blob(42, lo_cells=tuple(c - e - 3.5 for c, e in zip(n_cells, (5, 4, 6))), **kw)
    for name in ("x", "v", "B", "F", "mat"):
        setattr(sc, name, np.concatenate([getattr(sc, name), getattr(end, name)]))
    return sc


def _crowded(n_cells, seed=43):
    """The bodies with CROWD particles in one block between them, in random creation order; returns the scene and
    the ids of the bodies' particles, in the order of _bodies."""
    sc = _bodies(n_cells)
    n = sc.n
    rng = np.random.default_rng(seed)
    block = np.array([c // 8 for c in n_cells])
    x = ((4 * block + 0.25 + 3.0 * rng.random((CROWD, 3))) * sc.dx).astype(np.float32)
    order = rng.permutation(n + CROWD)
    for name, more in (("x", x), ("v", np.zeros((CROWD, 3))), ("B", np.zeros((CROWD, 3, 3))),
                       ("F", np.tile(np.eye(3), (CROWD, 1, 1))), ("mat", np.zeros(CROWD))):
        a = getattr(sc, name)
        setattr(sc, name, np.concatenate([a, more.astype(a.dtype)])[order])
    assert np.unique(np.floor(x / sc.dx + 0.25).astype(int) >> 2, axis=0).shape[0] == 1
    return sc, np.argsort(order)[:n]


def first_by_id(parts, ids):
    """The first len(ids) stored particles, which are to be those with these ids, in the order of ids."""
    d = parts.read()
    d = {k: v[:len(ids)] for k, v in d.items()}
    assert np.array_equal(np.sort(d["id"]), np.sort(ids))
    at = np.argsort(d["id"])[np.argsort(np.argsort(ids))]
    return {k: v[at] for k, v in d.items()}


def _oracle(form, sc, steps):
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F))
    for _ in range(steps):
        if form in KINDS:
            _oracle_step(form, sc, st, sc.dt)
        else:
            oracle_step(sc, st, sc.dt, grids=False)
    return st


def _match(got, st, tag):
    for name in ("x", "v", "F"):
        e = nerr(got[name], getattr(st, name))
        log("%s: %s %.2e" % (tag, name, e))
        assert e <= TOL, name


@pytest.mark.parametrize("n_cells", [(32, 32, 32), (64, 92, 124)])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_context_after_a_crowded_block(form, n_cells):
    crowded, ids = _crowded(n_cells)
    sc = _bodies(n_cells)
    run = GpuRun(crowded, **FORMS[form])
    ck, p = run.ck, run.parts
    for steps in (4, 1, 3):
        ck.check(ck.mpm_step(run.ctx.h, p.c, sc.dt, steps, run.stream))
    assert ck.mpm_sync(run.ctx.h, run.stream) == ck.MPM_E_CAPACITY
    # the bodies' particles, which hold the first positions, went on as if the others were not there
    _match(first_by_id(p, ids), _oracle(form, sc, 8), "%s beside a crowded block" % form)
    p.c.n = p.n = sc.n
    p.load(sc.x, sc.v, sc.B, sc.F)
    ck.check(ck.mpm_invalidate(run.ctx.h))
    got = run.steps(sc.dt, 3)
    assert got["status"] == 0
    _match(got, _oracle(form, sc, 3), "%s after a crowded block" % form)
    run.close()


def test_noalloc_after_a_crowded_block():
    import torch
    from paper_2412_10399_amd import ckmpm
    sc, (crowded, _) = _bodies((32, 32, 32)), _crowded((32, 32, 32))
    for scene, want in ((crowded, ckmpm.MPM_E_CAPACITY), (sc, ckmpm.MPM_OK)):
        parts = ckmpm.particles_from_scene(scene, "cuda:0")
        status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        ckmpm.check(ckmpm.mpm_step_noalloc(ckmpm.scene_config(scene), ckmpm.scene_materials(scene), parts.c,
                                           scene.dt, 4, status.data_ptr(), torch.cuda.current_stream()))
        torch.cuda.synchronize()
        assert int(status.item()) == want
    _match(parts.read_by_id(), _oracle("mls", sc, 4), "no-alloc call after a crowded block")


@pytest.mark.parametrize("grouped", [False, True])
def test_crowded_job_fails_alone(grouped):
    from paper_2412_10399_amd import ckmpm
    sc, (crowded, _) = _bodies((32, 32, 32)), _crowded((32, 32, 32))
    srv = ckmpm.Server(memory_budget=1 << 30, max_jobs=4, n_streams=2, steps_per_launch=4, grouped=grouped)
    jids = [srv.submit_scene(s, 8) for s in (sc, crowded, sc)]
    srv.drain()
    info = srv.info(jids[1])
    assert info.state == ckmpm.MPM_JOB_FAILED and info.status == ckmpm.MPM_E_CAPACITY
    st = _oracle("mls", sc, 8)
    for j in (jids[0], jids[2]):
        assert srv.info(j).state == ckmpm.MPM_JOB_DONE
        _match(srv.read(j), st, "job beside a crowded one (%s)" % ("grouped" if grouped else "per job"))
    srv.close()


def test_deterministic_grid_beside_a_crowded_block():
    """The crowded block contributes nothing to the grid, and not what its place in the staging area last held."""
    n_cells = (32, 32, 32)
    crowded, ids = _crowded(n_cells)
    sc = _bodies(n_cells)
    run = GpuRun(crowded, deterministic=True)
    ck, p = run.ck, run.parts
    fewer = crowded.copy()
    keep = np.sort(np.concatenate([ids, np.setdiff1d(np.arange(crowded.n), ids)[:500]]))
    p.c.n = p.n = keep.size
    p.load(*(getattr(fewer, name)[keep] for name in ("x", "v", "B", "F")))
    ck.check(ck.mpm_p2g(run.ctx.h, p.c, sc.dt, run.stream))
    assert run.grids()[0].sum() > 1.2 * sc.n * sc.materials[0].rho * sc.materials[0].vol0
    p.c.n = p.n = crowded.n
    p.load(crowded.x, crowded.v, crowded.B, crowded.F)
    ck.check(ck.mpm_invalidate(run.ctx.h))
    ck.check(ck.mpm_p2g(run.ctx.h, p.c, sc.dt, run.stream))
    m, mom = run.grids()
    assert ck.mpm_sync(run.ctx.h, run.stream) == ck.MPM_E_CAPACITY
    _, g = oracle_step(sc, oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F)), sc.dt)
    assert nerr(m, g["m"]) <= TOL and nerr(mom, g["p"]) <= TOL
    run.close()
