"""Block counts and the compaction that turns them into sorted ranges: lattices on either
side of a 1,024-block chunk and of the one-launch line (12 chunks), with bodies in the
first and the last blocks; and every way of leaving counts behind that the next sort must
not see (a P2G without its G2P, a sort for its keys alone, invalidation, another particle
count, an overflow of the block pool).  Against the FP64 checker."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state, oracle_step

pytestmark = pytest.mark.gpu


def _two_bodies(n_cells, seed=21):
    """Small bodies near both ends of the grid."""
    kw = dict(n_cells=n_cells, ext_cells=(5, 4, 3), model=scenes.FIXED_COROTATED, gravity=(0.0, -9.8, 0.0), bc_band=2,
              dt=1e-4, E=3.5e4, v_scale=0.3, B_scale=0.3, F_scale=0.01, dx=1.0 / 64)
    a = scenes.random_blob(seed, lo_cells=(2.25, 2.5, 2.25), **kw)
    b = scenes.random_blob(seed + 1, lo_cells=tuple(c - e - 2.5 for c, e in zip(n_cells, (5, 4, 3))), **kw)
    for name in ("x", "v", "B", "F", "mat"):
        setattr(a, name, np.concatenate([getattr(a, name), getattr(b, name)]))
    return a


def _blocks(sc):
    c = np.floor(sc.x.astype(np.float64) / sc.dx + 0.25).astype(np.int64) >> 2
    return np.unique(c, axis=0, return_counts=True)[1]


def _match(got, sc, steps, tag):
    st = oracle_state(dict(x=sc.x, v=sc.v, B=sc.B, F=sc.F))
    for _ in range(steps):
        oracle_step(sc, st, sc.dt, grids=False)
    for name in ("x", "v", "F"):
        e = nerr(got[name], getattr(st, name))
        log("%s: %s %.2e" % (tag, name, e))
        assert e <= TOL, name


@pytest.mark.parametrize("n_cells", [(60, 28, 28), (64, 28, 28), (60, 92, 124), (64, 92, 124)])
def test_lattices_around_the_chunks(n_cells):
    nb = int(np.prod([c // 4 + 1 for c in n_cells]))
    assert nb in (1024, 1088, 12 * 1024, 13056)
    sc = _two_bodies(n_cells)
    run = GpuRun(sc)
    got = run.steps(sc.dt, 1)
    assert got["status"] == 0
    s, stats = run.ck.mpm_get_stats(run.ctx.h, run.stream)
    counts = _blocks(sc)
    assert s == 0 and stats.n_particle_blocks == len(counts) and stats.max_block_particles == counts.max()
    got = run.steps(sc.dt, 2)
    assert got["status"] == 0
    _match(got, sc, 3, "%d blocks" % nb)
    run.close()


def _restart(run, sc):
    cur = run.parts.current
    p = run.parts
    p.load(sc.x, sc.v, sc.B, sc.F)
    assert p.current == cur
    run.ck.check(run.ck.mpm_invalidate(run.ctx.h))


@pytest.mark.parametrize("leave", ["p2g", "p2g twice", "sort", "step", "steps"])
def test_counts_left_behind(leave):
    """After each way of leaving counts, a fresh start on the same context is exact."""
    import torch
    sc = _two_bodies((32, 32, 32))
    run = GpuRun(sc)
    ck, h, p = run.ck, run.ctx.h, run.parts.c
    for _ in range(2):
        if leave.startswith("p2g"):
            for _ in range(leave.count(" ") + 1):
                ck.check(ck.mpm_p2g(h, p, sc.dt, run.stream))
        elif leave == "sort":
            keys = torch.zeros(sc.n, dtype=torch.int32, device="cuda")
            ck.check(ck.mpm_sort_keys(h, p, keys.data_ptr(), None, run.stream))
        else:
            ck.check(ck.mpm_step(h, p, sc.dt, 1 if leave == "step" else 4, run.stream))
        _restart(run, sc)
        got = run.steps(sc.dt, 3)
        assert got["status"] == 0
        _match(got, sc, 3, "after " + leave)
        s, stats = ck.mpm_get_stats(h, run.stream)
        assert s == 0 and stats.n_particle_blocks <= 2 * len(_blocks(sc))
        _restart(run, sc)
    run.close()


def test_fewer_particles_then_all():
    sc = _two_bodies((32, 32, 32))
    run = GpuRun(sc)
    ck, p = run.ck, run.parts.c
    half = sc.n // 2
    p.n = half
    assert ck.mpm_step(run.ctx.h, p, sc.dt, 2, run.stream) == ck.MPM_OK
    assert ck.mpm_sync(run.ctx.h, run.stream) == ck.MPM_OK
    p.n = sc.n
    _restart(run, sc)
    got = run.steps(sc.dt, 3)
    assert got["status"] == 0
    _match(got, sc, 3, "all after half")
    run.close()


@pytest.mark.parametrize("many_particle_blocks", [False, True])
def test_pool_overflow_then_a_smaller_set(many_particle_blocks):
    """The overflow is reported (of grid blocks alone, and of particle blocks too); a set
    that fits then runs on the same context."""
    if many_particle_blocks:
        sc = scenes.random_blob(23, n_cells=(32, 32, 32), lo_cells=(4.25, 4.25, 4.25), ext_cells=(14, 14, 14),
                                model=scenes.FIXED_COROTATED, gravity=(0.0, -9.8, 0.0), bc_band=2, dt=1e-4, E=3.5e4,
                                v_scale=0.3, B_scale=0.3, F_scale=0.01, dx=1.0 / 64)
        run, fits = GpuRun(sc, max_blocks=27), 8
    else:
        sc = _two_bodies((32, 32, 32))
        run, fits = GpuRun(sc, max_blocks=60), sc.n // 2
    ck, p = run.ck, run.parts.c
    assert ck.mpm_step(run.ctx.h, p, sc.dt, 3, run.stream) == ck.MPM_OK
    assert ck.mpm_sync(run.ctx.h, run.stream) == ck.MPM_E_CAPACITY
    for name in ("x", "v", "B", "F", "mat"):
        setattr(sc, name, getattr(sc, name)[:fits].copy())
    p.n = run.parts.n = sc.n
    _restart(run, sc)
    run.steps(sc.dt, 1)   # its first sort still sees the grid stamps of the failed steps' last G2P
    for _ in range(2):
        _restart(run, sc)
        got = run.steps(sc.dt, 3)
        assert got["status"] == 0
        _match(got, sc, 3, "after an overflow")
    run.close()
