"""Small bodies in the first and the last blocks of large lattices: compaction by sums over the
chunks of 1,024 blocks before, and, above 24,576 chunks, after a scan of their counts; as a
context of its own and as a job of a grouped server.  The FP64 oracle steps each body on a
small grid around it, its origin moved by whole blocks."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, TOL, log, nerr, oracle_state, oracle_step

pytestmark = pytest.mark.gpu

BLOCKS = 512   # pool of every run here
LATTICES = [(60, 92, 128), (252, 252, 260), (1200, 1200, 1116)]


def _bodies(n_cells):
    """A body near either end: its scene on the whole grid and on a small grid around it."""
    out = []
    for seed, end in ((81, False), (82, True)):
        ext = (5, 4, 6)
        lo = np.array([c - e - 3.25 if end else 3.25 for c, e in zip(n_cells, ext)])
        sc = scenes.random_blob(seed, n_cells=n_cells, lo_cells=tuple(lo), ext_cells=ext, model=scenes.FIXED_COROTATED,
                                gravity=(0.0, -9.8, 0.0), dt=2e-5, E=3.5e4, v_scale=0.3, B_scale=0.3, F_scale=0.01,
                                dx=1.0 / 1024)
        small = sc.copy()
        small.n_cells = (16, 16, 16)
        small.origin = tuple(((np.floor(lo).astype(int) // 4) * 4 - 4 * (lo > 4)) * sc.dx)
        out.append((sc, small))
    return out


def _match(got, small, steps, tag):
    st = oracle_state(dict(x=small.x, v=small.v, B=small.B, F=small.F))
    for _ in range(steps):
        oracle_step(small, st, small.dt, grids=False)
    origin = np.asarray(small.origin)
    for name, a, b in (("x", got["x"] - origin, st.x - origin), ("v", got["v"], st.v), ("F", got["F"], st.F)):
        e = nerr(a, b)
        log("%s: %s %.2e" % (tag, name, e))
        assert e <= TOL, name


@pytest.mark.parametrize("n_cells", LATTICES)
def test_context_on_a_large_lattice(n_cells):
    bodies = _bodies(n_cells)
    both = bodies[0][0].copy()
    for name in ("x", "v", "B", "F", "mat"):
        setattr(both, name, np.concatenate([getattr(sc, name) for sc, _ in bodies]))
    run = GpuRun(both, max_blocks=BLOCKS)
    got = run.steps(both.dt, 4)
    assert got["status"] == 0
    n = bodies[0][0].n
    for part, (_, small) in zip((slice(0, n), slice(n, None)), bodies):
        _match({k: got[k][part] for k in ("x", "v", "F")}, small, 4, "%s, origin %s" % (n_cells, small.origin))
    run.close()


@pytest.mark.parametrize("n_cells", LATTICES)
def test_grouped_jobs_on_a_large_lattice(n_cells):
    import torch
    from paper_2412_10399_amd import ckmpm
    bodies = _bodies(n_cells)
    cfgs = [ckmpm.scene_config(sc, max_blocks=BLOCKS) for sc, _ in bodies]
    budget = sum(ckmpm.mpm_footprint(c, sc.n) + 4096 for c, (sc, _) in zip(cfgs, bodies))
    srv = ckmpm.Server(memory_budget=budget, max_jobs=2, n_streams=2, steps_per_launch=4, grouped=True)
    jids = []
    for cfg, (sc, _) in zip(cfgs, bodies):
        state = torch.from_numpy(ckmpm.state_planes(sc.x, sc.v, sc.B, sc.F)).cuda()
        jids.append(srv.submit(cfg, ckmpm.scene_materials(sc), state, 8, sc.dt))
    srv.drain()
    for j, (_, small) in zip(jids, bodies):
        assert srv.info(j).state == ckmpm.MPM_JOB_DONE
        _match(srv.read(j), small, 8, "job on %s, origin %s" % (n_cells, small.origin))
    srv.close()
