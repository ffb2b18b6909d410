"""The differentiable step where its kernels' branches meet: particle counts around a
workgroup's 128, bodies whose workgroups run over the end of a layer (two boxes split at
a jump in y) or of a long row (split in x), strains on the series and on the
eigen-decomposition side, calls of different kinds and sizes one after the other on one
context (the node arrays take turns and are cleared by the next call), and a captured
call replayed.  Forward and reverse step against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_util import TOL, log, nerr

pytestmark = pytest.mark.gpu


def _scene(seed, ext, n_cells, n=None, F_scale=0.003, lo=(2.2, 2.4, 2.1)):
    sc = scenes.random_blob(seed, n_cells=n_cells, lo_cells=lo, ext_cells=ext, model=scenes.FIXED_COROTATED,
                            v_scale=0.5, B_scale=2.0, F_scale=F_scale, gravity=(0.3, -9.8, 0.1), bc_band=2, dt=1e-4,
                            E=5e4, dx=1.0 / 64)
    if n is not None:
        for name in ("x", "v", "B", "F", "mat"):
            setattr(sc, name, getattr(sc, name)[:n])
    rng = np.random.default_rng(seed + 7)
    sc.logE = (np.log(5e4) + 0.2 * rng.standard_normal(sc.n)).astype(np.float32)
    return sc


def _context(sc, mode, n):
    from paper_2412_10399_amd import ckmpm, diff
    nb = int(np.prod([c // 4 + 1 for c in sc.n_cells]))
    cfg = ckmpm.scene_config(sc, max_particles=n, max_blocks=nb if mode == "direct" else nb - 1)
    return diff.AdContext(cfg, ckmpm.scene_materials(sc)[0])


def _planes(sc):
    import torch
    from paper_2412_10399_amd import ckmpm
    return torch.from_numpy(ckmpm.state_planes(sc.x, sc.v, sc.B, sc.F)).cuda()


def _forward(ad, sc):
    import torch
    from paper_2412_10399_amd import ckmpm
    s0, logE = _planes(sc), torch.from_numpy(sc.logE).cuda()
    out = torch.empty_like(s0)
    stream = torch.cuda.current_stream()
    ckmpm.check(ckmpm.mpm_ad_forward(ad.h, sc.n, sc.n, s0.data_ptr(), logE.data_ptr(), out.data_ptr(), sc.dt, stream))
    ckmpm.check(ckmpm.mpm_ad_sync(ad.h, stream))
    return ckmpm.unpack_state(out.cpu().numpy())


def _check_forward(got, sc, tag):
    st = oracle.State(sc.x, sc.v, sc.B, sc.F, sc.mat, sc.logE)
    status, _, _ = oracle.step(oracle.scene_config(sc), oracle.scene_materials(sc), st, sc.dt)
    assert status == 0
    for k in ("x", "v", "F"):
        e = nerr(got[k], getattr(st, k))
        log("%s forward: %s %.2e" % (tag, k, e))
        assert e <= TOL, k


def _check_backward(ad, sc, tag, seed=3):
    import torch
    from paper_2412_10399_amd import ckmpm
    n = sc.n
    rng = np.random.default_rng(seed)
    cot = [rng.standard_normal((n, 3)), rng.standard_normal((n, 3)), 64 * rng.standard_normal((n, 3, 3)),
           rng.standard_normal((n, 3, 3))]
    st = oracle.State(sc.x, sc.v, sc.B, sc.F, sc.mat, sc.logE)
    status, ref = oracle.step_vjp(oracle.scene_config(sc), oracle.scene_materials(sc), st, sc.dt, *cot)
    assert status == 0
    s0, logE = _planes(sc), torch.from_numpy(sc.logE).cuda()
    rows = [cot[0].T, cot[1].T, cot[2].reshape(n, 9).T, cot[3].reshape(n, 9).T, np.zeros((3, n))]
    cot_out = torch.from_numpy(np.concatenate(rows).astype(np.float32)).cuda().contiguous()
    cot_in = torch.full_like(cot_out, float("nan"))
    lcot = torch.zeros(n, dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream()
    ckmpm.check(ckmpm.mpm_ad_backward(ad.h, n, n, s0.data_ptr(), logE.data_ptr(), cot_out.data_ptr(),
                                      cot_in.data_ptr(), lcot.data_ptr(), sc.dt, stream))
    ckmpm.check(ckmpm.mpm_ad_sync(ad.h, stream))
    g = cot_in.cpu().numpy().astype(np.float64)
    assert np.array_equal(g[24:27], g[0:3])
    got = dict(x=g[0:3].T, v=g[3:6].T, B=g[6:15].T.reshape(n, 3, 3), F=g[15:24].T.reshape(n, 3, 3),
               logE=lcot.cpu().numpy())
    for k in ("x", "v", "B", "F", "logE"):
        e = nerr(got[k], ref[k])
        log("%s reverse: d/d%s %.2e" % (tag, k, e))
        assert e <= 1e-4, k


CASES = [((2, 2, 2), (16, 16, 16), 1), ((2, 2, 2), (16, 16, 16), 2), ((4, 3, 2), (16, 16, 16), 127),
         ((4, 2, 2), (16, 16, 16), 128), ((5, 3, 2), (16, 16, 16), 129), ((9, 5, 3), (16, 16, 16), 1025),
         ((27, 24, 3), (32, 32, 16), None),     # workgroups run over the end of a layer
         ((70, 3, 3), (80, 16, 16), None)]      # rows too long for one box over two of them


@pytest.mark.parametrize("mode", ["direct", "sparse"])
@pytest.mark.parametrize("F_scale", [0.003, 0.05])
@pytest.mark.parametrize("ext,n_cells,n", CASES)
def test_step_and_adjoint_at_tile_edges(ext, n_cells, n, F_scale, mode):
    sc = _scene(51, ext, n_cells, n, F_scale)
    ad = _context(sc, mode, sc.n)
    tag = "%s n=%d F %g %s" % (ext, sc.n, F_scale, mode)
    _check_forward(_forward(ad, sc), sc, tag)
    _check_backward(ad, sc, tag)
    ad.close()


@pytest.mark.parametrize("mode", ["direct", "sparse"])
def test_calls_in_turn_on_one_context(mode):
    """Forward and reverse calls of different bodies in every order: each finds clean
    node arrays."""
    a = _scene(52, (9, 5, 4), (16, 16, 16))
    b = _scene(53, (5, 6, 3), (16, 16, 16), 611, lo=(5.2, 4.4, 6.1))
    ad = _context(a, mode, a.n)
    for k, step in enumerate("fa fb ba bb ba fa fa bb fb ba".split()):
        sc = a if step[1] == "a" else b
        if step[0] == "f":
            _check_forward(_forward(ad, sc), sc, "call %d" % k)
        else:
            _check_backward(ad, sc, "call %d" % k, seed=k)
    ad.close()


@pytest.mark.parametrize("mode", ["direct", "sparse"])
def test_captured_forward_replays(mode):
    """One captured forward call replayed on changing inputs, with eager calls between."""
    import torch
    from paper_2412_10399_amd import ckmpm
    sc = _scene(54, (6, 5, 4), (16, 16, 16))
    ad = _context(sc, mode, sc.n)
    first = _planes(sc)
    s0, logE = first.clone(), torch.from_numpy(sc.logE).cuda()
    out = torch.empty_like(s0)
    _forward(ad, sc)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ckmpm.check(ckmpm.mpm_ad_forward(ad.h, sc.n, sc.n, s0.data_ptr(), logE.data_ptr(), out.data_ptr(), sc.dt,
                                         torch.cuda.current_stream()))
    for k in range(4):
        sc.v = (sc.v * np.float32(1.1)).astype(np.float32)
        s0.copy_(_planes(sc))
        graph.replay()
        torch.cuda.synchronize()
        _check_forward(ckmpm.unpack_state(out.cpu().numpy()), sc, "replay %d" % k)
        if k % 2:
            _check_backward(ad, sc, "between replays")
    ad.close()
