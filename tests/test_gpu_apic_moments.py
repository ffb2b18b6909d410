"""The affine matrix of the APIC kernel's G2P against the sums taken node by node.  Both start
from the same grid velocities (read back after the update): B is formed in FP64 from them, in
FP32 node by node (weight times velocity difference to one node of the stencil times offset),
and by the GPU.  The GPU's sums share their products, so they are held to be as accurate: root
mean square error at most 1.1 times that of the FP32 sums node by node (0.1 for the sampling
of some 10^4 values and the kernel's sine, which is within 1.3e-7)."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, log

pytestmark = pytest.mark.gpu


def _affine(x, vt, dx, T):
    """B = dx/2 sum over both grids of w (v - c) (o - xi)^T in type T, one node after the other; x exact positions."""
    X = x / dx
    n = x.shape[0]
    B = np.zeros((n, 3, 3), T)
    c = None
    for g, k in ((0, -0.25), (1, 0.25)):
        base = np.floor(X - k).astype(np.int64)
        xi = (X - k - base).astype(T)
        s = (np.sin(2 * np.pi * (X - k - base)) / (2 * np.pi)).astype(T)
        w = np.stack([T(1) - xi + s, xi - s], -1)
        if c is None:
            c = vt[0][base[:, 2], base[:, 1], base[:, 0]].astype(T)
        for oz in range(2):
            for oy in range(2):
                for ox in range(2):
                    v = vt[g][base[:, 2] + oz, base[:, 1] + oy, base[:, 0] + ox].astype(T) - c
                    wt = w[:, 0, ox] * w[:, 1, oy] * w[:, 2, oz]
                    off = np.array([ox, oy, oz], T)[None, :] - xi
                    B += (wt[:, None] * v)[:, :, None] * off[:, None, :]
    return B * T(0.5 * dx)


@pytest.mark.parametrize("lo", [0.0, 0.25, 0.5, 0.75])   # quarters of the cells
def test_affine_matrix_is_as_accurate_as_node_by_node(lo):
    sc = scenes.random_blob(96, n_cells=(32, 32, 32), lo_cells=(8.0, 8.0, 8.0), ext_cells=(12, 12, 12),
                            model=scenes.FIXED_COROTATED, dt=1e-4, E=1e4, v_scale=1.0, B_scale=0.0, F_scale=0.0)
    rng = np.random.default_rng(12)
    cell = np.floor(sc.x.astype(np.float64) / sc.dx)
    sc.x = ((cell + lo + 0.2499 * rng.random((sc.n, 3))) * sc.dx).astype(np.float32)
    run = GpuRun(sc, transfer=1)
    got = run.phase_step(sc.dt)
    assert got["status"] == 0
    x = sc.x.astype(np.float64)
    exact = _affine(x, got["vt"], sc.dx, np.float64)
    plain = _affine(x, got["vt"], sc.dx, np.float32)

    def rms(a):
        return float(np.sqrt(np.mean((a.astype(np.float64) - exact) ** 2)))
    gpu, ref = rms(got["B"]), rms(plain)
    log("fractions from %.2f: rms of B %.2e, error of the GPU %.2e, node by node %.2e (%.2f)" %
        (lo, np.sqrt(np.mean(exact ** 2)), gpu, ref, gpu / ref))
    assert gpu <= 1.1 * ref
    run.close()
