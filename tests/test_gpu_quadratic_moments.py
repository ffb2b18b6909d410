"""First moments of the quadratic kernel's G2P against the sums taken node by node.  Both start
from the same grid velocities (read back after the update); the affine part of the step, H' =
dt C for F = I, is formed in FP64 from them, in FP32 node by node (weight times velocity
difference to the middle node times offset), and by the GPU.  The GPU's sums share their
products, so they are held to be as accurate: root mean square error at most 1.1 times that
of the FP32 sums node by node (0.1 for the sampling of some 10^4 values)."""
import numpy as np
import pytest

import scenes
from gpu_util import GpuRun, log

pytestmark = pytest.mark.gpu


def _weights(xi, T):
    u, c, l = T(1.5) - xi, T(1) - xi, xi - T(0.5)
    return np.stack([T(0.5) * u * u, T(0.75) - c * c, T(0.5) * l * l], -1)   # (n, axis, node)


def _affine(x, vt, dx, dt, T):
    """dt C / dt: C = 4 / dx * sum w (v - c) (o - xi)^T in type T, one node after the other; x exact positions."""
    X = x / dx
    base = np.floor(X - 0.5).astype(np.int64)
    xi = (X - base).astype(T)
    w = _weights(xi, T)
    n = x.shape[0]
    mid = vt[base[:, 2] + 1, base[:, 1] + 1, base[:, 0] + 1].astype(T)
    B = np.zeros((n, 3, 3), T)
    for oz in range(3):
        for oy in range(3):
            for ox in range(3):
                v = vt[base[:, 2] + oz, base[:, 1] + oy, base[:, 0] + ox].astype(T) - mid
                wt = w[:, 0, ox] * (w[:, 1, oy] * w[:, 2, oz])
                off = np.array([ox, oy, oz], T)[None, :] - xi
                B += (wt[:, None] * v)[:, :, None] * off[:, None, :]
    return B * T(4.0 * dt / dx)


@pytest.mark.parametrize("lo", [0.0, 0.5])   # the halves of the cells below and above the middle node
def test_first_moments_are_as_accurate_as_node_by_node(lo):
    sc = scenes.random_blob(95, n_cells=(32, 32, 32), lo_cells=(8.0, 8.0, 8.0), ext_cells=(12, 12, 12),
                            model=scenes.FIXED_COROTATED, dt=1e-4, E=1e4, v_scale=1.0, B_scale=0.0, F_scale=0.0)
    rng = np.random.default_rng(11)
    cell = np.floor(sc.x.astype(np.float64) / sc.dx)
    sc.x = ((cell + lo + 0.499 * rng.random((sc.n, 3))) * sc.dx).astype(np.float32)
    run = GpuRun(sc, quadratic=True)
    got = run.phase_step(sc.dt)
    assert got["status"] == 0
    vt = got["vt"][0]
    x = sc.x.astype(np.float64)
    exact = _affine(x, vt, sc.dx, sc.dt, np.float64)
    plain = _affine(x, vt, sc.dx, sc.dt, np.float32)

    def rms(a):
        return float(np.sqrt(np.mean((a.astype(np.float64) - exact) ** 2)))
    gpu, ref = rms(got["H"]), rms(plain)
    log("fractions from %.1f: rms of H %.2e, error of the GPU %.2e, node by node %.2e (%.2f)" %
        (lo, np.sqrt(np.mean(exact ** 2)), gpu, ref, gpu / ref))
    assert gpu <= 1.1 * ref
    run.close()
