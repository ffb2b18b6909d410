"""The differentiable step on particles in random order, whose workgroups reach nodes all over
the body and add to the grid directly instead of through a tile; odd counts, and particles
outside the domain among them.  Forward and reverse step against the FP64 oracle."""
import numpy as np
import pytest

from gpu_util import TOL, log, nerr
from test_gpu_adjoint_tiles import _check_backward, _check_forward, _context, _forward, _scene

pytestmark = pytest.mark.gpu


def _shuffled(n=None):
    sc = _scene(91, (13, 11, 12), (32, 32, 32), n)
    order = np.random.default_rng(5).permutation(sc.n)
    for name in ("x", "v", "B", "F", "mat", "logE"):
        setattr(sc, name, getattr(sc, name)[order])
    return sc, order


@pytest.mark.parametrize("mode", ["direct", "sparse"])
@pytest.mark.parametrize("n", [131, 2000, 13 * 11 * 12 * 8 - 5])
def test_random_order_matches_oracle(n, mode):
    sc, _ = _shuffled(n)
    ad = _context(sc, mode, sc.n)
    tag = "random order, n=%d %s" % (sc.n, mode)
    _check_forward(_forward(ad, sc), sc, tag)
    _check_backward(ad, sc, tag)
    ad.close()


@pytest.mark.parametrize("mode", ["direct", "sparse"])
def test_random_order_with_particles_outside(mode):
    """Every seventh particle outside the domain: unchanged by the step, and without effect on the others."""
    import torch
    from paper_2412_10399_amd import ckmpm
    sc, _ = _shuffled(3001)
    out = np.arange(0, sc.n, 7)
    keep = np.setdiff1d(np.arange(sc.n), out)
    sc.x[out] = np.array([0.1, 0.5, 0.5], np.float32) * sc.dx
    rest = sc.copy()
    for name in ("x", "v", "B", "F", "mat", "logE"):
        setattr(rest, name, getattr(sc, name)[keep])
    ad = _context(sc, mode, sc.n)
    s0 = torch.from_numpy(ckmpm.state_planes(sc.x, sc.v, sc.B, sc.F)).cuda()
    new = torch.empty_like(s0)
    stream = torch.cuda.current_stream()
    logE = torch.from_numpy(sc.logE).cuda()
    ckmpm.check(ckmpm.mpm_ad_forward(ad.h, sc.n, sc.n, s0.data_ptr(), logE.data_ptr(), new.data_ptr(), sc.dt, stream))
    assert ckmpm.mpm_ad_sync(ad.h, stream) == ckmpm.MPM_E_DOMAIN
    assert torch.equal(new[:, out], s0[:, out])
    got = ckmpm.unpack_state(new[:, keep].contiguous().cpu().numpy())
    _check_forward(got, rest, "with particles outside, %s" % mode)
    ad.close()
