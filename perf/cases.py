"""Performance cases of the compact-kernel MPM framework: the work its users have it do, through the public
entry points of paper_2412_10399_amd (ckmpm and diff), with 64-bit results of the same work in plain torch.

Kinds of case (field "kind"):
  step     a rollout of `steps` time steps from a given state: the state is loaded into the particle buffers and
           advanced by one mpm_step call ("call": "step"), by mpm_step_noalloc, or phase by phase with the grid read
           at the end ("phases"); the particles come back in creation order, as Particles.read_by_id returns them.
           Kernel and transfer options: compact or quadratic kernel, MLS / APIC / PIC, deterministic mode.
  adjoint  a differentiated rollout (diff.rollout, checkpointed): final state, and the gradients of a
           trajectory-matching loss in the initial state and the per-particle log modulus.
  serve    a set of independent jobs through the job server: submission, drain, results, release.

Bodies are boxes of `cx` x `cy` x `cz` cells filled with 8 jittered particles per cell (less `trim` at the end, for
odd counts) on a grid of `grid`^3 cells over the unit box, sand on the floor or an elastic body in mid-air, at rest or
moving with a smooth velocity and strain field (a body in the middle of a simulation).
"""
import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2412_10399_amd import ckmpm, diff

ELASTIC, SAND = ckmpm.MPM_FIXED_COROTATED, ckmpm.MPM_DRUCKER_PRAGER
GRAVITY = (0.0, -9.8, 0.0)
BAND = 2   # sticky walls, cells


def _step(name, cx, cy, cz, grid, steps, material, moving=True, trim=0, call="step", kernel="compact", transfer="mls",
          deterministic=False):
    c = dict(kind="step", cx=cx, cy=cy, cz=cz, trim=trim, grid=grid, steps=steps, material=material, moving=moving,
             call=call, kernel=kernel, transfer=transfer, deterministic=deterministic)
    return dict(c, name=name) if name else c


def _adjoint(name, cx, cy, cz, grid, steps, every=8, trim=0):
    c = dict(kind="adjoint", cx=cx, cy=cy, cz=cz, trim=trim, grid=grid, steps=steps, every=every)
    return dict(c, name=name) if name else c


def _serve(name, jobs, smallest, largest, steps, grouped):
    c = dict(kind="serve", jobs=jobs, smallest=smallest, largest=largest, steps=steps, grouped=grouped)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest served simulations (a thousand particles): launches and latency only
        _step("job_1k", 5, 5, 5, 32, 20, "elastic"),
        # the 32,768-particle falling elastic cube of the test suite and the smoke runs
        _step("elastic_cube_32k", 16, 16, 16, 32, 20, "elastic"),
        # the same size through the call for programs that may not allocate, a few steps at a time
        _step("noalloc_cube_20k", 13, 15, 13, 32, 4, "elastic", trim=277, call="noalloc"),
        # flowing sand of the middle of the serving mix, odd sizes, most blocks reordered every step
        _step("sand_flow_300k", 37, 31, 33, 128, 20, "sand", trim=5),
        # the headline sand column: 4,194,304 particles settling from rest
        _step("sand_column_4M", 64, 128, 64, 256, 40, "sand", moving=False),
        # stress scale: 12.6M particles, sand below and a stiff elastic body above, two materials
        _step("two_materials_12M", 128, 96, 128, 512, 10, "both"),
        # the paper's comparison kernel on a sand block
        _step("quadratic_500k", 40, 41, 39, 128, 10, "sand", kernel="quadratic", trim=3),
        # the exact-gradient transfer on an elastic body
        _step("apic_500k", 41, 40, 39, 128, 10, "elastic", transfer="apic", trim=1),
        # bitwise reproducible runs (regression and replay)
        _step("deterministic_260k", 32, 32, 32, 128, 20, "elastic", deterministic=True),
        # the differentiation workload, a quarter of its 64 steps (dense grids)
        _adjoint("adjoint_box_65k", 32, 16, 16, 64, 16),
        # a differentiated body in a large domain (block-sparse grids), odd count
        _adjoint("adjoint_sparse_120k", 27, 24, 23, 256, 8, trim=9),
        # a burst of small and middling jobs through the server
        _serve("serve_12_jobs", 12, 1000, 120000, 60, False),
    ]


def _box(rng, n, flat=2.0):
    """Sides in cells of a box of about n particles at 8 per cell, aspect ratios up to `flat`."""
    s = (n / 8.0) ** (1.0 / 3.0)
    a, b = flat ** rng.uniform(-0.5, 0.5), flat ** rng.uniform(-0.5, 0.5)
    return tuple(max(3, int(round(s * f))) for f in (a, b, 1.0 / (a * b)))


def _grid_for(side):
    return next((g for g in (32, 64, 128, 256) if g >= 2 * side + 8), 256)


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["noalloc", "phases", "quadratic", "gradient", "deterministic"] + ["adjoint"] * 2 +
                      ["serve"])
    if kind == "serve":
        return _serve(None, rng.randint(4, 14), int(_log_uniform(rng, 1e3, 4e3)), int(_log_uniform(rng, 1e4, 2e5)),
                      10 * rng.randint(3, 8), rng.random() < 0.5)
    if kind == "adjoint":
        cells = _box(rng, _log_uniform(rng, 4e3, 1.5e5))
        grid = rng.choice([_grid_for(max(cells)), 256])
        return _adjoint(None, *cells, grid, rng.randint(3, 16), rng.choice([4, 8]), rng.randint(0, 300))
    top = {"step": 3e6, "noalloc": 4e4, "phases": 3e5, "deterministic": 1e6}.get(kind, 1e6)
    cells = _box(rng, _log_uniform(rng, 1e3, top))
    grid = 32 if kind == "noalloc" else _grid_for(max(cells))
    if kind == "noalloc":
        cells = tuple(min(c, 24) for c in cells)
    n = 8 * cells[0] * cells[1] * cells[2]
    steps = rng.randint(2, 6) if kind in ("noalloc", "phases") else rng.randint(8, max(8, min(30, int(4e7 / n))))
    material = rng.choice(["elastic", "sand", "both"])
    # (an elastic body at rest in mid-air only falls: nothing to compute)
    moving = material == "elastic" or rng.random() < 0.7
    return _step(None, *cells, grid, steps, material, moving, rng.randint(0, min(300, n // 4)),
                 kind if kind in ("noalloc", "phases") else "step", "quadratic" if kind == "quadratic" else "compact",
                 rng.choice(["apic", "pic"]) if kind == "gradient" else "mls", kind == "deterministic")


# ------------------------------------------------------------------ inputs
def _device():
    return torch.device("cuda:0")


def _materials(case):
    """Materials (model, E, nu, rho, friction angle) and the time step of a body."""
    sand, elastic = (SAND, 3.5e5, 0.3, 1600.0, 30.0), (ELASTIC, 1e4, 0.3, 1000.0, 30.0)
    if case["material"] == "both":
        return [sand, (ELASTIC, 1e7, 0.3, 2000.0, 30.0)], 5e-6
    return ([sand], 2e-5) if case["material"] == "sand" else ([elastic], 1e-4)


def _body(case, seed):
    """dict of a body's inputs as FP32 GPU tensors: x (3, n), v (3, n), B, H (9, n), mat (n,), and n."""
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    host = np.random.default_rng(int(seed))
    cx, cy, cz, grid = case["cx"], case["cy"], case["cz"], case["grid"]
    dx = 1.0 / grid
    n = 8 * cx * cy * cz - case.get("trim", 0)
    p = torch.arange(n, device=dev)
    cell, sub = p // 8, p % 8
    at = torch.stack([cell % cx, (cell // cx) % cy, cell // (cx * cy)]).double()
    part = torch.stack([sub & 1, (sub >> 1) & 1, sub >> 2]).double()
    jitter = torch.rand((3, n), generator=gen, device=dev).double()
    floor = case["material"] != "elastic"
    corner = torch.tensor([(grid - cx) // 2, BAND if floor else (grid - cy) // 2, (grid - cz) // 2], device=dev).double()
    x = (corner[:, None] + at + (part + jitter) * 0.5) * dx
    v = torch.zeros((3, n), dtype=torch.float64, device=dev)
    B = torch.zeros((3, 3, n), dtype=torch.float64, device=dev)
    H = torch.zeros((3, 3, n), dtype=torch.float64, device=dev)
    mat = ((at[1] >= (cy + 1) // 2) if case["material"] == "both" else torch.zeros(n, device=dev)).to(torch.uint8)
    if case["moving"]:
        # a few long waves: amplitude, wave vector (per extent of the body) and phase of every component
        ext = max(cx, cy, cz) * dx
        speed, strain = (0.3, 2e-3) if floor else (0.3, 5e-3)
        for a in range(3):
            k = torch.tensor(host.uniform(-2.0, 2.0, 3) * math.pi / ext, device=dev)
            arg = (k[:, None] * x).sum(0) + host.uniform(0.0, 2.0 * math.pi)
            v[a] = speed * torch.sin(arg)
            B[a] = speed * torch.cos(arg) * k[:, None] * (dx * dx / 8.0)   # about (grad v) D
            for b in range(3):
                k = torch.tensor(host.uniform(-2.0, 2.0, 3) * math.pi / ext, device=dev)
                H[a, b] = strain * torch.sin((k[:, None] * x).sum(0) + host.uniform(0.0, 2.0 * math.pi))
    if not floor:
        v[1] -= 1.0
    return dict(n=n, x=x.float(), v=v.float(), B=B.reshape(9, n).float(), H=H.reshape(9, n).float(), mat=mat)


def _planes(body):
    r = torch.zeros((3, body["n"]), dtype=torch.float32, device=_device())
    return torch.cat([body["x"], body["v"], body["B"], body["H"], r]).contiguous()


def _config(case, n, blocks=None):
    lattice = (case["grid"] // 4 + 1) ** 3
    return ckmpm.make_config((case["grid"],) * 3, 1.0 / case["grid"], (0.0, 0.0, 0.0), GRAVITY, BAND, n,
                             blocks or min(lattice, 2 * (n // 256) + 4096), quadratic=case.get("kernel") == "quadratic",
                             transfer={"mls": 0, "apic": 1, "pic": 2}[case.get("transfer", "mls")],
                             deterministic=case.get("deterministic", False))


def _mats(case):
    mats, dt = _materials(case)
    vol0 = (1.0 / case["grid"]) ** 3 / 8
    return [ckmpm.make_material(m[0], m[1], m[2], m[3], vol0, m[4]) for m in mats], dt


def _jobs(case, seed):
    """The bodies of a served burst: sizes spread evenly over the logarithm of the range, alternating materials."""
    out = []
    for j in range(case["jobs"]):
        f = j / max(1, case["jobs"] - 1)
        n = case["smallest"] ** (1.0 - f) * case["largest"] ** f
        side = max(2, int(round((n / 8.0) ** (1.0 / 3.0))))
        out.append((dict(cx=side, cy=side, cz=side, grid=_grid_for(side), material="sand" if j % 2 else "elastic",
                         moving=True), seed * 1000 + j))
    return out


def prepare(case, seed):
    if case["kind"] == "serve":
        jobs, budget = [], 0
        for c, s in _jobs(case, seed):
            body = _body(c, s)
            mats, dt = _mats(c)
            blocks = 2 * (c["cx"] // 4 + 8) ** 3 + 64
            cfg = _config(c, body["n"], blocks)
            budget += ckmpm.mpm_footprint(cfg, body["n"]) + 4096
            jobs.append((cfg, mats, _planes(body), dt))
        srv = ckmpm.Server(budget + (64 << 20), max_jobs=len(jobs), n_streams=4, steps_per_launch=10,
                           grouped=case["grouped"])
        return dict(case=case, server=srv, jobs=jobs)
    if case["kind"] == "adjoint":
        body = _body(dict(case, material="elastic", moving=True), seed)
        n, grid = body["n"], case["grid"]
        vol0 = (1.0 / grid) ** 3 / 8
        lattice = (grid // 4 + 1) ** 3
        blocks = lattice if lattice * 7168 <= 256 * 2 ** 20 else min(lattice, 2 * (n // 256) + 4096)
        ad = diff.AdContext(_config(case, n, blocks), ckmpm.make_material(ELASTIC, 5e4, 0.3, 1000.0, vol0))
        logE, target = _learned(body, seed)
        return dict(case=case, ad=ad, state0=_planes(body), logE=logE, target=target, dt=_adjoint_dt(case))
    body = _body(case, seed)
    mats, dt = _mats(case)
    parts = ckmpm.Particles(body["n"], device=_device(), with_mat=len(mats) > 1)
    cfg = _config(case, body["n"])
    st = dict(case=case, parts=parts, cfg=cfg, mats=mats, dt=dt, start=_planes(body), mat=body["mat"],
              ids=torch.arange(body["n"], dtype=torch.int32, device=_device()))
    if case["call"] != "noalloc":
        st["ctx"] = ckmpm.Context(cfg, mats)
    return st


def _adjoint_dt(case):
    return 1e-4 * min(1.0, 64.0 / case["grid"])


def _learned(body, seed):
    """Log modulus field and target positions of the trajectory-matching loss."""
    gen = torch.Generator(device=_device()).manual_seed(int(seed) + 7)
    logE = math.log(5e4) + 0.1 * torch.randn(body["n"], generator=gen, device=_device())
    return logE, body["x"] + 0.01 * torch.randn((3, body["n"]), generator=gen, device=_device())


# ------------------------------------------------------------------ one pass
def run(state):
    kind = state["case"]["kind"]
    return _run_serve(state) if kind == "serve" else _run_adjoint(state) if kind == "adjoint" else _run_step(state)


def _fields(planes):
    """A state as its user reads it: position x + r in FP64, velocity, affine matrix, H = F - I."""
    return dict(x=planes[0:3].double() + planes[24:27].double(), v=planes[3:6], B=planes[6:15], H=planes[15:24])


def _by_id(planes, ids):
    return torch.empty_like(planes).index_copy_(1, ids.long(), planes)


def _run_step(s):
    case, parts, dt = s["case"], s["parts"], s["dt"]
    stream = torch.cuda.current_stream()
    parts.c.current = 0
    parts.state[0].copy_(s["start"])
    parts.ids[0].copy_(s["ids"])
    if parts.mats is not None:
        parts.mats[0].copy_(s["mat"])
    out = {}
    if case["call"] == "noalloc":
        ckmpm.check(ckmpm.mpm_step_noalloc(s["cfg"], s["mats"], parts.c, dt, case["steps"], None, stream))
    else:
        h = s["ctx"].h
        ckmpm.check(ckmpm.mpm_invalidate(h))
        if case["call"] == "phases":
            for _ in range(case["steps"]):
                ckmpm.check(ckmpm.mpm_p2g(h, parts.c, dt, stream))
                ckmpm.check(ckmpm.mpm_grid_update(h, dt, stream))
                ckmpm.check(ckmpm.mpm_g2p(h, parts.c, dt, stream))
            m = case["grid"] + 1
            out["mass"] = torch.empty((2, m, m, m), device=_device())
            out["velocity"] = torch.empty((2, m, m, m, 3), device=_device())
            ckmpm.check(ckmpm.mpm_grid_read(h, 0, out["mass"].data_ptr(), out["velocity"].data_ptr(), stream))
        else:
            ckmpm.check(ckmpm.mpm_step(h, parts.c, dt, case["steps"], stream))
    cur = parts.current
    return dict(_fields(_by_id(parts.state[cur], parts.ids[cur])), **out)


def _loss(final, target):
    return ((final[0:3] - target) ** 2).sum() / target.shape[1]


def _run_adjoint(s):
    state0 = s["state0"].detach().requires_grad_(True)
    logE = s["logE"].detach().requires_grad_(True)
    final = diff.rollout(s["ad"], state0, logE, s["case"]["steps"], s["dt"], checkpoint_every=s["case"]["every"])
    _loss(final, s["target"]).backward()
    g = state0.grad
    return dict(_fields(final.detach()), gx=g[0:3], gv=g[3:6], gB=g[6:15], gH=g[15:24], glogE=logE.grad)


def _run_serve(s):
    srv, out = s["server"], []
    ids = [srv.submit(cfg, mats, planes, s["case"]["steps"], dt) for cfg, mats, planes, dt in s["jobs"]]
    srv.drain()
    for jid, (_, _, planes, _) in zip(ids, s["jobs"]):
        state = torch.empty_like(planes)
        pid = torch.empty(planes.shape[1], dtype=torch.int32, device=planes.device)
        ckmpm.check(ckmpm.mpm_server_job_read(srv.h, jid, state.data_ptr(), pid.data_ptr()))
        srv.release(jid)
        out.append(_fields(_by_id(state, pid)))
    return out


# ------------------------------------------------------------------ work
def work(case):
    """Particles are read and written once a step (x, H in; x, v, B, H out; x, v, B, H into the transfer: 240 B, the
    reverse step about three times that), each touched 4^3-node block of both grids is summed, updated and read."""
    if case["kind"] == "serve":
        bodies = [c for c, _ in _jobs(case, 0)]
    else:
        bodies = [case]
    nbytes = flops = 0.0
    for c in bodies:
        n = 8 * c["cx"] * c["cy"] * c["cz"] - c.get("trim", 0)
        blocks = 1
        for a in ("cx", "cy", "cz"):
            blocks *= c[a] // 4 + 3
        steps = case["steps"]
        if case["kind"] == "adjoint":   # forward, recomputed forward, and the reverse step
            nbytes += steps * (2 * 240.0 + 480.0) * n
            flops += steps * 6000.0 * n
        else:
            nbytes += steps * (240.0 * n + 9216.0 * blocks)
            flops += steps * (2200.0 if case.get("kernel") == "quadratic" else 1500.0) * n
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits
# One explicit MLS-MPM step on the two staggered grids, written from its definition in torch FP64; matrices are
# (n, 3, 3).  Differentiable for the fixed corotated material.
def _mul(a, b):
    return (a[:, :, :, None] * b[:, None, :, :]).sum(2)


def _cof(a):
    c = torch.linalg.cross
    return torch.stack([c(a[:, 1], a[:, 2]), c(a[:, 2], a[:, 0]), c(a[:, 0], a[:, 1])], 1)


def _inv(a):
    c = _cof(a)
    return c.transpose(1, 2) / (a[:, 0] * c[:, 0]).sum(1)[:, None, None]


def _polar(F):
    R = F
    for _ in range(7):   # Newton's iteration for the orthogonal factor, F near a rotation
        c = _cof(R)
        R = 0.5 * (R + c / (R[:, 0] * c[:, 0]).sum(1)[:, None, None])
    return R


def _eig(A):
    """Eigenvalues (n, 3) and eigenvectors (columns) of symmetric matrices by cyclic Jacobi rotations."""
    A = A.clone()
    V = torch.eye(3, dtype=A.dtype, device=A.device).expand_as(A).clone()
    for _ in range(6):
        for p, q in ((0, 1), (0, 2), (1, 2)):
            apq, d = A[:, p, q], A[:, q, q] - A[:, p, p]
            den = d.abs() + torch.sqrt(d * d + 4 * apq * apq)
            t = torch.where(den > 0, 2 * apq * torch.where(d >= 0, 1.0, -1.0) / den.clamp_min(1e-300), 0.0)
            c = 1 / torch.sqrt(1 + t * t)
            s = t * c
            for M, both in ((A, True), (V, False)):
                x, y = M[:, :, p].clone(), M[:, :, q].clone()
                M[:, :, p], M[:, :, q] = c[:, None] * x - s[:, None] * y, s[:, None] * x + c[:, None] * y
                if both:
                    x, y = M[:, p].clone(), M[:, q].clone()
                    M[:, p], M[:, q] = c[:, None] * x - s[:, None] * y, s[:, None] * x + c[:, None] * y
    return torch.diagonal(A, dim1=1, dim2=2), V


def _eye(F):
    return torch.eye(3, dtype=F.dtype, device=F.device)


def _corotated(H, mu, lam):
    F = H + _eye(H)
    J = torch.linalg.det(F) if not H.requires_grad else (F[:, 0] * _cof(F)[:, 0]).sum(1)
    k = lam * (J - 1) * J
    return 2 * mu[:, None, None] * _mul(F - _polar(F), F.transpose(1, 2)) + k[:, None, None] * _eye(F)


def _hencky(H):
    """Log strains and the left and right singular vectors of F = I + H."""
    F = H + _eye(H)
    e, V = _eig(H + H.transpose(1, 2) + _mul(H.transpose(1, 2), H))
    eps = (0.5 * torch.log1p(e)).clamp_min(math.log(1e-4))
    return eps, _mul(F, V) / torch.exp(eps)[:, None, :], V


def _sand_stress(H, mu, lam):
    eps, U, _ = _hencky(H)
    t = 2 * mu * eps + lam * eps.sum(1, keepdim=True)
    return _mul(U * t[:, None, :], U.transpose(1, 2))


def _sand_return(H, mu, lam, friction):
    eps, U, V = _hencky(H)
    s = math.sin(math.radians(friction))
    alpha = math.sqrt(2.0 / 3.0) * 2 * s / (3 - s)
    tr = eps.sum(1, keepdim=True)
    dev = eps - tr / 3
    dn = torch.sqrt((dev * dev).sum(1, keepdim=True))
    gamma = dn + (3 * lam + 2 * mu) / (2 * mu) * tr * alpha
    tip = (tr > 0) | (dn == 0)
    new = torch.where(tip, 0.0, torch.where(gamma > 0, eps - gamma * dev / dn.clamp_min(1e-300), eps))
    grown = _mul(U * (torch.exp(new) - torch.exp(eps))[:, None, :], V.transpose(1, 2))
    return H + grown


def _stencils(X, kernel):
    """Per grid: offset, base node (n, 3), weights and their derivatives (n, 3, nodes per axis)."""
    if kernel == "quadratic":
        base = torch.floor(X.detach() - 0.5)
        xi = X - base
        w = torch.stack([0.5 * (1.5 - xi) ** 2, 0.75 - (1 - xi) ** 2, 0.5 * (xi - 0.5) ** 2], 2)
        return [(0.0, base.long(), w, None, xi)]
    out = []
    for k in (-0.25, 0.25):
        base = torch.floor(X.detach() - k)
        xi = X - k - base
        s = torch.sin(2 * math.pi * xi) / (2 * math.pi)
        c = torch.cos(2 * math.pi * xi) - 1
        out.append((k, base.long(), torch.stack([1 - xi + s, xi - s], 2), torch.stack([c, -c], 2), xi))
    return out


def _nodes(st, dx, m):
    """Flat node index, weight, weight gradient and x_i - x_p of every node of one grid's stencil."""
    _, base, w, dw, xi = st
    r = range(w.shape[2])
    for oz in r:
        for oy in r:
            for ox in r:
                at = ((base[:, 2] + oz) * m + base[:, 1] + oy) * m + base[:, 0] + ox
                wx, wy, wz = w[:, 0, ox], w[:, 1, oy], w[:, 2, oz]
                g = None
                if dw is not None:
                    g = torch.stack([dw[:, 0, ox] * wy * wz, wx * dw[:, 1, oy] * wz, wx * wy * dw[:, 2, oz]], 1) / dx
                off = torch.tensor([ox, oy, oz], dtype=xi.dtype, device=xi.device)
                yield at, wx * wy * wz, g, (off - xi) * dx


def _free(k, grid, dev):
    """Whether node (z, y, x) of the grid at offset k lies inside the sticky walls."""
    p = torch.arange(grid + 1, device=dev).double() + k
    ok = (p >= BAND) & (p <= grid - BAND)
    return (ok[:, None, None] & ok[None, :, None] & ok[None, None, :]).reshape(-1)


def _exact_step(S, dt, grid, mass, vol0, stress, finish, kernel="compact", transfer="mls", grids=None):
    """(x, v, B, H) after one step; mass (n,), stress(H) -> tau, finish(H) -> H after the return mapping."""
    x, v, B, H = S
    dx, m = 1.0 / grid, grid + 1
    sts = _stencils(x / dx, kernel)
    share = 1.0 / len(sts)
    if kernel == "quadratic":
        Di = (4.0 / dx ** 2) * _eye(x)[None]
    else:
        D = 0.0
        for _, _, w, _, xi in sts:
            d = torch.stack([-xi, 1 - xi], 2) * dx
            m1, m2 = (w * d).sum(2), (w * d * d).sum(2)
            D = D + share * (m1[:, :, None] * m1[:, None, :] * (1 - _eye(x)) + torch.diag_embed(m2))
        Di = _inv(D)
    T = -dt * vol0 * stress(H)
    affine = mass[:, None, None] * B
    if transfer == "mls":
        affine = affine + T
    Q = _mul(affine, Di.expand_as(affine)) if transfer != "pic" else torch.zeros_like(affine)
    vn, Bn, C = 0.0, 0.0, 0.0
    g = dt * torch.tensor(GRAVITY, dtype=x.dtype, device=x.device)
    for st in sts:
        node = torch.zeros((m ** 3, 4), dtype=x.dtype, device=x.device)
        for at, w, gw, d in _nodes(st, dx, m):
            p = w[:, None] * (mass[:, None] * v + (Q * d[:, None, :]).sum(2))
            if transfer != "mls":
                p = p + (T * gw[:, None, :]).sum(2)
            node = node.index_add(0, at, torch.cat([(w * mass)[:, None], p], 1))
        live = (node[:, 0] > 0) & _free(st[0], grid, x.device)
        vel = torch.where(live[:, None], node[:, 1:] / torch.where(live, node[:, 0], 1.0)[:, None] + g, 0.0)
        if grids is not None:
            grids.append((node[:, 0], vel))
        for at, w, gw, d in _nodes(st, dx, m):
            vi = share * vel[at]
            vn = vn + w[:, None] * vi
            Bn = Bn + w[:, None, None] * vi[:, :, None] * d[:, None, :]
            if transfer != "mls":
                C = C + vi[:, :, None] * gw[:, None, :]
        del node, vel
    if transfer == "mls":
        C = _mul(Bn, Di.expand_as(Bn))
    Hn = H + dt * (C + _mul(C, H))
    if transfer == "pic":
        Bn = torch.zeros_like(Bn)
    return x + dt * vn, vn, Bn, finish(Hn)


def _lame(E, nu):
    return E / (2 * (1 + nu)), E * nu / ((1 + nu) * (1 - 2 * nu))


def _matrices(a):
    return a.t().reshape(-1, 3, 3).double()


def _rows(S):
    x, v, B, H = S
    n = x.shape[0]
    return dict(x=x.t(), v=v.t(), B=B.reshape(n, 9).t(), H=H.reshape(n, 9).t())


def _exact_rollout(case, body, steps):
    mats, dt = _materials(case)
    dt, grid = float(np.float32(dt)), case["grid"]
    vol0 = (1.0 / grid) ** 3 / 8
    kind = body["mat"].long()
    mass = torch.tensor([q[3] * vol0 for q in mats], dtype=torch.float64, device=_device())[kind]
    lame = [_lame(q[1], q[2]) for q in mats]
    split = [torch.nonzero(kind == i).reshape(-1) for i in range(len(mats))]

    def by_material(H, elastic, sand):
        out = torch.empty_like(H)
        for (mu, lam), q, at in zip(lame, mats, split):
            for part in at.split(1 << 21):   # bounds the temporaries
                h = H[part]
                out[part] = elastic(h, mu, lam) if q[0] == ELASTIC else sand(h, mu, lam, q[4])
        return out

    def stress(H):
        return by_material(H, lambda h, mu, lam: _corotated(h, torch.full_like(h[:, 0, 0], mu), lam),
                           lambda h, mu, lam, _: _sand_stress(h, mu, lam))

    def finish(H):
        return by_material(H, lambda h, mu, lam: h, _sand_return)

    S = (body["x"].t().double(), body["v"].t().double(), _matrices(body["B"]), _matrices(body["H"]))
    grids = []
    for k in range(steps):
        last = grids if case.get("call") == "phases" and k + 1 == steps else None
        S = _exact_step(S, dt, grid, mass, vol0, stress, finish, case.get("kernel", "compact"),
                        case.get("transfer", "mls"), last)
    out = _rows(S)
    if case.get("call") == "phases":
        m = grid + 1
        out["mass"] = torch.stack([a.reshape(m, m, m) for a, _ in grids])
        out["velocity"] = torch.stack([b.reshape(m, m, m, 3) for _, b in grids])
    return out


def exact(case, seed):
    if case["kind"] == "serve":
        return [_exact_rollout(c, _body(c, s), case["steps"]) for c, s in _jobs(case, seed)]
    n = 8 * case["cx"] * case["cy"] * case["cz"]
    if case["kind"] == "step":
        if n * case["steps"] > 2e8:
            return None
        return _exact_rollout(case, _body(case, seed), case["steps"])
    if n * case["steps"] > 2.5e6:   # the saved tensors of every step
        return None
    body = _body(dict(case, material="elastic", moving=True), seed)
    logE, target = (t.double() for t in _learned(body, seed))
    n, grid, dt = body["n"], case["grid"], float(np.float32(_adjoint_dt(case)))
    vol0 = (1.0 / grid) ** 3 / 8
    first = [body["x"].t().double(), body["v"].t().double(), _matrices(body["B"]), _matrices(body["H"])]
    first = [t.clone().requires_grad_(True) for t in first]
    logE.requires_grad_(True)
    mu, lam = _lame(1.0, 0.3)
    mass = torch.full((n,), 1000.0 * vol0, dtype=torch.float64, device=_device())
    E = torch.exp(logE)

    def one(x, v, B, H, E):
        return _exact_step((x, v, B, H), dt, grid, mass, vol0, lambda h: _corotated(h, mu * E, lam * E), lambda h: h)

    S = tuple(first)
    for _ in range(case["steps"]):
        S = torch.utils.checkpoint.checkpoint(one, *S, E, use_reentrant=False)
    _loss(S[0].t(), target).backward()
    g = _rows([t.grad for t in first])
    return dict(_rows([t.detach() for t in S]), gx=g["x"], gv=g["v"], gB=g["B"], gH=g["H"], glogE=logE.grad)
