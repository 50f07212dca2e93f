"""Performance cases of the patch-batch library.

Each case is the work of one call sequence that a program built on this
package makes: time steps of a resident patch batch (finite volumes, FD4 +
Kreiss-Oliger + RK4), of a special-relativistic batch with its nonlinear
solve, one gradient of the guess network, one offload call on host chunks.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and the objects a program keeps between calls
    run(state)          one pass
    work(case)          bytes and operations the pass cannot do without
    exact(case, seed)   what run() returns for these inputs, in plain float64

Inputs are synthetic: smooth sums of Fourier modes, or values drawn per cell,
as each recipe below says.  The state of a batch advances from pass to pass,
as in a simulation, unless the case restarts: then every pass is the step on
the batch's initial state.
"""
import math

import numpy as np
import torch

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

DEV = "cuda"
GAMMA = 1.4          # Euler
GAM_R = 5.0 / 3.0    # relativistic
CFL_FV, CFL_FD, SIGMA = 0.4, 0.5, 0.1


def listed():
    return [
        # the smallest call: one step of the 2D entropy wave on 64 patches of 8^2, launch-bound
        dict(name="euler2d_wave", kind="fv", dim=2, gx=8, gy=8, gz=1, p=8, own=False, storage="fp64", steps=1,
             graph=False),
        # the resident 3D run at its full size: 2048 patches of 16^3, ten steps a call
        dict(name="euler3d_fp64", kind="fv", dim=3, gx=16, gy=16, gz=8, p=16, own=False, storage="fp64", steps=10,
             graph=False),
        # binary32 storage on a middling grid of patches that fill no 16 x 16 plane
        dict(name="euler3d_fp32_ragged", kind="fv", dim=3, gx=11, gy=9, gz=7, p=13, own=False, storage="fp32",
             steps=5, graph=False),
        # many small independent patches handed over at once, as a task-fusing mesh code does
        dict(name="euler3d_small_patches", kind="fv", dim=3, gx=8694, gy=1, gz=1, p=6, own=True, storage="fp64",
             steps=5, graph=False),
        # the fourth-order scheme on the full grid
        dict(name="euler3d_fd4", kind="fd", gx=16, gy=16, gz=8, p=16, own=False, steps=2, graph=False),
        # the fourth-order scheme on small independent patches, one step a call
        dict(name="euler3d_fd4_small", kind="fd", gx=1024, gy=1, gz=1, p=6, own=True, steps=1, graph=False),
        # 58 unknowns on 4096 patches of 4^3, 8^3 and 16^3 in ratio 1:2:1, the largest work
        dict(name="linsym58_uneven", kind="linsym", n=58, k4=1024, k8=2048, k16=1024, steps=1, graph=False),
        # the same system on a handful of patches, two steps replayed from a graph: latency counts
        dict(name="linsym58_few", kind="linsym", n=58, k4=4, k8=8, k16=4, steps=2, graph=True),
        # relativistic run with the plain Newton start: ten steps a call
        dict(name="srhd_plain", kind="srhd", gx=16, gy=16, gz=8, p=16, guess="plain", steps=10, restart=False),
        # relativistic step on cell values drawn independently, with the trained network's start
        dict(name="srhd_learned", kind="srhd", gx=16, gy=16, gz=8, p=16, guess="learned", steps=1, restart=True),
        # loss and gradient of the guess network on one training batch
        dict(name="mlp_grad", kind="mlp", n=8192),
        # host chunks in, updated interiors out
        dict(name="offload_p6", kind="offload", k=4096, p=6, halo=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fv", "fv", "fv", "fd", "fd", "linsym", "linsym", "srhd", "srhd", "mlp", "offload"])
    if kind == "mlp":
        return dict(kind=kind, n=_log(rng, 1000, 200000))
    if kind == "offload":
        p = rng.choice([3, 5, 6, 8, 11, 16])
        return dict(kind=kind, k=_log(rng, 16, 1200000 // (p + 2) ** 3), p=p, halo=rng.choice([1, 1, 3]) if p >= 3 else 1)
    if kind == "linsym":
        k = _log(rng, 4, 1500)
        a, b = sorted((rng.randint(0, k), rng.randint(0, k)))
        return dict(kind=kind, n=rng.choice([58, 58, 58, rng.randint(5, 60)]), k4=a, k8=b - a, k16=max(1, k - b),
                    steps=rng.choice([1, 2]), graph=rng.random() < 0.5)
    if kind == "fv" and rng.random() < 0.25:
        g = _log(rng, 4, 64)
        return dict(kind=kind, dim=2, gx=g, gy=max(1, g - rng.randint(0, 3)), gz=1, p=rng.randint(5, 16), own=False,
                    storage=rng.choice(["fp64", "fp32"]), steps=rng.choice([1, 2, 10]), graph=rng.random() < 0.3)
    own = kind != "srhd" and rng.random() < 0.4
    p = rng.randint(3, 8) if own else rng.choice([16, 16, rng.randint(7, 16)])
    cells = _log(rng, 20000, 8000000 if not own else 2000000)
    k = max(1, cells // p ** 3)
    if own:
        g = (k, 1, 1)
    else:
        gz = max(1, int(round(k ** (1.0 / 3.0) * rng.uniform(0.6, 1.2))))
        gy = max(1, int(round((k / gz) ** 0.5 * rng.uniform(0.8, 1.2))))
        g = (max(1, k // (gz * gy)), gy, gz)
    c = dict(kind=kind, gx=g[0], gy=g[1], gz=g[2], p=p)
    if kind == "srhd":
        restart = rng.random() < 0.5
        return dict(c, guess=rng.choice(["plain", "learned", "warm"]), steps=1 if restart else rng.randint(1, 5),
                    restart=restart)
    c = dict(c, own=own, steps=rng.randint(1, 5 if kind == "fv" else 2), graph=rng.random() < 0.3)
    return dict(c, dim=3, storage=rng.choice(["fp64", "fp64", "fp32"])) if kind == "fv" else c


# ------------------------------------------------------------------ inputs --
# Fields live as groups [G, N, Z, Y, X] of separately periodic boxes: one box
# for a patch grid, one per patch for patches that are periodic on themselves.


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + salt)


def _modes(seed, salt, groups, shape, n_modes, kmax):
    """[groups, *shape]: per group a normalised sum of n_modes sines with wave
    vectors in {-kmax..kmax}^dim, values in [-1, 1]"""
    g = _gen(seed, salt)
    dim = len(shape)
    r = torch.rand((groups, n_modes, 2), generator=g, device=DEV, dtype=torch.float64)
    k = torch.randint(-kmax, kmax + 1, (groups, n_modes, dim), generator=g, device=DEV)
    k[..., 0] += (k.abs().sum(-1) == 0).long()
    amp = 0.1 + 0.9 * r[..., 0]
    out = torch.zeros((groups,) + tuple(shape), dtype=torch.float64, device=DEV)
    for m in range(n_modes):
        e = (amp[:, m] * torch.exp(2j * math.pi * r[:, m, 1])).reshape((groups,) + (1,) * dim)
        for d in range(dim):
            x = (torch.arange(shape[d], device=DEV, dtype=torch.float64) + 0.5) / shape[d]
            w = torch.exp(2j * math.pi * k[:, m, d, None] * x[None])
            s = [groups] + [1] * dim
            s[1 + d] = shape[d]
            e = e * w.reshape(s)
        out += e.imag
    return out / amp.sum(1).reshape((groups,) + (1,) * dim)


def _euler(rho, vel, pr):
    ke = 0.5 * rho * sum(v * v for v in vel)
    return torch.stack([rho] + [rho * v for v in vel] + [pr / (GAMMA - 1.0) + ke], dim=1)


def _euler_smooth(seed, groups, shape):
    """density and pressure in [0.5, 1.5], speeds below 0.5"""
    dim = len(shape)
    s = [_modes(seed, f, groups, shape, 8, 4) for f in range(dim + 2)]
    return _euler(1.0 + 0.5 * s[0], [0.49 / math.sqrt(3.0) * f for f in s[1:1 + dim]], 1.0 + 0.5 * s[dim + 1])


def _euler_wave(seed, groups, shape):
    """entropy wave carried by a uniform flow, with small sound waves on it
    (the unlimited fourth-order scheme keeps it smooth over long runs)"""
    dim = len(shape)
    s = [_modes(seed, f, groups, shape, 4, 2) for f in range(dim + 2)]
    u = torch.rand((dim, groups) + (1,) * dim, generator=_gen(seed, 50), device=DEV, dtype=torch.float64) * 0.6 - 0.3
    return _euler(1.0 + 0.2 * s[0], [u[d] + 0.005 * s[1 + d] for d in range(dim)], 1.0 + 0.005 * s[dim + 1])


def _euler_iid(seed, groups, shape):
    """values drawn per cell: density and pressure in [0.8, 1.2], |v_d| < 0.3"""
    r = torch.rand((len(shape) + 2, groups) + tuple(shape), generator=_gen(seed, 7), device=DEV, dtype=torch.float64)
    return _euler(0.8 + 0.4 * r[0], [0.6 * f - 0.3 for f in r[1:-1]], 0.8 + 0.4 * r[-1])


def _srhd_prims(seed, shape):
    """per cell: rho, eps log-uniform in [1e-3, 10], W uniform in [1, 10], isotropic direction"""
    u = torch.rand((5,) + tuple(shape), generator=_gen(seed, 11), device=DEV, dtype=torch.float64)
    lo, hi = math.log(1e-3), math.log(10.0)
    rho, eps, W = torch.exp(lo + (hi - lo) * u[0]), torch.exp(lo + (hi - lo) * u[1]), 1.0 + 9.0 * u[2]
    ct = 2.0 * u[3] - 1.0
    st = torch.sqrt(torch.clamp(1.0 - ct * ct, min=0.0))
    vm = torch.sqrt(1.0 - 1.0 / (W * W))
    v = [vm * st * torch.cos(2 * math.pi * u[4]), vm * st * torch.sin(2 * math.pi * u[4]), vm * ct]
    p = (GAM_R - 1.0) * rho * eps
    E = (rho + GAM_R / (GAM_R - 1.0) * p) * W * W
    return torch.stack([rho * W, E * v[0], E * v[1], E * v[2], E - p - rho * W]), p


def _box(case):
    """(groups, cells per direction with z first, patch grid) of a grid case"""
    p, dim = case["p"], case.get("dim", 3)
    if case.get("own"):
        return case["gx"], (p,) * dim, None
    grid = (case["gx"], case["gy"], case["gz"])[:dim]
    return 1, tuple(g * p for g in reversed(grid)), grid


def _initial(case, seed):
    """[G, N, (Z,) Y, X] initial state of a grid case"""
    groups, shape, _ = _box(case)
    if case["kind"] == "srhd":
        return _srhd_prims(seed, shape)[0].unsqueeze(0)
    if case["kind"] == "fd":
        return _euler_wave(seed, groups, shape)
    return _euler_iid(seed, groups, shape) if case["own"] else _euler_smooth(seed, groups, shape)


def _to_patches(q, case):
    """[G, N, (Z,) Y, X] -> the library's patch-blocked layout, flat"""
    _, _, grid = _box(case)
    if grid is None:
        return q.reshape(-1)
    p, N = case["p"], q.shape[1]
    if len(grid) == 2:
        gx, gy = grid
        return q.reshape(N, gy, p, gx, p).permute(1, 3, 0, 2, 4).reshape(-1)
    gx, gy, gz = grid
    return q.reshape(N, gz, p, gy, p, gx, p).permute(1, 3, 5, 0, 2, 4, 6).reshape(-1)


def _matrices(seed, n):
    """three symmetric matrices of spectral radius 1, and the radii"""
    rng = np.random.default_rng([int(seed), 58])
    out, rad = [], []
    for _ in range(3):
        g = rng.standard_normal((n, n))
        a = 0.5 * (g + g.T)
        a /= np.max(np.abs(np.linalg.eigvalsh(a)))
        out.append(a)
        rad.append(float(np.max(np.abs(np.linalg.eigvalsh(a)))))
    return np.stack(out), rad


def _linsym_sizes(case, seed):
    """patch sizes in shuffled order"""
    s = np.array([4] * case["k4"] + [8] * case["k8"] + [16] * case["k16"], np.int32)
    return s[np.random.default_rng([int(seed), 4]).permutation(len(s))]


def _linsym_class(case, seed, p, k):
    """[k, n, p, p, p] initial values of the k patches of size p: per unknown four modes"""
    n = case["n"]
    out = torch.empty((k, n, p, p, p), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 19) // p ** 3)
    for a in range(0, k, step):
        b = min(k, a + step)
        out[a:b] = 0.5 * _modes(seed, 100 * p + a, (b - a) * n, (p, p, p), 4, 1).reshape(b - a, n, p, p, p)
    return out


def _linsym_initial(case, seed):
    """flat state in patch order, the sizes, and per size (p, patches, values)"""
    sizes = _linsym_sizes(case, seed)
    off = np.concatenate([[0], np.cumsum(sizes.astype(np.int64) ** 3)]) * case["n"]
    flat = torch.empty(int(off[-1]), dtype=torch.float64, device=DEV)
    classes = []
    for p in (4, 8, 16):
        ks = np.nonzero(sizes == p)[0]
        if len(ks):
            q = _linsym_class(case, seed, p, len(ks))
            for j, k in enumerate(ks):
                flat[off[k]:off[k + 1]] = q[j].reshape(-1)
            classes.append((p, ks, q))
    return flat, sizes, off, classes


def _mlp_data(seed, n):
    cons, p = _srhd_prims(seed, (n,))
    return cons.contiguous(), p.contiguous()


def _network(seed, epochs=0, pairs=1 << 16, batch=4096):
    """the guess network, trained for a few epochs (or with its initial weights)"""
    rng = np.random.default_rng([int(seed), 64])
    h = 64
    w = np.concatenate([rng.standard_normal(h * 5) * math.sqrt(2 / 5), np.zeros(h),
                        rng.standard_normal(h * h) * math.sqrt(2 / h), np.zeros(h),
                        rng.standard_normal(h) / math.sqrt(h), [0.0]]).astype(np.float32)
    net = pb.Mlp(w, np.array([0.0] * 5 + [1.0] * 5 + [0.0, 1.0], np.float32))
    cons, p = _mlp_data(seed + 77, pairs)
    x, y = pb.pb_mlp_prepare(cons, p)
    net.fit_norm(x, y)
    t = net.standardise_target(y)
    per = pairs // batch
    for ep in range(epochs):
        net.train_epoch(x, t, batch, seed, ep, 3e-3, ep * per, epochs * per)
    return net


def _chunks(case, seed):
    """[K, B, B, B, 5] host halo boxes, values drawn per point, and the cell widths"""
    b = case["p"] + 2 * case["halo"]
    q = _euler_iid(seed, case["k"], (b, b, b)).permute(0, 2, 3, 4, 1).contiguous().cpu().numpy()
    return q, np.full(case["k"], 1.0 / case["p"])


# -------------------------------------------------------------------- pass --


def _batch(case, seed):
    """the patch batch of a case, its initial state on the device"""
    if case["kind"] == "linsym":
        flat, sizes, _, _ = _linsym_initial(case, seed)
        Bs, rad = _matrices(seed, case["n"])
        K, dim, N = len(sizes), 3, case["n"]
        p, dx, nbr, halo = sizes, 1.0 / sizes.astype(np.float64), I.self_periodic(K, 3), 3
        pde, prm = "linsym", I.linsym_params(Bs, rad)
    else:
        q = _initial(case, seed)
        flat, N, dim = _to_patches(q, case), q.shape[1], q.dim() - 2
        groups, shape, grid = _box(case)
        K = groups if grid is None else int(np.prod(grid))
        p = np.full(K, case["p"], np.int32)
        dx = np.full(K, 1.0 / shape[-1])
        nbr = I.self_periodic(K, dim) if grid is None else I.periodic_grid(grid)
        halo = 3 if case["kind"] == "fd" else 1
        pde, prm = ("srhd", [GAM_R, 1e-12, 50.0]) if case["kind"] == "srhd" else ("euler", [GAMMA])
    b = I.Batch(dim=dim, p=p, dx=dx, nbr=nbr, halo=halo, pde=pde, params=np.asarray(prm, np.float64), n_unknowns=N,
                state=np.zeros(flat.numel()))
    B = pb.PatchBatch(b, storage=case.get("storage", "fp64"))
    b.state = b.state[:0]
    B.bufs[0].copy_(flat)
    return B


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        net = _network(seed)
        cons, p = _mlp_data(seed, case["n"])
        x, y = pb.pb_mlp_prepare(cons, p)
        return dict(case=case, net=net, x=x, t=net.standardise_target(y))
    if kind == "offload":
        q, dx = _chunks(case, seed)
        out = np.zeros((case["k"],) + (case["p"],) * 3 + (5,))
        return dict(case=case, off=pb.Offload(case["p"], case["halo"], "euler", [GAMMA], 5), ins=list(q),
                    out=out, outs=list(out), dx=dx, dt=0.05 / case["p"])
    s = dict(case=case, B=_batch(case, seed), cur=0)
    if kind == "srhd":
        if case["guess"] == "learned":
            s["net"] = _network(1, epochs=20)
            s["B"].set_c2p_guess("learned", s["net"])
        else:
            s["B"].set_c2p_guess(case["guess"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mlp":
        return s["net"].grad(s["x"], s["t"])
    if kind == "offload":
        s["off"].fv_step(s["ins"], s["outs"], s["dx"], s["dt"])
        return s["out"]
    B = s["B"]
    if case.get("restart"):
        B.reset()
        s["cur"] = 0
    if kind in ("fd", "linsym"):
        B.fd_ko_step(cfl=CFL_FD, sigma_ko=SIGMA, n_steps=case["steps"], use_graph=case["graph"])
    else:
        B.fv_rusanov_step(cfl=CFL_FV, n_steps=case["steps"], use_graph=case.get("graph", False))
    s["cur"] ^= case["steps"] & 1
    return B.bufs[s["cur"]]


def work(case):
    """The state read once and written once per step (and per Runge-Kutta
    stage: Q, the stage value and the running sum), at the storage width.
    Operations are those of the scheme's formulas."""
    kind = case["kind"]
    if kind == "mlp":
        return dict(bytes=case["n"] * 24.0 + 2 * 4 * pb.MLP_NPARAM, flops=case["n"] * 6.0 * (5 * 64 + 64 * 64 + 64))
    if kind == "offload":
        return dict(bytes=40.0 * case["k"] * ((case["p"] + 2 * case["halo"]) ** 3 + case["p"] ** 3),
                    flops=150.0 * case["k"] * case["p"] ** 3)
    if kind == "linsym":
        cells, n = 64 * case["k4"] + 512 * case["k8"] + 4096 * case["k16"], case["n"]
        return dict(bytes=case["steps"] * cells * 16.0 * n * 8,
                    flops=case["steps"] * cells * 4.0 * (6.0 * n * n + 35.0 * n))
    groups, shape, _ = _box(case)
    cells = float(groups * int(np.prod(shape)))
    N = len(shape) + 2
    if kind == "fd":
        return dict(bytes=case["steps"] * cells * 16 * N * 8, flops=case["steps"] * cells * 1100.0)
    es = 4 if case.get("storage") == "fp32" else 8
    per = 600.0 if kind == "srhd" else 50.0 * len(shape)
    return dict(bytes=case["steps"] * cells * 2 * N * es, flops=case["steps"] * cells * per)


# --------------------------------------------------------------- reference --
# The schemes in plain torch float64 on [G, N, (Z,) Y, X] boxes; direction 0
# is x, the last axis.


def _sh(q, d, n):
    """q at the cell n steps up in direction d"""
    return torch.roll(q, -n, dims=q.dim() - 1 - d)


def _euler_terms(q, dims):
    rho, m, E = q[:, 0], [q[:, 1 + d] for d in range(dims)], q[:, dims + 1]
    pr = (GAMMA - 1.0) * (E - 0.5 * sum(x * x for x in m) / rho)
    c = torch.sqrt(GAMMA * pr / rho)
    F, lam = [], []
    for d in range(dims):
        u = m[d] / rho
        F.append(torch.stack([m[d]] + [m[e] * u + (pr if e == d else 0.0) for e in range(dims)] + [(E + pr) * u], 1))
        lam.append(u.abs() + c)
    return F, lam


def _pressure(q):
    """root of the relativistic equation of state in p, Newton from (Gamma - 1) tau"""
    D, S2, E = q[:, 0], (q[:, 1:4] ** 2).sum(1), q[:, 0] + q[:, 4]
    p = (GAM_R - 1.0) * q[:, 4]
    k = (GAM_R - 1.0) / GAM_R
    for _ in range(40):
        ep = E + p
        v2 = S2 / (ep * ep)
        w = torch.sqrt(1.0 - v2)
        f = k * (ep * (1.0 - v2) - D * w) - p
        df = k * (1.0 + v2 - D * v2 / (w * ep)) - 1.0
        p = torch.clamp(p - f / df, min=1e-30)
    return p


def _srhd_terms(q):
    pr = _pressure(q)
    Ep = q[:, 4] + q[:, 0] + pr
    v = [q[:, 1 + d] / Ep for d in range(3)]
    v2 = sum(x * x for x in v)
    cs2 = GAM_R * pr / (q[:, 0] * torch.sqrt(1.0 - v2) + GAM_R / (GAM_R - 1.0) * pr)
    cs, den = torch.sqrt(cs2), 1.0 - v2 * cs2
    F, lam = [], []
    for d in range(3):
        rt = torch.sqrt((1.0 - v2) * (1.0 - v2 * cs2 - v[d] * v[d] * (1.0 - cs2)))
        a, b = v[d] * (1.0 - cs2), cs * rt
        lam.append(torch.maximum(((a + b) / den).abs(), ((a - b) / den).abs()))
        F.append(torch.stack([q[:, 0] * v[d]] + [q[:, 1 + e] * v[d] + (pr if e == d else 0.0) for e in range(3)]
                             + [q[:, 1 + d] - q[:, 0] * v[d]], 1))
    return F, lam


def _fv(q, dx, steps, terms, dims, f32=False, dt_fixed=None):
    if f32:
        q = q.float().double()
    for _ in range(steps):
        F, lam = terms(q)
        dt = dt_fixed if dt_fixed else CFL_FV / sum(l.max() / dx for l in lam)
        acc = torch.zeros_like(q)
        for d in range(dims):
            s = torch.maximum(lam[d], _sh(lam[d], d, 1)).unsqueeze(1)
            fs = 0.5 * (F[d] + _sh(F[d], d, 1)) - 0.5 * s * (_sh(q, d, 1) - q)
            acc += fs - _sh(fs, d, -1)
        q = q - dt / dx * acc
        if f32:
            q = q.float().double()
    return q


def _d4(f, d, dx):
    return (8.0 * (_sh(f, d, 1) - _sh(f, d, -1)) - (_sh(f, d, 2) - _sh(f, d, -2))) / (12.0 * dx)


def _ko(q, dx):
    out = torch.zeros_like(q)
    for d in range(3):
        out += (_sh(q, d, 3) + _sh(q, d, -3)) - 6.0 * (_sh(q, d, 2) + _sh(q, d, -2)) \
            + 15.0 * (_sh(q, d, 1) + _sh(q, d, -1)) - 20.0 * q
    return SIGMA / (64.0 * dx) * out


def _rk4(q, dt, rhs):
    k1 = rhs(q)
    k2 = rhs(q + 0.5 * dt * k1)
    k3 = rhs(q + 0.5 * dt * k2)
    k4 = rhs(q + dt * k3)
    return q + dt / 6.0 * (k1 + 2.0 * (k2 + k3) + k4)


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if kind == "offload":
        return _exact_offload(case, seed)
    if kind == "linsym":
        flat, sizes, off, classes = _linsym_initial(case, seed)
        Bs, rad = _matrices(seed, case["n"])
        Bt = torch.from_numpy(Bs).to(DEV)
        dt = CFL_FD / sum(r / (1.0 / float(sizes.max())) for r in rad)
        for p, ks, q in classes:
            step = max(1, (1 << 18) // p ** 3)
            for a in range(0, len(ks), step):
                x = q[a:a + step]

                def rhs(y):
                    r = _ko(y, 1.0 / p)
                    for d in range(3):
                        g = _d4(y, d, 1.0 / p).transpose(0, 1).reshape(case["n"], -1)
                        r -= (Bt[d] @ g).reshape(y.transpose(0, 1).shape).transpose(0, 1)
                    return r

                for _ in range(case["steps"]):
                    x = _rk4(x, dt, rhs)
                for j, k in enumerate(ks[a:a + step]):
                    flat[off[k]:off[k + 1]] = x[j].reshape(-1)
        return flat
    q = _initial(case, seed)
    _, shape, _ = _box(case)
    dx, dims = 1.0 / shape[-1], len(shape)
    if kind == "fd":
        for _ in range(case["steps"]):
            _, lam = _euler_terms(q, 3)
            dt = CFL_FD / sum(l.max() / dx for l in lam)

            def rhs(y):
                F, _ = _euler_terms(y, 3)
                r = _ko(y, dx)
                for d in range(3):
                    r -= _d4(F[d], d, dx)
                return r

            q = _rk4(q, dt, rhs)
    elif kind == "srhd":
        q = _fv(q, dx, case["steps"], _srhd_terms, 3)
    else:
        q = _fv(q, dx, case["steps"], lambda y: _euler_terms(y, dims), dims, case["storage"] == "fp32")
    return _to_patches(q, case)


def _exact_offload(case, seed):
    b, dx = _chunks(case, seed)
    h, p = case["halo"], case["p"]
    q = torch.from_numpy(b).to(DEV).permute(0, 4, 1, 2, 3)
    q = _fv(q, float(dx[0]), 1, lambda y: _euler_terms(y, 3), 3, dt_fixed=0.05 / p)
    return q[:, :, h:h + p, h:h + p, h:h + p].permute(0, 2, 3, 4, 1).contiguous().cpu().numpy()


def _exact_mlp(case, seed):
    """loss and gradient of the network in float64, the weights as stored"""
    h = 64
    net = _network(seed)
    w, norm = net.get_params()
    net.close()
    norm = norm.astype(np.float64)
    cons, p = _mlp_data(seed, case["n"])
    E, s2 = cons[4] + cons[0], (cons[1:4] ** 2).sum(0)
    sE = torch.sqrt(s2) / E
    x = torch.stack([torch.log(cons[0] / E), sE, torch.log(1.0 - sE), torch.log(cons[4] / E),
                     torch.log((cons[4] * (cons[4] + 2.0 * cons[0]) - s2) / (E * E))], 1)
    t = (torch.log(p / E) - norm[10]) / norm[11]
    x = (x - torch.from_numpy(norm[:5]).to(DEV)) / torch.from_numpy(norm[5:10]).to(DEV)
    w = torch.from_numpy(w).to(DEV).double().requires_grad_(True)
    o = np.cumsum([0, h * 5, h, h * h, h, h, 1])
    a = [w[o[i]:o[i + 1]] for i in range(6)]
    y = torch.relu(torch.relu(x @ a[0].reshape(h, 5).T + a[1]) @ a[2].reshape(h, h).T + a[3]) @ a[4] + a[5]
    loss = ((y - t) ** 2).mean()
    loss.backward()
    return w.grad, loss.detach().reshape(1)
