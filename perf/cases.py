"""Workloads of the reconstruction library on one GPU, as a user's program runs them.

The work is the chain of an initial-density reconstruction: particles are deposited on a mesh, the
mass-conservation equation is solved for the displacement potential (FP64, mixed precision, with
Anderson-accelerated cycles, or many boxes at once), the potential is mapped back to the particles,
and a loss on the potential is differentiated with respect to the density. Every kind is run over the
mesh sizes that the library supports (4, 6 or 10 cells times a power of two), powers of two and others.

Inputs are the repository's own synthetic fields: lognormal densities with the spectrum
k^-1.5 exp(-(k R_c)^2), and Zel'dovich particles displaced by two cells rms. Solves run to the default
relative residual, 1e-10; the adjoint and the batched form, whose residuals level off near 1e-10 on the
rougher fields, to 1e-9.

    listed(), draw(rng)      the cases
    prepare(case, seed)      inputs and the context a program keeps
    run(state)               one pass through the public entry points
    work(case)               bytes of inputs and outputs, and a lower bound of the arithmetic
    exact(case, seed)        the same outputs in plain torch, 64 bits
"""
import math

import torch

from paper_1709_06350_amd import autograd, mr

TOL = 1e-10
TOL_LINEAR = 1e-9   # adjoint and batched form
# Settings of the mixed-precision solve as the benchmark runs it.
MIXED = {"precision": mr.PREC_MIXED, "npre": 2, "npost": 2, "inner_cycles": 4, "ncoarse": 8}
BATCH_SIZES = (64, 96, 128)


def listed():
    return [
        # One small box: the quickest check of a configuration, bound by latency (32^3 is the smallest
        # workload of the test-suite and of the benchmark's CPU comparison).
        {"name": "solve_32", "kind": "solve", "n": 32, "sigma": 0.5, "rc": 4.0, "depth": 0},
        # An ordinary box whose side is not a power of two (coarsest mesh 6^3).
        {"name": "solve_96", "kind": "solve", "n": 96, "sigma": 0.8, "rc": 3.0, "depth": 0},
        # A production mesh with Anderson-accelerated cycles, the fastest FP64 setting.
        {"name": "anderson_256", "kind": "solve", "n": 256, "sigma": 1.0, "rc": 2.0, "depth": 2},
        # The benchmark's FP64 solve.
        {"name": "solve_512", "kind": "solve", "n": 512, "sigma": 1.0, "rc": 2.0, "depth": 0},
        # The paper's smaller mesh in mixed precision.
        {"name": "mixed_128", "kind": "mixed", "n": 128, "sigma": 1.0, "rc": 2.0},
        # The benchmark's mixed-precision solve.
        {"name": "mixed_512", "kind": "mixed", "n": 512, "sigma": 1.0, "rc": 2.0},
        # One step of a fit of the density: solve forward, adjoint backward, through autograd.
        {"name": "grad_64", "kind": "grad", "n": 64, "sigma": 0.7, "rc": 3.0},
        # The backward pass alone on a production mesh.
        {"name": "adjoint_256", "kind": "adjoint", "n": 256, "sigma": 1.0, "rc": 2.0},
        # Many independent boxes of uneven sizes on a reusable batch.
        {"name": "batch_64", "kind": "batch", "boxes": 64},
        # A full catalogue, one particle per cell, in the order of a simulation's lattice.
        {"name": "deposit_cic_256", "kind": "deposit", "n": 256, "np": 256 ** 3, "scheme": "cic", "shuffled": False},
        # A smaller, shuffled catalogue with an odd count on a mesh that is no power of two.
        {"name": "deposit_tsc_96", "kind": "deposit", "n": 96, "np": 884735, "scheme": "tsc", "shuffled": True},
        # The displacement of every particle of the full catalogue.
        {"name": "lagrangian_256", "kind": "lagrangian", "n": 256, "np": 256 ** 3, "shuffled": False, "psi": False},
    ]


def draw(rng):
    kind = rng.choice(["solve", "solve", "anderson", "mixed", "mixed", "grad", "adjoint", "batch", "deposit",
                       "deposit", "lagrangian"])
    if kind in ("solve", "anderson", "mixed", "grad", "adjoint"):
        # (4, 6, 10) x 2^k, about evenly spread over the logarithm of the side
        sides = {"solve": (16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320),
                 "anderson": (16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320),
                 "mixed": (32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384),
                 "grad": (16, 20, 24, 32, 40, 48, 64, 80, 96, 128),
                 "adjoint": (16, 24, 32, 48, 64, 80, 96, 128, 160, 192, 256)}[kind]
        n = rng.choice(sides)
        # smooth fields: the correlation length stays below a quarter of the smallest boxes
        rc = round(rng.uniform(2.0, 4.0 if n >= 32 else 3.0), 2)
        case = {"kind": kind, "n": n, "sigma": round(rng.uniform(0.5, 1.0), 3), "rc": rc}
        if kind in ("solve", "anderson"):
            case["kind"] = "solve"
            case["depth"] = rng.choice([1, 2, 3]) if kind == "anderson" else 0
        return case
    if kind == "batch":
        return {"kind": "batch", "boxes": int(round(2 ** rng.uniform(1.0, 6.0)))}
    n = rng.choice((32, 40, 48, 64, 80, 96, 128, 160, 192, 256))
    case = {"kind": kind, "n": n, "np": max(1, int(n ** 3 * 2 ** rng.uniform(-3.0, 0.0)) - rng.randrange(64)),
            "shuffled": rng.random() < 0.5}
    if kind == "deposit":
        case["scheme"] = rng.choice(["ngp", "cic", "cic", "tsc"])
    else:
        case["psi"] = rng.random() < 0.3
    return case


# ---- inputs ---------------------------------------------------------------------------------


def _wavenumbers(n):
    k = 2.0 * math.pi * torch.fft.fftfreq(n, dtype=torch.float64, device="cuda")
    kz = 2.0 * math.pi * torch.fft.rfftfreq(n, dtype=torch.float64, device="cuda")
    return k[:, None, None], k[None, :, None], kz[None, None, :]


def _gaussian_spectrum(n, rc, seed):
    """Half-complex spectrum of white noise filtered to P(k) = k^-1.5 exp(-(k rc)^2), no mean."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    w = torch.randn((n, n, n), generator=g, dtype=torch.float64, device="cuda")
    kx, ky, kz = _wavenumbers(n)
    k2 = kx * kx + ky * ky + kz * kz
    k2[0, 0, 0] = 1.0
    amp = k2.pow(-0.375) * torch.exp(-0.5 * k2 * rc * rc)
    amp[0, 0, 0] = 0.0
    return torch.fft.rfftn(w) * amp


def _lognormal(n, sigma, rc, seed):
    f = torch.fft.irfftn(_gaussian_spectrum(n, rc, seed), s=(n, n, n))
    f = torch.exp(f * (sigma / f.std(correction=0)) - 0.5 * sigma * sigma)
    return (f / f.mean() - 1.0).contiguous()


def _zeldovich(n, npart, shuffled, seed):
    """npart particles of the smallest lattice that holds them, displaced by two cells rms, and the
    potential theta of that displacement on the n^3 mesh."""
    kx, ky, kz = _wavenumbers(n)
    k2 = kx * kx + ky * ky + kz * kz
    k2[0, 0, 0] = 1.0
    phi = _gaussian_spectrum(n, 4.0, seed) / k2
    psi = torch.stack([torch.fft.irfftn(1j * kc * phi, s=(n, n, n)) for kc in (kx, ky, kz)], dim=-1)
    scale = 2.0 / psi.square().sum(-1).mean().sqrt()
    theta = (-torch.fft.irfftn(phi, s=(n, n, n)) * scale).contiguous()
    m = int(math.ceil(npart ** (1.0 / 3.0) - 1e-9))
    at = torch.arange(m ** 3, device="cuda")
    if m ** 3 > npart:   # leave particles out evenly
        at = at[(torch.arange(npart, device="cuda", dtype=torch.float64) * (m ** 3 / npart)).long()]
    q = torch.stack([at // (m * m), at // m % m, at % m], dim=-1).double() * (n / m)
    cell = q.floor().long().clamp_(0, n - 1)
    pos = torch.remainder(q + scale * psi[cell[:, 0], cell[:, 1], cell[:, 2]], float(n))
    if shuffled:
        g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
        pos = pos[torch.randperm(npart, generator=g, device="cuda")]
    return theta, pos.contiguous()


def _batch_boxes(boxes, seed):
    """(n, sigma) of each box: sizes in turn, so that every batch of three holds all of them."""
    g = torch.Generator().manual_seed(int(seed))
    sigma = 0.5 + 0.5 * torch.rand(boxes, generator=g, dtype=torch.float64)
    return [(BATCH_SIZES[b % 3], float(sigma[b])) for b in range(boxes)]


def _loss_gradient(theta):
    """dL/dtheta of the loss L = |theta|^2 / 2."""
    return (theta - theta.mean()).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "batch":
        boxes = _batch_boxes(case["boxes"], seed)
        state["delta"] = [_lognormal(n, s, 4.0, seed * 1000 + b) for b, (n, s) in enumerate(boxes)]
        state["batch"] = mr.Batch([n for n, _ in boxes], tol=TOL_LINEAR)
        return state
    n = case["n"]
    if kind in ("deposit", "lagrangian"):
        theta, state["pos"] = _zeldovich(n, case["np"], case["shuffled"], seed)
        if kind == "lagrangian":
            state["theta"] = theta
        state["ctx"] = mr.Context(n, tol=TOL)
        return state
    state["delta"] = _lognormal(n, case["sigma"], case["rc"], seed)
    tol = TOL_LINEAR if kind in ("grad", "adjoint") else TOL
    state["ctx"] = mr.Context(n, tol=tol, **(MIXED if kind == "mixed" else {}))
    if kind == "grad":
        state["delta"].requires_grad_(True)
    elif kind == "adjoint":   # a converged potential and the loss's gradient with respect to it
        with mr.Context(n, tol=1e-11) as c:
            state["theta"], _ = c.solve(state["delta"])
        state["g"] = _loss_gradient(state["theta"])
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "batch":
        return state["batch"].solve(state["delta"])[0]
    ctx = state["ctx"]
    if kind == "deposit":
        return ctx.deposit(state["pos"], scheme=case["scheme"])
    if kind == "lagrangian":
        return ctx.lagrangian(state["theta"], state["pos"], want_psi=case["psi"])
    if kind == "adjoint":
        return ctx.adjoint_solve(state["delta"], state["theta"], state["g"])[0]
    if kind == "grad":
        theta = autograd.solve(state["delta"], ctx)
        (grad,) = torch.autograd.grad(0.5 * theta.square().sum(), state["delta"])
        return theta.detach(), grad
    if case.get("depth"):
        return ctx.solve_anderson(state["delta"], depth=case["depth"])[0]
    return ctx.solve(state["delta"])[0]


def work(case):
    kind = case["kind"]
    if kind == "batch":
        cells = sum(n ** 3 for n, _ in _batch_boxes(case["boxes"], 0))
        return {"bytes": 16.0 * cells, "flops": 1000.0 * cells}
    cells = float(case["n"]) ** 3
    if kind == "deposit":
        points = {"ngp": 1, "cic": 8, "tsc": 27}[case["scheme"]]
        return {"bytes": 24.0 * case["np"] + 8.0 * cells, "flops": 4.0 * points * case["np"]}
    if kind == "lagrangian":
        return {"bytes": 48.0 * case["np"] + (32.0 if case["psi"] else 8.0) * cells, "flops": 60.0 * case["np"]}
    # read delta, write theta (adjoint: delta, theta and g in, the gradient out); every solve evaluates
    # the cubic's root, about 50 operations a cell, in some tens of relaxations
    arrays = {"solve": 2, "mixed": 2, "grad": 3, "adjoint": 4}[kind]
    return {"bytes": 8.0 * arrays * cells, "flops": 1000.0 * cells}


# ---- the same outputs in plain torch --------------------------------------------------------


def _root(p, q):
    """Largest real root of s^3 + p s + q (p <= 0): Cardano or the trigonometric form, polished by
    Newton's method; the last step carries the derivative with respect to p and q."""
    with torch.no_grad():
        disc = q * q / 4.0 + p * p * p / 27.0
        a = q.abs() / 2.0 + disc.clamp_min(0.0).sqrt()
        a = -torch.sign(q) * a.pow(1.0 / 3.0)
        one = a - p / (3.0 * torch.where(a == 0.0, torch.ones_like(a), a))
        r = (-p / 3.0).clamp_min(1e-300).sqrt()
        three = 2.0 * r * torch.cos(torch.acos((-q / (2.0 * r * r * r)).clamp(-1.0, 1.0)) / 3.0)
        s = torch.where(disc >= 0.0, one, three)
        for _ in range(3):
            s = s - (s * (s * s + p) + q) / (3.0 * s * s + p)
    return s - (s * (s * s + p) + q) / (3.0 * s * s + p).detach()


def _operator(theta, delta):
    """Laplacian of theta minus the source, with the source's mean taken out."""
    def at(*shift):
        return torch.roll(theta, [-s for s in shift], dims=(0, 1, 2))

    sx, sy, sz = at(1, 0, 0) + at(-1, 0, 0), at(0, 1, 0) + at(0, -1, 0), at(0, 0, 1) + at(0, 0, -1)
    total = sx + sy + sz
    ux, uy, uz = sx - total / 3.0, sy - total / 3.0, sz - total / 3.0
    wxy = (at(1, 1, 0) + at(-1, -1, 0) - at(1, -1, 0) - at(-1, 1, 0)) / 4.0
    wxz = (at(1, 0, 1) + at(-1, 0, -1) - at(1, 0, -1) - at(-1, 0, 1)) / 4.0
    wyz = (at(0, 1, 1) + at(0, -1, -1) - at(0, 1, -1) - at(0, -1, 1)) / 4.0
    t2 = ux * ux + uy * uy + uz * uz + 2.0 * (wxy * wxy + wxz * wxz + wyz * wyz)
    t3 = 3.0 * (ux * uy * uz - uz * wxy * wxy - uy * wxz * wxz - ux * wyz * wyz) + 6.0 * wxy * wxz * wyz
    source = _root(-4.5 * t2, 9.0 * t3 - 27.0 * (1.0 + delta)) - 3.0
    return total - 6.0 * theta - source + source.mean()


def _accelerated(residual, x, depth=8, steps=200, tol=1e-13):
    """Solves residual(x) = 0 for an operator close to the Laplacian: Fourier-preconditioned defect
    correction, each step mixed with the last ones (Anderson)."""
    n = x.shape[0]
    kx, ky, kz = _wavenumbers(n)
    symbol = 2.0 * (torch.cos(kx) + torch.cos(ky) + torch.cos(kz)) - 6.0
    symbol[0, 0, 0] = 1.0
    xs, fs, first = [], [], None
    for _ in range(steps):
        r = torch.fft.rfftn(residual(x))
        r[0, 0, 0] = 0.0
        f = -torch.fft.irfftn(r / symbol, s=(n, n, n))
        norm = float(f.norm())
        first = first or norm
        if norm <= tol * first:
            return x
        xs, fs = (xs + [x])[-depth - 1:], (fs + [f])[-depth - 1:]
        x = x + f
        if len(fs) > 1:
            df = [b - a for a, b in zip(fs, fs[1:])]
            gram = torch.tensor([[float((a * b).sum()) for a in df] for b in df], dtype=torch.float64)
            rhs = torch.tensor([float((a * f).sum()) for a in df], dtype=torch.float64)
            scale = gram.diagonal().rsqrt()
            gram = gram * scale[:, None] * scale[None, :] + 1e-13 * torch.eye(len(df), dtype=torch.float64)
            for c, a, b, d in zip((torch.linalg.solve(gram, rhs * scale) * scale).tolist(), xs, xs[1:], df):
                x = x - c * (b - a + d)
    return None


def _exact_solve(delta):
    theta = _accelerated(lambda t: _operator(t, delta), torch.zeros_like(delta))
    return None if theta is None else theta - theta.mean()


def _exact_adjoint(delta, theta, g):
    t, d = theta.detach().requires_grad_(True), delta.detach().requires_grad_(True)
    value = _operator(t, d)

    def pulled_back(lam, of):
        return torch.autograd.grad(value, of, lam, retain_graph=True)[0]

    lam = _accelerated(lambda x: pulled_back(x, t) - (g - g.mean()), torch.zeros_like(g))
    return None if lam is None else -pulled_back(lam, d)


def _axis_weights(x, scheme):
    """First mesh point and the weights of the points from there on, of one coordinate."""
    b = x.floor()
    f = x - b
    if scheme == "cic":
        return b.long(), [1.0 - f, f]
    i = torch.where(f >= 0.5, b + 1.0, b)
    if scheme == "ngp":
        return i.long(), [torch.ones_like(x)]
    d = x - i
    return i.long() - 1, [0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2]


def _points(pos, n, scheme):
    """(flat mesh index, weight) of every mesh point of every particle."""
    (bx, wx), (by, wy), (bz, wz) = (_axis_weights(pos[:, a], scheme) for a in range(3))
    for i, u in enumerate(wx):
        for j, v in enumerate(wy):
            for k, w in enumerate(wz):
                yield ((bx + i) % n * n + (by + j) % n) * n + (bz + k) % n, u * v * w


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return None
    n = case["n"]
    if kind in ("deposit", "lagrangian"):
        theta, pos = _zeldovich(n, case["np"], case["shuffled"], seed)
        if kind == "deposit":
            rho = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
            for at, w in _points(pos, n, case["scheme"]):
                rho.index_add_(0, at, w)
            return (rho * (n ** 3 / case["np"]) - 1.0).reshape(n, n, n)
        psi = torch.stack([(torch.roll(theta, -1, a) - torch.roll(theta, 1, a)) / 2.0 for a in range(3)], dim=-1)
        flat = psi.reshape(-1, 3)
        disp = torch.zeros_like(pos)
        for at, w in _points(pos, n, "cic"):
            disp += w[:, None] * flat[at]
        return disp, (psi if case["psi"] else None)
    if n > 256:   # takes too long
        return None
    delta = _lognormal(n, case["sigma"], case["rc"], seed)
    theta = _exact_solve(delta)
    if theta is None or kind in ("solve", "mixed"):
        return theta
    grad = _exact_adjoint(delta, theta, theta if kind == "grad" else _loss_gradient(theta))
    return (theta, grad) if kind == "grad" else grad
