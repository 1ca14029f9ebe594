"""Performance cases: the work that a program using this package has it do.

Each case is one call of a public entry point, as such a program makes it:
the objective with its gradient or alone (``Context.eval_J_grad``), the
differentiable objective (``autograd.ngf_objective``, forward and backward),
the float64 evaluation (``Context.eval_J_grad_f64``), the grid conversion and
its adjoint (``Context.apply_P`` / ``apply_PT``), a registration
(``Context.register``) and a batch of registrations (``Batch.register``).

Inputs are CT-like pairs in Hounsfield units made on the GPU from a seed: a
body with lungs and a spine, the template being the same phantom at
x + u(x) for a smooth u of a few voxels.  Single evaluations take the setting
of ``bench.py``: 20 HU of noise, alpha = 0.1, edge parameters of 10; their
deformations are the identity plus a smooth displacement of up to 2.5 voxels,
what an optimiser holds midway.  Registrations take smooth reconstructions (5
HU) with alpha = 10 and edge parameters of 100, under which noise does not
steer the optimiser and its path is well determined.
"""

from __future__ import annotations

import math

import torch

from paper_1812_06765_amd import ngf
from paper_1812_06765_amd.autograd import ngf_objective

DEV = "cuda"


def _case(name, kind, m, h=(1.0, 1.0, 1.0), ratio=2, nodes=(0, 0, 0), levels=1, grad=True,
          iters=0, pairs=0):
    """nodes: deformation-grid nodes per axis (0: m / ratio + 1)."""
    whole = kind in ("register", "batch")
    return {"name": name, "kind": kind, "mx": m[0], "my": m[1], "mz": m[2], "hx": h[0],
            "hy": h[1], "hz": h[2], "ratio": ratio, "nx": nodes[0], "ny": nodes[1],
            "nz": nodes[2], "levels": levels, "grad": grad, "iters": iters, "pairs": pairs,
            "alpha": 10.0 if whole else 0.1, "eps": 100.0 if whole else 10.0,
            "noise": 5.0 if whole else 20.0}


def listed():
    return [
        # the smallest problem of the package (its smoke run, the coarsest
        # pyramid level of the 256^3 workload): launches and latency
        _case("eval_32", "eval", (32, 32, 32)),
        # a cropped scan: anisotropic voxels, extents that fill no tile
        _case("eval_ragged", "eval", (90, 106, 74), h=(0.9, 1.1, 2.5)),
        # the finest level of the benchmark
        _case("eval_256", "eval", (256, 256, 256)),
        # a full-resolution thorax scan on a quarter-resolution deformation grid
        _case("eval_scan_ratio4", "eval", (512, 512, 320), h=(0.75, 0.75, 1.25), ratio=4),
        # odd image sizes and a deformation grid of about three cells per node cell
        _case("eval_nodes", "eval", (191, 203, 157), nodes=(64, 68, 53)),
        # the objective alone: a line-search trial of an optimiser of one's own
        _case("value_160", "eval", (160, 128, 192), grad=False),
        # both gradients through torch.autograd, forward and backward
        _case("autograd_128", "autograd", (128, 128, 128)),
        # the float64 evaluation of precision studies
        _case("eval_f64", "f64", (128, 112, 96)),
        # dense positions of a deformation, and the adjoint of that conversion
        _case("convert_256", "convert", (256, 256, 192)),
        # the benchmark's registration with a short iteration budget
        _case("register_256", "register", (256, 256, 256), levels=4, iters=10),
        # a region of interest registered while a user waits
        _case("register_roi", "register", (64, 80, 48), levels=3, iters=12),
        # an uneven cohort in one call
        _case("batch_12", "batch", (160, 160, 160), levels=3, iters=8, pairs=12),
    ]


def _even(v, q):
    return max(q, int(round(v / q)) * q)


def draw(rng):
    """One more case of the listed kinds and ranges."""
    def extent(lo, hi, q):
        return _even(math.exp(rng.uniform(math.log(lo), math.log(hi))), q)

    def spacing():
        if rng.random() < 0.5:
            return (1.0, 1.0, 1.0)
        return tuple(round(rng.uniform(0.6, 3.0), 2) for _ in range(3))

    kind = rng.choice(["eval", "eval", "nodes", "value", "autograd", "f64", "convert",
                       "register", "batch"])
    if kind == "eval":
        r = rng.choice([2, 2, 4])
        return _drawn("eval", [extent(24, 400, r) for _ in range(3)], h=spacing(), ratio=r)
    if kind == "nodes":
        m = [extent(40, 220, 1) for _ in range(3)]
        n = [int(v / rng.uniform(2.2, 6.0)) + 1 for v in m]
        return _drawn("eval", m, h=spacing(), nodes=n)
    if kind == "value":
        return _drawn("eval", [extent(24, 300, 2) for _ in range(3)], h=spacing(), grad=False)
    if kind == "autograd":
        return _drawn("autograd", [extent(24, 180, 2) for _ in range(3)], h=spacing())
    if kind == "f64":
        return _drawn("f64", [extent(24, 140, 2) for _ in range(3)], h=spacing())
    if kind == "convert":
        r = rng.choice([2, 4])
        return _drawn("convert", [extent(24, 256, r) for _ in range(3)], ratio=r)
    if kind == "register":
        return _drawn("register", [extent(40, 200, 8) for _ in range(3)], h=spacing(), levels=3,
                      iters=rng.randint(4, 10))
    return _drawn("batch", [extent(64, 128, 8) for _ in range(3)], levels=3, iters=8,
                  pairs=rng.randint(3, 12))


def _drawn(kind, m, **kw):
    c = _case("", kind, m, **kw)
    del c["name"]
    return c


# -- inputs -----------------------------------------------------------------


def _shape(c):
    return (c["mx"], c["my"], c["mz"])


def _spacing(c):
    return (c["hx"], c["hy"], c["hz"])


def _node_shape(c):
    return tuple(n if n else m // c["ratio"] + 1
                 for n, m in zip((c["nx"], c["ny"], c["nz"]), _shape(c)))


def _waves(gen, axes, amp):
    """A smooth field (3, *shape) of about ``amp`` at its peaks: per component
    two products of sines over the unit extent.  axes: unit coordinates of the
    three axes (float32, on the GPU)."""
    f = (0.5 + 1.5 * torch.rand((3, 2, 3), generator=gen, device=DEV)).tolist()
    p = (2 * math.pi * torch.rand((3, 2, 3), generator=gen, device=DEV)).tolist()
    out = []
    for k in range(3):
        s = 0.0
        for t in range(2):
            a = [torch.sin(2 * math.pi * f[k][t][d] * axes[d] + p[k][t][d]) for d in range(3)]
            s = s + a[0][:, None, None] * a[1][None, :, None] * a[2][None, None, :]
        out.append(s)
    return torch.stack(out) * (0.45 * amp)


def _soft(d):
    return 0.5 * (1.0 + torch.tanh(d))


def _thorax(p, m):
    """CT-like values at the points p (three tensors, voxel units): air, body,
    two lungs, spine, with edges about a voxel wide."""
    q = [p[d] / m[d] for d in range(3)]

    def ball(c, s):
        r = torch.sqrt(sum(((q[d] - c[d]) / s[d]) ** 2 for d in range(3)))
        return _soft((1.0 - r) * min(s[d] * m[d] for d in range(3)))

    body = ball((0.5, 0.5, 0.5), (0.42, 0.32, 0.45))
    val = -1000.0 + 1040.0 * body
    for sx in (-0.18, 0.18):
        val = val - 890.0 * ball((0.5 + sx, 0.47, 0.5), (0.14, 0.18, 0.30)) * body
    rad = 0.06 * min(m[0], m[1])
    spine = _soft(rad - torch.sqrt((p[0] - 0.5 * m[0]) ** 2 + (p[1] - 0.72 * m[1]) ** 2))
    return val + 660.0 * spine * body


def _pair(m, gen, noise):
    ax = [torch.arange(v, device=DEV, dtype=torch.float32) + 0.5 for v in m]
    x = [ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]]
    u = _waves(gen, [a / v for a, v in zip(ax, m)], min(5.0, 0.06 * min(m)))
    out = []
    for p in (x, [x[d] + u[d] for d in range(3)]):
        v = _thorax(p, m).expand(m)
        out.append((v + noise * torch.randn(m, generator=gen, device=DEV)).contiguous())
    return out


def _deformation(m, h, n, gen):
    """Identity plus a smooth displacement (float32, node positions in mm)."""
    ax = [torch.arange(n[d], device=DEV, dtype=torch.float32) for d in range(3)]
    u = _waves(gen, [ax[d] / (n[d] - 1) for d in range(3)], 2.5)
    for d in range(3):
        shape = [1, 1, 1]
        shape[d] = n[d]
        hy = m[d] * h[d] / (n[d] - 1)
        u[d] = u[d] * h[d] + (ax[d].double() * hy).float().view(shape)
    return u.contiguous()


def _batch_shapes(c):
    """Uneven shapes around the case's: every axis scaled by its own draw."""
    g = torch.Generator().manual_seed(1234)  # the cohort's shapes are the case's, not the seed's
    f = (0.6 + 0.4 * torch.rand((c["pairs"], 3), generator=g)).tolist()
    q = c["ratio"] << (c["levels"] - 1)
    return [tuple(max(2 * q, int(v * s) // q * q) for v, s in zip(_shape(c), fs)) for fs in f]


def _context(c):
    ctx = ngf.Context(alpha=c["alpha"], tau=c["eps"], rho=c["eps"], levels=c["levels"],
                      ratio=c["ratio"], max_iter=c["iters"] or 50, lbfgs_mem=5,
                      early_stop=False)
    if c["nx"]:
        ctx.set_node_grid((c["nx"], c["ny"], c["nz"]))
    return ctx


def _inputs(c, seed):
    """What prepare() and exact() share: the tensors of a case."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    kind, m, h = c["kind"], _shape(c), _spacing(c)
    if kind == "batch":
        prs = [_pair(s, gen, c["noise"]) for s in _batch_shapes(c)]
        return {"Rs": [p[0] for p in prs], "Ts": [p[1] for p in prs]}
    if kind == "convert":
        y = _deformation(m, h, _node_shape(c), gen)
        return {"y": y, "z": torch.randn((3,) + m, generator=gen, device=DEV)}
    R, T = _pair(m, gen, c["noise"])
    if kind == "register":
        return {"R": R, "T": T}
    return {"R": R, "T": T, "y": _deformation(m, h, _node_shape(c), gen)}


def prepare(case, seed):
    s = {"case": case, **_inputs(case, seed)}
    kind, h = case["kind"], _spacing(case)
    if kind == "batch":
        s["batch"] = ngf.Batch(alpha=case["alpha"], tau=case["eps"], rho=case["eps"],
                               levels=case["levels"], ratio=case["ratio"],
                               max_iter=case["iters"], lbfgs_mem=5, early_stop=False)
        s["batch"].build(s["Rs"], s["Ts"])
        return s
    s["ctx"] = ctx = _context(case)
    if kind == "autograd":
        s["y"].requires_grad_(True)
        s["T"].requires_grad_(True)
        return s
    if kind == "convert":
        blank = torch.zeros(_shape(case), device=DEV)
        ctx.build_pyramid(blank, blank, h)
        return s
    # the timed choice of kernels and the buffers belong to the context, which
    # a program keeps; register() builds the pyramid of its pair again
    ctx.build_pyramid(s["R"], s["T"], h)
    if kind == "f64":
        s["y64"] = s["y"].double()
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "eval":
        J, g, (D, S) = s["ctx"].eval_J_grad(0, s["y"], want_grad=case["grad"])
        return {"J": J, "D": D, "S": S, "grad": g}
    if kind == "autograd":
        J = ngf_objective(s["y"], s["T"], s["R"], _spacing(case), s["ctx"])
        gy, gT = torch.autograd.grad(J, (s["y"], s["T"]))
        return {"J": J.detach(), "grad_y": gy, "grad_T": gT}
    if kind == "f64":
        J, g, (D, S) = s["ctx"].eval_J_grad_f64(0, s["y64"])
        return {"J": J, "D": D, "S": S, "grad": g}
    if kind == "convert":
        return {"P": s["ctx"].apply_P(0, s["y"]), "PT": s["ctx"].apply_PT(0, s["z"])}
    if kind == "register":
        y, _ = s["ctx"].register(s["R"], s["T"], _spacing(case))
        return {"y": y}
    ys, _ = s["batch"].register(s["Rs"], s["Ts"])
    return {"ys": ys}


# -- work -------------------------------------------------------------------


def _eval_work(N, Ny, grad=True):
    """R, T and y read once, the gradient written; about 192 flops a voxel
    (P 63, warp and its derivative 49, NGF term and v 48, adjoint 32) or 130
    for the value alone, and 40 a node component for the regulariser."""
    return (8 * N + 12 * Ny * (2 if grad else 1), (192 if grad else 130) * N + 120 * Ny)


def _register_work(m, c):
    """The pyramid, and per iteration one evaluation and the history of five
    pairs read for the direction and for the new pair's inner products."""
    b = f = 0
    for lev in range(c["levels"]):
        N = math.prod(v >> lev for v in m)
        Ny = math.prod((v >> lev) // c["ratio"] + 1 for v in m)
        eb, ef = _eval_work(N, Ny)
        pairs = sum(min(k, 5) for k in range(c["iters"])) * 2
        b += 8 * N + (c["iters"] + 1) * eb + 12 * Ny * (2 * pairs + 8 * c["iters"])
        f += (c["iters"] + 1) * ef + 3 * Ny * 8 * pairs
    return b, f


def work(case):
    m, kind = _shape(case), case["kind"]
    N, Ny = math.prod(m), math.prod(_node_shape(case))
    if kind == "eval":
        b, f = _eval_work(N, Ny, case["grad"])
    elif kind == "autograd":  # the value, then both gradients
        b, f = 8 * N + 12 * Ny + 12 * N + 24 * Ny, (130 + 192 + 24) * N + 240 * Ny
    elif kind == "f64":
        b, f = 8 * N + 48 * Ny, 192 * N + 120 * Ny
    elif kind == "convert":
        b, f = 24 * (N + Ny), (63 + 42) * N
    elif kind == "register":
        b, f = _register_work(m, case)
    else:
        w = [_register_work(s, case) for s in _batch_shapes(case)]
        b, f = sum(v[0] for v in w), sum(v[1] for v in w)
    return {"bytes": b, "flops": f}


# -- the same in float64, plain torch ----------------------------------------


def _matrix(m, n):
    """Interpolation from n nodes to m cell centres along one axis, (m, n)."""
    x = (torch.arange(m, dtype=torch.float64, device=DEV) + 0.5) * (n - 1) / m
    num = (2 * torch.arange(m, device=DEV) + 1) * (n - 1)
    j = num // (2 * m)
    w1 = (num - j * 2 * m).double() / (2 * m)
    A = torch.zeros((m, n), dtype=torch.float64, device=DEV)
    i = torch.arange(m, device=DEV)
    A[i, j] = 1.0 - w1
    A[i, j + 1] = w1
    assert float((A @ torch.arange(n, dtype=torch.float64, device=DEV) - x).abs().max()) < 1e-9
    return A


def _along(v, mats):
    """mats[d] applied along axis d of v (three axes)."""
    v = torch.tensordot(mats[0], v, dims=([1], [0]))
    v = torch.tensordot(mats[1], v, dims=([1], [1])).movedim(0, 1)
    return torch.tensordot(v, mats[2], dims=([2], [1])).contiguous()


def _diff(u, d, h):
    k = torch.arange(u.shape[d], device=DEV)
    up = u.index_select(d, (k + 1).clamp_(max=u.shape[d] - 1))
    return (up - u.index_select(d, (k - 1).clamp_(min=0))) / (2.0 * h)


def _diff_adjoint(w, d, h):
    m = w.shape[d]
    first, last = w.narrow(d, 0, 1), w.narrow(d, m - 1, 1)
    prev = torch.cat([-first, w.narrow(d, 0, m - 1)], d)
    nxt = torch.cat([w.narrow(d, 1, m - 1), -last], d)
    return (prev - nxt) / (2.0 * h)


def _laplace(u, hy):
    out = torch.zeros_like(u)
    for d in range(3):
        k = torch.arange(u.shape[d], device=DEV)
        up = u.index_select(d, (k + 1).clamp_(max=u.shape[d] - 1))
        dn = u.index_select(d, (k - 1).clamp_(min=0))
        out += (up - 2.0 * u + dn) / (hy[d] * hy[d])
    return out


def _objective(R, T, y, m, h, n, alpha, eps, grad=True, grad_T=False):
    """J, D, S and the gradients in float64."""
    mats = [_matrix(m[d], n[d]) for d in range(3)]
    y = y.double()
    i0, f, s = [], [], []
    for d in range(3):
        xi = _along(y[d], mats) / h[d] - 0.5
        s.append((xi >= 0) & (xi <= m[d] - 1))
        xi.clamp_(0, m[d] - 1)
        i0.append(xi.floor().clamp_(max=m[d] - 2))
        f.append(xi - i0[d])
        del xi
    base = ((i0[0].long() * m[1] + i0[1].long()) * m[2] + i0[2].long()).reshape(-1)
    del i0
    Tv = T.reshape(-1).double()
    corner = {(a, b, c): (a * m[1] + b) * m[2] + c
              for a in (0, 1) for b in (0, 1) for c in (0, 1)}

    def weight(a, d):
        return f[d] if a else 1.0 - f[d]

    Ty = torch.zeros(m, dtype=torch.float64, device=DEV)
    dT = [torch.zeros(m, dtype=torch.float64, device=DEV) for _ in range(3)] if grad else []
    for k, o in corner.items():
        v = Tv[base + o].view(m)
        Ty += weight(k[0], 0) * weight(k[1], 1) * weight(k[2], 2) * v
        for d in range(3 if grad else 0):
            p, q = [e for e in range(3) if e != d]
            dT[d] += (1.0 if k[d] else -1.0) * weight(k[p], p) * weight(k[q], q) * v
        del v
    gT = [_diff(Ty, d, h[d]) for d in range(3)]
    Rd = R.double()
    gR = [_diff(Rd, d, h[d]) for d in range(3)]
    nT = sum(g * g for g in gT) + eps * eps
    nR = sum(g * g for g in gR) + eps * eps
    c = sum(a * b for a, b in zip(gT, gR)) + eps * eps
    hbar = h[0] * h[1] * h[2]
    D = 0.5 * hbar * float((1.0 - c * c / (nT * nR)).sum())
    hy = [m[d] * h[d] / (n[d] - 1) for d in range(3)]
    hbary = hy[0] * hy[1] * hy[2]
    u = y.clone()
    for d in range(3):
        shape = [1, 1, 1]
        shape[d] = n[d]
        u[d] -= (torch.arange(n[d], dtype=torch.float64, device=DEV) * hy[d]).view(shape)
    Au = [_laplace(u[k], hy) for k in range(3)]
    S = 0.5 * hbary * sum(float((a * a).sum()) for a in Au)
    out = {"J": D + alpha * S, "D": D, "S": S}
    if not grad:
        return out
    k = -hbar * c / (nT * nR)
    ct = c / nT
    e = sum(_diff_adjoint(k * (gR[d] - ct * gT[d]), d, h[d]) for d in range(3))
    del gT, gR, nT, nR, c, k, ct
    back = [a.t().contiguous() for a in mats]
    out["grad"] = torch.stack([_along(e * dT[d] * s[d] / h[d], back)
                               + alpha * hbary * _laplace(Au[d], hy) for d in range(3)])
    if grad_T:
        g = torch.zeros(T.numel(), dtype=torch.float64, device=DEV)
        for q, o in corner.items():
            w = weight(q[0], 0) * weight(q[1], 1) * weight(q[2], 2) * e
            g.index_add_(0, base + o, w.reshape(-1))
        out["grad_T"] = g.view(m)
    return out


def exact(case, seed):
    """run()'s answer in float64.  None for registrations: an optimiser's path
    has no closed value."""
    kind = case["kind"]
    if kind in ("register", "batch"):
        return None
    m, h, n = _shape(case), _spacing(case), _node_shape(case)
    s = _inputs(case, seed)
    if kind == "convert":
        mats = [_matrix(m[d], n[d]) for d in range(3)]
        back = [a.t().contiguous() for a in mats]
        return {"P": torch.stack([_along(s["y"][d].double(), mats) for d in range(3)]),
                "PT": torch.stack([_along(s["z"][d].double(), back) for d in range(3)])}
    o = _objective(s["R"], s["T"], s["y"], m, h, n, case["alpha"], case["eps"], case["grad"],
                   kind == "autograd")
    if kind == "autograd":
        return {"J": torch.tensor(o["J"], dtype=torch.float64), "grad_y": o["grad"],
                "grad_T": o["grad_T"]}
    return {"J": o["J"], "D": o["D"], "S": o["S"], "grad": o.get("grad")}
