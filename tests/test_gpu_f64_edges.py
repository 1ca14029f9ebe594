"""The float64 evaluation where its tiles and chunks end and on every kind of
node grid, against the FP64 oracle: both compute in float64, in different
orders, so J and grad J agree to 1e-10 (sums of up to about 1e5 terms)."""

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

CASES = [
    ((4, 4, 4), 2, None, (1.0, 1.0, 1.0)),
    ((12, 16, 20), 4, None, (1.0, 0.5, 2.0)),
    ((10, 56, 74), 2, None, (1.0, 1.0, 1.0)),     # tile windows of 1024 points filled
    ((36, 60, 78), 2, None, (0.7, 1.0, 1.1)),
    ((40, 300, 36), 2, None, (1.0, 1.0, 1.0)),
    ((32, 64, 48), 2, (3, 5, 4), (1.0, 1.0, 1.0)),  # 16 points a cell
    ((37, 45, 71), 2, (10, 19, 24), (1.0, 1.0, 1.0)),  # no integer ratio
    ((50, 47, 90), 2, (11, 23, 46), (1.0, 1.5, 1.0)),
]


@pytest.mark.parametrize("m,ratio,nodes,h", CASES)
def test_f64_edges(gpu_lib, m, ratio, nodes, h):
    import torch
    ngf = gpu_lib
    print(f"[f64 edges] m={m} ratio={ratio} nodes={nodes} h={h}", flush=True)
    rng = np.random.default_rng(5)
    R = (100.0 * rng.standard_normal(m)).astype(np.float32)
    T = (100.0 * rng.standard_normal(m)).astype(np.float32)
    with ngf.Context(alpha=3.0, tau=10.0, rho=10.0, levels=1, ratio=ratio) as ctx:
        if nodes is not None:
            ctx.set_node_grid(nodes)
        ctx.build_pyramid(torch.from_numpy(R).cuda(), torch.from_numpy(T).cuda(), h)
        prob = O.Problem(R, T, h, ctx.level_info(0).my, 3.0, 10.0, 10.0)
        y = prob.identity() + 1.3 * rng.standard_normal((3,) + tuple(prob.my))
        Jo, go, _ = O.eval_J_grad(prob, y)
        yt = torch.from_numpy(y).cuda()
        J, g, _ = ctx.eval_J_grad_f64(0, yt)
        Jv, none, _ = ctx.eval_J_grad_f64(0, yt, want_grad=False)
        assert abs(J - Jo) <= 1e-10 * abs(Jo) and Jv == J and none is None
        assert np.linalg.norm(g.cpu().numpy() - go) <= 1e-10 * np.linalg.norm(go)


def test_f64_quotients_are_correctly_rounded(gpu_lib):
    """Blank images and single displaced nodes: grad J two nodes from one along an
    axis is alpha hbar^y ((u / h^y^2) / h^y^2), one quotient of another, in which
    a product with a rounded reciprocal shows.  Spacings whose squares are no
    powers of two, node positions and displacements exact."""
    import torch
    ngf = gpu_lib
    rng = np.random.default_rng(8)
    m, h, alpha = (48, 48, 48), (0.75, 1.25, 2.5), 1.0
    blank = torch.zeros(m, device="cuda")
    with ngf.Context(alpha=alpha, tau=10.0, rho=10.0, levels=1) as ctx:
        ctx.build_pyramid(blank, blank, h)
        my, hy = ctx.level_info(0).my, ctx.level_info(0).hy
        assert hy == (1.5, 2.5, 5.0)
        y = np.stack(np.meshgrid(*[np.arange(my[d]) * hy[d] for d in range(3)], indexing="ij"))
        at = [(a, b, c) for a in (4, 12, 20) for b in (4, 12, 20) for c in (4, 12, 20)]
        u = 1.0 + rng.integers(0, 2 ** 40, size=(len(at), 3)) * 2.0 ** -41
        for k, p in enumerate(at):
            y[(slice(None),) + p] += u[k]
        _, g, _ = ctx.eval_J_grad_f64(0, torch.from_numpy(y).cuda())
        g = g.cpu().numpy()
    scale = alpha * (hy[0] * hy[1] * hy[2])
    wrong = 0
    for k, p in enumerate(at):
        for c in range(3):
            for d in range(3):
                want = scale * ((u[k, c] / (hy[d] * hy[d])) / (hy[d] * hy[d]))
                for s in (-2, 2):
                    q = list(p)
                    q[d] += s
                    wrong += g[(c,) + tuple(q)] != want
    assert wrong == 0
