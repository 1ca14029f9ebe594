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
