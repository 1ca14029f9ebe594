"""The node pass where its tiles and chunks end, in each of its forms (small
tiles below 100 K nodes are also covered by test_gpu_image_pass), against the
library's own FP64 evaluation, itself checked against the oracle in
test_gpu_parity (against the oracle on a grid without an integer ratio).  Bars as there: J within 1e-5 relative, grad J within 1e-4
relative L2; and no single node off by more than 1e-3 of the largest entry."""

import pytest

import oracle as O

pytestmark = pytest.mark.gpu

# (m, ratio, node grid or None): node counts below, at and past multiples of
# the tiles' 4, 7, 8, 15, 17 and 33 nodes, on both sides of the form limits
# (1e5 and 1e6 nodes)
CASES = [
    ((30, 32, 66), 2, None),         # 16 x 17 x 34
    ((14, 234, 202), 2, None),       # 8 x 118 x 102, under 1e5
    ((14, 236, 236), 2, None),       # 8 x 119 x 119, over 1e5
    ((94, 82, 134), 2, None),        # 48 x 42 x 68
    ((112, 96, 100), 2, None),       # 57 x 49 x 51
    ((152, 160, 172), 2, (50, 54, 56)),
    ((36, 1084, 172), 4, None),      # 10 x 272 x 44
    ((198, 196, 200), 2, None),      # 100 x 99 x 101, under 1e6
    ((198, 196, 206), 2, None),      # 100 x 99 x 104, over 1e6
    ((4, 1168, 1188), 2, None),      # 3 x 585 x 595
    ((214, 178, 326), 2, None),      # 108 x 90 x 164
    ((214, 180, 196), 2, None),      # 108 x 91 x 99, under 1e6
]


@pytest.mark.parametrize("m,ratio,nodes", CASES)
def test_node_pass(gpu_lib, m, ratio, nodes):
    import torch
    ngf = gpu_lib
    print(f"[node pass] m={m} ratio={ratio} nodes={nodes}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(23)
    R = 100.0 * torch.randn(m, device="cuda", generator=gen)
    T = 100.0 * torch.randn(m, device="cuda", generator=gen)
    # curvature and image terms of like size
    with ngf.Context(alpha=3.0, tau=10.0, rho=10.0, levels=1, ratio=ratio) as ctx:
        if nodes is not None:
            ctx.set_node_grid(nodes)
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T, (1.0, 0.9, 1.1))
        y = ctx.identity(0)
        y += 0.3 * torch.randn(y.shape, device="cuda", generator=gen)
        J, g, _ = ctx.eval_J_grad(0, y)
        Jv, _, _ = ctx.eval_J_grad(0, y, want_grad=False)
        grads = [g]
        if nodes is None:
            J64, g64, _ = ctx.eval_J_grad_f64(0, y.double())
            grads.append(ctx.eval_J_grad_T(0, y)[1])
        else:
            prob = O.Problem(R.cpu().numpy(), T.cpu().numpy(), (1.0, 0.9, 1.1), nodes, 3.0, 10.0,
                             10.0)
            J64, g64, _ = O.eval_J_grad(prob, y.double().cpu().numpy())
            g64 = torch.from_numpy(g64).cuda()
        assert abs(J - J64) <= 1e-5 * abs(J64) and abs(Jv - J) <= 1e-12 * abs(J)
        for gi in grads:
            e = gi.double() - g64
            assert float(e.norm()) <= 1e-4 * float(g64.norm())
            assert float(e.abs().max()) <= 1e-3 * float(g64.abs().max())
