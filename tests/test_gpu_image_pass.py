"""GPU parity of the image-pass kernels where a tile, a chunk or the halo ends:
levels that are narrower than a tile, fill it exactly or leave one node cell
over, on every axis, against the FP64 oracle.  Bars as in test_gpu_parity: J
within 1e-5 relative, grad J within 1e-4 relative L2."""

import sys

import numpy as np
import pytest

import oracle as O
from paper_1812_06765_amd import synth

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


KERNELS = ("march32x8", "march32fit", "march64fit", "march32sq", "tile3d_tiny")

# (m, h, ratio): below, at and just past the tiles' 16, 32 and 64 rows and
# columns, chunks cut to one node cell, spacings with and without an exact
# reciprocal
EDGES = [
    ((4, 4, 4), (1.0, 1.0, 1.0), 2),
    ((10, 16, 32), (1.0, 1.0, 1.0), 2),
    ((6, 18, 34), (0.9, 1.1, 2.5), 2),
    ((18, 30, 62), (1.0, 0.5, 2.0), 2),
    ((12, 34, 66), (0.75, 0.75, 1.25), 2),
    ((8, 8, 12), (1.0, 1.0, 1.0), 4),
    ((12, 36, 68), (1.1, 0.9, 0.7), 4),
    ((20, 16, 64), (1.0, 1.0, 1.0), 4),
]


@pytest.mark.parametrize("m,h,ratio", EDGES)
@pytest.mark.parametrize("amp", [0.4, 30.0])
def test_edges(gpu_lib, m, h, ratio, amp):
    """amp 30: many points outside the domain."""
    ngf = gpu_lib
    rng = np.random.default_rng(17)
    R = (100.0 * rng.standard_normal(m)).astype(np.float32)
    T = (100.0 * rng.standard_normal(m)).astype(np.float32)
    my = tuple(v // ratio + 1 for v in m)
    prob = O.Problem(R, T, h, my, 0.1, 10.0, 10.0)
    y = (prob.identity() + synth.smooth_node_perturbation(my, 6.0, amp, 5)).astype(np.float32)
    Jo, go, _ = O.eval_J_grad(prob, y.astype(np.float64))
    with ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1, ratio=ratio) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(_t(R), _t(T), h)
        for v in KERNELS:
            print(f"[edges] m={m} h={h} ratio={ratio} amp={amp} kernel={v}", flush=True)
            sys.stdout.flush()
            ctx.set_kernel(v)
            J, g, _ = ctx.eval_J_grad(0, _t(y))
            g = g.cpu().numpy().astype(np.float64)
            assert abs(J - Jo) <= 1e-5 * abs(Jo), (v, J, Jo)
            assert np.linalg.norm(g - go) <= 1e-4 * np.linalg.norm(go), v
            Jv, _, _ = ctx.eval_J_grad(0, _t(y), want_grad=False)
            assert abs(Jv - J) <= 1e-12 * abs(J), v


@pytest.mark.parametrize("variant", ["march32sq", "tile3d_tiny"])
def test_infinite_and_nan_positions(gpu_lib, variant):
    """A non-finite deformation is reported, whatever the kernel makes of it."""
    ngf = gpu_lib
    m = (16, 32, 32)
    rng = np.random.default_rng(3)
    img = _t(rng.standard_normal(m))
    for h in ((1.0, 1.0, 1.0), (0.9, 0.9, 0.9)):
        with ngf.Context(alpha=0.1, tau=1.0, rho=1.0, levels=1) as ctx:
            ctx.set_kernel(variant)
            ctx.build_pyramid(img, img, h)
            for bad in (float("nan"), float("inf"), float("-inf")):
                y = ctx.identity(0)
                y[1, 3, 4, 5] = bad
                print(f"[non-finite] h={h} value={bad}", flush=True)
                with pytest.raises(ngf.NgfError) as e:
                    ctx.eval_J_grad(0, y)
                assert e.value.status == ngf.E_NONFINITE


@pytest.mark.parametrize("h", [(1.0, 1.0, 1.0), (0.9, 1.1, 1.3)])
def test_general_pass_long_chunks(gpu_lib, h):
    """The general pass with more than 64 planes a workgroup (its tables along x
    hold 64), against the library's float64 evaluation."""
    import torch
    ngf = gpu_lib
    m, nodes = (72, 500, 509), (30, 200, 211)  # 16 x 16 tiles: one chunk along x
    gen = torch.Generator(device="cuda").manual_seed(9)
    R, T = (100.0 * torch.randn(m, device="cuda", generator=gen) for _ in range(2))
    print(f"[general] m={m} nodes={nodes} h={h}", flush=True)
    with ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1) as ctx:
        ctx.set_node_grid(nodes)
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T, h)
        y = ctx.identity(0)
        y += 0.4 * torch.randn(y.shape, device="cuda", generator=gen)
        J, g, _ = ctx.eval_J_grad(0, y)
        Jv, _, _ = ctx.eval_J_grad(0, y, want_grad=False)
        J64, g64, _ = ctx.eval_J_grad_f64(0, y.double())
    assert abs(J - J64) <= 1e-5 * abs(J64) and abs(Jv - J) <= 1e-12 * abs(J)
    assert float((g.double() - g64).norm()) <= 1e-4 * float(g64.norm())
