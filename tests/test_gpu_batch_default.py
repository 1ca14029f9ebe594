"""The graph-mode batch with its default selection, which takes the image-pass
variant and the chunks along x from all pairs of a level: each pair's
evaluation equals the single-pair one up to the rounding of sums split at other
places (J to 1e-10, the float32 gradient to 1e-5 relative L2)."""

import pytest

pytestmark = pytest.mark.gpu

# (shapes, ratio): levels whose total takes the tile kernel, the 16 x 32 and the
# 32 x 32 marching tile, with unlike lengths along x; a general node grid's pair
# cannot be in a batch
BATCHES = [
    ([(16, 24, 40), (40, 16, 16)], 2),
    ([(64, 48, 32), (32, 64, 48), (24, 96, 80), (104, 24, 40)], 2),
    ([(136, 72, 96), (40, 104, 96), (72, 96, 40), (8, 200, 72)], 2),
    ([(96, 64, 96), (32, 160, 64), (192, 32, 96)], 4),
]


@pytest.mark.parametrize("shapes,ratio", BATCHES)
def test_default_batch_eval_equals_single(gpu_lib, shapes, ratio):
    import torch
    ngf = gpu_lib
    kw = dict(alpha=0.5, tau=10.0, rho=10.0, levels=1, ratio=ratio)
    gen = torch.Generator(device="cuda").manual_seed(7)
    imgs = [[100.0 * torch.randn(m, device="cuda", generator=gen) for m in shapes]
            for _ in range(2)]
    b = ngf.Batch(max_iter=3, **kw)
    b.build(*imgs)
    ys = []
    with ngf.Context(**kw) as ctx:
        ctx.set_kernel("by_size")
        want = []
        for i, m in enumerate(shapes):
            print(f"[batch default] pair {m} ratio={ratio}", flush=True)
            ctx.build_pyramid(imgs[0][i], imgs[1][i])
            y = ctx.identity(0)
            y += 0.4 * torch.randn(y.shape, device="cuda", generator=gen)
            ys.append(y)
            J, g, _ = ctx.eval_J_grad(0, y)
            want.append((J, g))
    Js, gs = b.eval(0, ys)
    for J, g, (Jw, gw) in zip(Js, gs, want):
        assert abs(J - Jw) <= 1e-10 * abs(Jw)
        assert float((g - gw).double().norm()) <= 1e-5 * float(gw.double().norm())
    out, reps = b.register(*imgs)
    for y, rep in zip(out, reps):
        assert bool(torch.isfinite(y).all())
        assert rep[0]["info"] in (ngf.INFO_CONVERGED, ngf.INFO_MAX_ITER,
                                  ngf.INFO_LINESEARCH_FAIL)
    b.close()
