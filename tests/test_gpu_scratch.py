"""The scratch of a context: which calls enlarge it, and what is left of it when
an allocation fails (forced from the host by the allocation fault, so that every
kernel that runs has its buffers)."""

import pytest

pytestmark = pytest.mark.gpu

KW = dict(alpha=0.1, tau=10.0, rho=10.0, levels=1)


def _images(m, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [100.0 * torch.randn(m, device="cuda", generator=gen) for _ in range(2)]


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_only_the_template_gradient_takes_room_per_voxel(gpu_lib):
    """A pair of the pyramid's own shape: J alone and grad y alone use the
    scratch that is there; grad T takes 4 bytes a voxel (33.6 MB here) once."""
    import torch
    ngf = gpu_lib
    m = (256, 256, 128)
    R, T = _images(m, 1)
    with ngf.Context(**KW) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T)
        y = ctx.identity(0)
        del_y, del_T = torch.empty_like(y), torch.empty_like(T)  # torch keeps their room
        del del_y, del_T
        n0 = _free()
        ctx.eval_pair(R, T, y, grad_y=False, grad_T=False)
        ctx.eval_pair(R, T, y, grad_T=False)
        assert n0 - _free() < 8 << 20
        ctx.eval_pair(R, T, y)
        n1 = _free()
        assert n0 - n1 >= 32 << 20
        ctx.eval_pair(R, T, y)
        assert n1 - _free() < 8 << 20


def test_no_room_for_the_sensitivities(gpu_lib):
    """Without that room both gradients are scattered (bar: float32 sums in
    another order), nothing is reported, and the pyramid's evaluation keeps its
    bits."""
    import torch
    ngf = gpu_lib
    m = (40, 48, 56)
    R, T = _images((64, 64, 64), 2)
    Rp, Tp = _images(m, 3)
    gen = torch.Generator(device="cuda").manual_seed(4)
    with ngf.Context(**KW) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T)
        y = ctx.identity(0)
        y += 0.4 * torch.randn(y.shape, device="cuda", generator=gen)
        before = ctx.eval_J_grad(0, y)
        with ngf.Context(**KW) as other:
            other.build_pyramid(Rp, Tp)
            yp = other.identity(0)
            yp += 0.4 * torch.randn(yp.shape, device="cuda", generator=gen)
            want = other.eval_pair(Rp, Tp, yp)
        ctx.eval_pair(Rp, Tp, yp, grad_y=False, grad_T=False)  # the index maps
        ctx.set_faults(ngf.Context.FAULT_ALLOC)
        got = ctx.eval_pair(Rp, Tp, yp)
        assert ctx.lib.ngf_last_error(ctx.h) == b""
        ctx.set_faults(0)
        assert abs(got[0] - want[0]) <= 1e-10 * abs(want[0])
        for g, w in zip(got[1:], want[1:]):
            assert float((g - w).double().norm()) <= 1e-5 * float(w.double().norm())
        after = ctx.eval_J_grad(0, y)
        assert after[0] == before[0] and torch.equal(after[1], before[1])


def test_failed_build_leaves_no_levels(gpu_lib):
    """A build whose images fit the storage that is there but whose partial sums
    do not: the levels it could not fill are not evaluated, and the next build
    works (bits of a fresh context)."""
    import torch
    ngf = gpu_lib
    m = (62, 62, 66)  # fewer voxels than 64^3 and more tiles
    with ngf.Context(**KW) as ctx, ngf.Context(**KW) as other:
        for c in (ctx, other):
            c.set_kernel("by_size")
        ctx.build_pyramid(*_images((64, 64, 64), 5))
        R, T = _images(m, 6)
        ctx.set_faults(ngf.Context.FAULT_ALLOC)
        with pytest.raises(ngf.NgfError) as e:
            ctx.build_pyramid(R, T)
        assert e.value.status == ngf.E_OOM
        ctx.set_faults(0)
        with pytest.raises(ngf.NgfError) as e:
            ctx.level_info(0)
        assert e.value.status == ngf.E_STATE
        ctx.build_pyramid(R, T)
        other.build_pyramid(R, T)
        y = other.identity(0) + 0.3
        a, b = ctx.eval_J_grad(0, y), other.eval_J_grad(0, y)
        assert a[0] == b[0] and torch.equal(a[1], b[1])


def test_pair_form_after_a_change_of_ratio(gpu_lib):
    """The same images on another deformation grid, which a context without a
    pyramid may be set to: the index maps are the new grid's (J as of a context of
    that ratio, the gradients up to the rounding of atomic sums)."""
    ngf = gpu_lib
    m = (32, 40, 48)
    R, T = _images(m, 7)
    with ngf.Context(**KW) as ctx:
        for ratio in (2, 4, 2):
            ctx.set_params(ratio=ratio)
            with ngf.Context(ratio=ratio, **KW) as other:
                other.build_pyramid(R, T)
                y = other.identity(0) + 0.3
                want = other.eval_pair(R, T, y)
            got = ctx.eval_pair(R, T, y)
            assert got[0] == want[0]
            for g, w in zip(got[1:], want[1:]):
                assert float((g - w).double().norm()) <= 1e-6 * float(w.double().norm())
