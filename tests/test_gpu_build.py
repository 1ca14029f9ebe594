"""The pyramid build's own paths: images in host and in device memory, at
addresses with and without 16-byte alignment, sizes with and without a
remainder, and a non-finite value at every place a thread can miss.  The images
are copies and exact float64 means: compared bit for bit."""

import pytest

pytestmark = pytest.mark.gpu


def _at(t, offset):
    """A contiguous copy of t that starts `offset` floats into its storage."""
    import torch
    buf = torch.empty(t.numel() + offset, device=t.device)
    v = buf[offset:].view(t.shape)
    v.copy_(t)
    return v


def _mean(t):
    v = t.double()
    v = v[..., 0::2] + v[..., 1::2]
    v = v[:, 0::2] + v[:, 1::2]
    return ((v[0::2] + v[1::2]) * 0.125).float()


@pytest.mark.parametrize("m,levels", [((8, 8, 8), 2), ((10, 6, 14), 1), ((40, 72, 88), 3)])
@pytest.mark.parametrize("where", ["device", "offset", "host"])
def test_images(gpu_lib, m, levels, where):
    import torch
    ngf = gpu_lib
    print(f"[build] m={m} levels={levels} {where}", flush=True)
    gen = torch.Generator().manual_seed(3)
    R, T = (100.0 * torch.randn(m, generator=gen) for _ in range(2))
    if where != "host":
        R, T = R.cuda(), T.cuda()
    if where == "offset":
        R, T = _at(R, 1), _at(T, 3)
    with ngf.Context(alpha=0.1, tau=1.0, rho=1.0, levels=levels) as ctx:
        ctx.set_kernel("by_size")
        for _ in range(2):  # and again into the same storage
            ctx.build_pyramid(R, T)
            for lev in range(levels):
                a, b = ctx.level_images(lev)
                r, t = R.cuda(), T.cuda()
                for _ in range(lev):
                    r, t = _mean(r), _mean(t)
                assert torch.equal(a, r) and torch.equal(b, t), lev


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("m,nodes", [((6, 10, 14), None), ((5, 7, 9), (3, 3, 4))])
def test_non_finite_values(gpu_lib, m, nodes, offset):
    import torch
    ngf = gpu_lib
    good = torch.randn(m, device="cuda")
    with ngf.Context(alpha=0.1, tau=1.0, rho=1.0, levels=1) as ctx:
        ctx.set_kernel("by_size")
        if nodes is not None:
            ctx.set_node_grid(nodes)
        for where in (0, 1, good.numel() // 2, good.numel() - 2, good.numel() - 1):
            for value in (float("nan"), float("inf"), float("-inf")):
                bad = good.clone()
                bad.view(-1)[where] = value
                for pair in ((bad, good), (good, bad)):
                    print(f"[build] value {value} at {where}", flush=True)
                    with pytest.raises(ngf.NgfError) as e:
                        ctx.build_pyramid(*(_at(p, offset) for p in pair))
                    assert e.value.status == ngf.E_NONFINITE
        ctx.build_pyramid(good, good)


def test_batch_reports_the_first_pair_that_failed(gpu_lib):
    import torch
    ngf = gpu_lib
    good = torch.randn((16, 16, 16), device="cuda")
    nan = good.clone()
    nan[2, 3, 4] = float("nan")
    odd = torch.zeros((15, 16, 16), device="cuda")
    b = ngf.Batch(alpha=0.1, tau=1.0, rho=1.0, levels=1, max_iter=2)
    for Rs, Ts, status, pair in (([good, good, odd], [nan, good, odd], ngf.E_NONFINITE, 0),
                                 ([good, odd, good], [good, odd, nan], ngf.E_SHAPE, 1),
                                 ([good, good], [good, nan], ngf.E_NONFINITE, 1)):
        with pytest.raises(ngf.NgfError) as e:
            b.build(Rs, Ts)
        assert e.value.status == status and f"pair {pair}" in str(e.value)
    b.build([good], [good])
    b.close()


def test_general_pass_chosen_after_the_build(gpu_lib):
    """The reference side that only the general pass reads is formed when that
    pass is chosen, and again with a new rho."""
    import torch
    ngf = gpu_lib
    gen = torch.Generator(device="cuda").manual_seed(5)
    R, T = (100.0 * torch.randn((32, 48, 40), device="cuda", generator=gen) for _ in range(2))
    with ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=2) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T)
        y = ctx.identity(1)
        y += 0.3
        for rho in (10.0, 25.0):
            ctx.set_params(rho=rho)
            ctx.set_kernel("by_size")
            J, g, _ = ctx.eval_J_grad(1, y)
            ctx.set_kernel("general")
            Jg, gg, _ = ctx.eval_J_grad(1, y)
            assert abs(Jg - J) <= 1e-5 * abs(J)
            assert float((gg - g).norm()) <= 1e-4 * float(g.norm())


@pytest.mark.parametrize("where", ["pageable", "pinned", "one of them"])
def test_memory_that_kernels_cannot_read_in_place(gpu_lib, where):
    """Image and J_dev pointers that are not this device's memory, without
    host_ptrs: copied, as every pointer was before kernels read and wrote them."""
    import ctypes

    import torch
    ngf = gpu_lib
    m = (16, 24, 20)
    print(f"[build] {where}", flush=True)
    gen = torch.Generator().manual_seed(9)
    R, T = (100.0 * torch.randn(m, generator=gen) for _ in range(2))
    if where == "pinned":
        R, T = R.pin_memory(), T.pin_memory()
    elif where == "one of them":
        T = T.cuda()
    with ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1) as ctx:
        ctx.set_kernel("by_size")
        g = ngf._grid(m, (1.0, 1.0, 1.0))
        ctx._chk(ctx.lib.ngf_build_pyramid(ctx.h, ngf._ptr(R), ngf._ptr(T), ctypes.byref(g), 0))
        a, b = ctx.level_images(0)
        assert torch.equal(a.cpu(), R.cpu()) and torch.equal(b.cpu(), T.cpu())
        y = ctx.identity(0) + 0.3
        want = ctx.eval_pair(a, b, y)[0]
        J = torch.zeros(1, dtype=torch.float64)
        J = J.pin_memory() if where == "pinned" else J
        my = (ctypes.c_int32 * 3)(*(v // 2 + 1 for v in m))
        gy = torch.empty_like(y)
        for grad in (None, ngf._ptr(gy)):
            J.zero_()
            ctx._chk(ctx.lib.ngf_eval_pair(ctx.h, ctypes.byref(g), ctypes.byref(my), ngf._ptr(a),
                                           ngf._ptr(b), ngf._ptr(y), None, None, ngf._ptr(J), grad,
                                           None))
            torch.cuda.synchronize()
            assert abs(float(J) - want) <= 1e-10 * abs(want)


def test_general_pass_chosen_under_capture(gpu_lib):
    """A choice of the general pass that is only recorded has formed nothing: an
    evaluation before the first replay, and the replays, have the values of a
    choice made outside."""
    import torch
    ngf = gpu_lib
    gen = torch.Generator(device="cuda").manual_seed(5)
    R, T = (100.0 * torch.randn((32, 48, 40), device="cuda", generator=gen) for _ in range(2))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s), ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T)
        y = ctx.identity(0) + 0.3
        g = torch.empty_like(y)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            ctx.set_kernel("general")
            ctx.eval_J_grad_async(0, y, g)
        eager = ctx.eval_J_grad(0, y)
        with ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1) as other:
            other.set_kernel("general")
            other.build_pyramid(R, T)
            want = other.eval_J_grad(0, y)
        assert eager[0] == want[0] and torch.equal(eager[1], want[1])
        for _ in range(3):
            g.zero_()
            graph.replay()
            s.synchronize()
            assert torch.equal(g, want[1])


def test_pair_form_under_capture(gpu_lib):
    """The pair form captured after a call for J alone, when there is no room yet
    for the template gradient's sensitivities, and after one with them: replays
    against the eager results (atomic sums: up to rounding)."""
    import torch
    ngf = gpu_lib
    gen = torch.Generator(device="cuda").manual_seed(6)
    R, T = (100.0 * torch.randn((32, 48, 40), device="cuda", generator=gen) for _ in range(2))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s), ngf.Context(alpha=0.1, tau=10.0, rho=10.0, levels=1) as ctx:
        ctx.set_kernel("by_size")
        ctx.build_pyramid(R, T)
        y = ctx.identity(0) + 0.3
        want = ctx.eval_J_grad(0, y)
        J = torch.zeros(1, dtype=torch.float64, device="cuda")
        ctx.eval_pair(R, T, y, grad_y=False, grad_T=False)
        for warm in (False, True):
            if warm:
                ref = ctx.eval_pair(R, T, y)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s):
                _, gy, gT = ctx.eval_pair(R, T, y, J_dev=J, sync=False)
            for _ in range(3):
                J.zero_()
                graph.replay()
                s.synchronize()
                assert abs(float(J) - want[0]) <= 1e-10 * abs(want[0])
                assert float((gy - want[1]).norm()) <= 1e-5 * float(want[1].norm())
                if warm:
                    assert float((gT - ref[2]).norm()) <= 1e-5 * float(ref[2].norm())
