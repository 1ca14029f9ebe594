"""The grid-conversion kernels where their tiles, windows and chunks end, on
every kind of node grid, against the oracle's P and Eq. 3 gather.  Bars as in
test_gpu_parity: 1e-6 and 1e-5 of the largest entry."""

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

# (m, ratio, node grid or None)
CASES = [
    ((4, 4, 4), 2, None),
    ((6, 58, 136), 2, None),            # below the window's rows and width
    ((10, 62, 142), 2, None),           # one tile more on each axis
    ((34, 66, 130), 2, None),
    ((96, 20, 22), 2, None),
    ((12, 60, 140), 4, None),
    ((40, 124, 68), 4, None),
    ((32, 64, 96), 2, (3, 5, 7)),       # 16 points a cell: the widest index sets
    ((37, 45, 71), 2, (10, 19, 24)),    # no integer ratio
    ((21, 160, 33), 2, (11, 11, 5)),
    ((90, 91, 64), 2, (46, 12, 33)),    # an integer ratio along some axes only
]


@pytest.mark.parametrize("m,ratio,nodes", CASES)
def test_P_and_gather(gpu_lib, m, ratio, nodes):
    import torch
    ngf = gpu_lib
    print(f"[gridconv] m={m} ratio={ratio} nodes={nodes}", flush=True)
    rng = np.random.default_rng(29)
    blank = torch.zeros(m, device="cuda")
    with ngf.Context(alpha=1.0, tau=1.0, rho=1.0, levels=1, ratio=ratio) as ctx:
        if nodes is not None:
            ctx.set_node_grid(nodes)
        ctx.build_pyramid(blank, blank, (1.0, 0.5, 2.0))
        my = ctx.level_info(0).my
        y = rng.standard_normal((3,) + my).astype(np.float32)
        z = rng.standard_normal((3,) + m).astype(np.float32)
        got = ctx.apply_P(0, torch.from_numpy(y).cuda()).cpu().numpy().astype(np.float64)
        want = O.apply_P(y.astype(np.float64), m, my)
        assert np.max(np.abs(got - want)) <= 1e-6 * np.abs(want).max()
        got = ctx.apply_PT(0, torch.from_numpy(z).cuda(), "gather").cpu().numpy()
        want = O.apply_PT(z.astype(np.float64), m, my)
        assert np.max(np.abs(got.astype(np.float64) - want)) <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("m,ratio", [((8, 10, 12), 2), ((6, 70, 142), 2), ((8, 12, 16), 4),
                                     ((8, 64, 72), 4)])
def test_gather_of_an_infinity(gpu_lib, m, ratio):
    """An infinity reaches the nodes whose index sets hold its point, as an
    infinity, and no other value: at the grid's ends, next to them and inside."""
    import torch
    ngf = gpu_lib
    print(f"[gridconv] infinity m={m} ratio={ratio}", flush=True)
    rng = np.random.default_rng(30)
    blank = torch.zeros(m, device="cuda")
    with ngf.Context(alpha=1.0, tau=1.0, rho=1.0, levels=1, ratio=ratio) as ctx:
        ctx.build_pyramid(blank, blank)
        z = torch.from_numpy(rng.standard_normal((3,) + m).astype(np.float32)).cuda()
        places = [(x, y, w) for x in (0, m[0] - 1) for y in (0, ratio - 1, m[1] - 1)
                  for w in (0, ratio, m[2] - ratio, m[2] - 1)] + [tuple(v // 2 for v in m)]
        for i in places:
            for inf in (float("inf"), float("-inf")):
                one, without = torch.zeros_like(z), z.clone()
                one[(slice(None),) + i] = 1.0
                without[(slice(None),) + i] = 0.0
                bad = z.clone()
                bad[(slice(None),) + i] = inf
                reached = ctx.apply_PT(0, one, "redblack") != 0
                assert int(reached.sum()) == 24
                got, rest = ctx.apply_PT(0, bad), ctx.apply_PT(0, without)
                assert bool((got[reached] == inf).all())
                assert torch.equal(got[~reached], rest[~reached])
