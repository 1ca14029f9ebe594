"""The graph-mode batch with its default selection: a pair's image-pass variants
follow from its own levels' sizes, so its result is the single-pair one with the
same variant bit for bit, alone or among other pairs."""

import numpy as np
import pytest

from paper_1812_06765_amd import synth

pytestmark = pytest.mark.gpu

KW = dict(alpha=0.5, tau=10.0, rho=10.0, lbfgs_mem=5)
# one of every class of the rule, by voxels: 8, 11, 4, 10 and 32x32 chunks (6)
SHAPES = [(32, 40, 32), (64, 56, 48), (128, 56, 64), (128, 104, 112), (216, 224, 192)]


def _rule(m):
    ki = int(np.prod(m)) >> 10
    return 8 if ki < 96 else 11 if ki < 320 else 4 if ki < 1280 else 10 if ki < 4096 else 6


def _pairs(shapes, seed):
    import torch
    out = []
    for i, m in enumerate(shapes):
        pr = synth.blob_phantom_pair(m, seed_R=seed + 2 * i, seed_u=seed + 2 * i + 1,
                                     max_disp=1.5)
        out.append([torch.from_numpy(100.0 * v).cuda() for v in (pr.R, pr.T)])
    return [p[0] for p in out], [p[1] for p in out]


def _strip(rep):
    return [{k: v for k, v in r.items() if k != "ms"} for r in rep]


@pytest.mark.parametrize("ratio", [2, 4])
def test_default_equals_single_with_the_rules_variant(gpu_lib, ratio):
    import torch
    ngf = gpu_lib
    assert sorted({_rule(m) for m in SHAPES}) == [4, 6, 8, 10, 11]
    Rs, Ts = _pairs(SHAPES, 500)
    b = ngf.Batch(levels=1, max_iter=3, ratio=ratio, **KW)
    ys, reps = b.register(Rs, Ts)
    Js, gs = b.eval(0, ys)
    b.close()
    for i, m in enumerate(SHAPES):
        print(f"[batch rule] {m} variant {_rule(m)} ratio {ratio}", flush=True)
        with ngf.Context(levels=1, max_iter=3, ratio=ratio, **KW) as ctx:
            ctx.set_kernel(_rule(m))
            y, rep = ctx.register(Rs[i], Ts[i])
            assert torch.equal(y, ys[i]) and _strip(rep) == _strip(reps[i])
            assert rep[0]["iters"] >= 1 and rep[0]["info"] != ngf.INFO_LINESEARCH_FAIL
            J, g, _ = ctx.eval_J_grad(0, y)
            assert J == Js[i] and torch.equal(g, gs[i])


def test_default_does_not_depend_on_the_other_pairs(gpu_lib):
    """Three levels (the start points go from one to the next): each pair alone
    and among the others, and the smallest, all of whose levels take one variant,
    against the single-pair registration."""
    import torch
    ngf = gpu_lib
    shapes = [(64, 56, 48), (32, 40, 32), (96, 104, 112)]
    Rs, Ts = _pairs(shapes, 700)
    b = ngf.Batch(levels=3, max_iter=6, **KW)
    ys, reps = b.register(Rs, Ts)
    ys = [y.clone() for y in ys]
    for i, m in enumerate(shapes):
        print(f"[batch rule] {m} alone", flush=True)
        (y,), (rep,) = b.register([Rs[i]], [Ts[i]])
        assert torch.equal(y, ys[i]) and _strip(rep) == _strip(reps[i])
        for r in rep:
            assert r["iters"] >= 1 and r["info"] != ngf.INFO_LINESEARCH_FAIL, r
    b.close()
    with ngf.Context(levels=3, max_iter=6, **KW) as ctx:
        ctx.set_kernel(8)
        y, rep = ctx.register(Rs[1], Ts[1])
        assert torch.equal(y, ys[1]) and _strip(rep) == _strip(reps[1])
