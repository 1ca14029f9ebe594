"""L-BFGS steps with every way the memory can be filled (1 to 8 pairs, the
ring not yet full, full, and dropping its oldest pair) against the FP64
oracle.  Bars as in test_gpu_parity's steps: J within 1e-4 relative and the
displacement within 1e-3, per step taken."""

import numpy as np
import pytest

import oracle as O
from paper_1812_06765_amd import synth

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("mem", [1, 2, 4, 6, 7, 8])
def test_steps_follow_oracle(gpu_lib, mem):
    ngf = gpu_lib
    m, my = (32, 32, 32), (17, 17, 17)
    pr = synth.blob_phantom_pair(m, seed_R=1, seed_u=2, max_disp=2.0)
    prob = O.Problem(pr.R, pr.T, (1.0, 1.0, 1.0), my, 1.0, 1.0, 1.0)
    X = prob.identity()
    opt = O.LBFGS(lambda v: O.eval_J_grad(prob, v)[:2], X.astype(np.float32).astype(np.float64),
                  mem=mem, h_min=1.0)
    with ngf.Context(alpha=1.0, tau=1.0, rho=1.0, levels=1, lbfgs_mem=mem) as ctx:
        ctx.build_pyramid(_t(pr.R), _t(pr.T))
        ctx.lbfgs_reset(0, _t(X))
        for k in range(10):
            J, info = ctx.lbfgs_step()
            st, _ = opt.step()
            print(f"[lbfgs] mem={mem} step {k} gpu J={J} oracle J={opt.J}", flush=True)
            assert info == ngf.INFO_OK and st == O.INFO["OK"]
            assert abs(J - opt.J) <= 1e-4 * abs(opt.J) * (k + 1)
            y, _, _ = ctx.lbfgs_get(0)
            du = y.cpu().numpy().astype(np.float64) - X
            assert np.linalg.norm(du - (opt.y - X)) <= 1e-3 * (k + 1) * np.linalg.norm(opt.y - X)
