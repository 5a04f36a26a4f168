"""GPU kernels and dispatch branches at the sizes where they can go wrong (edges of tiles,
remainders, shortest and longest chains), each against the oracle or against the same steps
taken one by one."""
import numpy as np
import pytest
import torch

from oracle import blocks as bl
from paper_2403_08063_amd import RefinedBlocks

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def say(*a):
    print(*a, flush=True)


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


# The coarsest iterations in one workgroup, alone in a cycle without smoothing: every order's
# ghost rule, from the single first iteration (from zero) on, odd and even counts (the two LDS
# buffers).  An iteration is a contraction whose operations differ from the oracle's in
# rounding only: a few units of 1e-16 per iteration, 1e-13 of the magnitude over 40.
@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("iters", [1, 2, 3, 40])
def test_blocks_coarsest_iterations_in_one_workgroup(order, iters):
    say(f"blocks coarsest order={order} iters={iters}")
    rng = np.random.default_rng(900 + 10 * iters + order)
    m = 10
    u0 = np.zeros((120, m, m, m))
    f = np.zeros_like(u0)
    f[:, 1:-1, 1:-1, 1:-1] = rng.uniform(-1.0, 1.0, (120, 8, 8, 8))
    rb = RefinedBlocks(8, order, nu1=0, nu2=0, coarse_iters=iters, device=DEV)
    assert rb.levels == 2
    ug = torch.from_numpy(u0.copy()).to(DEV)
    for _ in range(2):  # the second cycle starts from a nonzero iterate
        rb.vcycle(torch.from_numpy(f).to(DEV), ug)
    uo = u0.copy().reshape(-1)
    for _ in range(2):
        uo = bl.vcycle(uo, f.reshape(-1), [8, 4], order, nu1=0, nu2=0, coarse_iters=iters)
    got = host(ug)[:, 1:-1, 1:-1, 1:-1]
    want = uo.reshape(u0.shape)[:, 1:-1, 1:-1, 1:-1]
    assert np.abs(got - want).max() <= 1e-13 * np.abs(want).max()
    rb.close()
