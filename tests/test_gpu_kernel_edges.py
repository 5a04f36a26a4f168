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


def _blocks_state(rb, seed, level=0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    shape = rb.zeros(level).shape
    return [torch.rand(shape, dtype=torch.float64, device=DEV, generator=g) - 0.5 for _ in range(2)]


# Two sweeps of the layout in one pass against two calls of one sweep: the smallest and largest
# block size that takes it, sizes that fill no row of lanes, every order's ghosts, the finest
# level (stored Dirichlet ghosts) and a correction level (2 g - u); the same operations, so
# bitwise.  count 3 leaves a single sweep behind the pass.
@pytest.mark.parametrize("B,level,order", [(64, 0, 2), (66, 0, 1), (72, 0, 0), (100, 0, 2), (128, 0, 2),
                                           (128, 1, 2), (144, 1, 1)])
def test_blocks_two_sweeps_in_one_pass(B, level, order):
    say(f"blocks pair B={B} level={level} order={order}")
    rb = RefinedBlocks(B, order, device=DEV)
    f, u0 = _blocks_state(rb, B + order, level)
    for count in (2, 3):
        got, want = u0.clone(), u0.clone()
        rb.smooth(level, f, got, count)
        for _ in range(count):
            rb.smooth(level, f, want, 1)
        inner = (slice(None),) + (slice(1, -1),) * 3
        assert torch.equal(got[inner], want[inner])
    rb.close()


# The residual norm riding on the first pass of the next cycle: cycles and iterate of the solve
# as by single V-cycles (bitwise), its norm as by the norm's own pass (sums of 3e7 squares in
# another order: 1e-11), whether the limit or the norm ends it.
@pytest.mark.parametrize("nu1,nu2", [(2, 1), (3, 3)])
def test_blocks_norm_rides_on_the_next_cycle(nu1, nu2):
    say(f"blocks riding norm nu=({nu1},{nu2})")
    rb = RefinedBlocks(64, 2, nu1=nu1, nu2=nu2, coarse_iters=8, max_cycles=3, device=DEV)
    f, u0 = _blocks_state(rb, 7)
    want, norms = u0.clone(), []
    for k in range(4):
        norms.append(rb.residual_norm2(f, want) ** 0.5)
        if k == 2:
            second = want.clone()
        if k < 3:
            rb.vcycle(f, want)
    assert norms[2] < norms[1] < norms[0]
    got, info = rb.mg_solve(f, u0.clone(), 0.0)
    assert info.cycles == 3 and torch.equal(got, want)
    assert abs(info.relres - norms[3]) <= 1e-11 * norms[3]
    got, info = rb.mg_solve(f, u0.clone(), 0.5 * (norms[1] + norms[2]))
    assert info.cycles == 2 and torch.equal(got, second)
    assert abs(info.relres - norms[2]) <= 1e-11 * norms[2]
    rb.close()
