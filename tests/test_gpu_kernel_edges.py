"""GPU kernels and dispatch branches at the sizes where they can go wrong (edges of tiles,
remainders, shortest and longest chains), each against the oracle or against the same steps
taken one by one."""
import numpy as np
import pytest
import torch

from conftest import relmax
from oracle import blocks as bl
from paper_2403_08063_amd import FVMultigrid, GalerkinMultigrid, Multigrid, RefinedBlocks, inputs
from paper_2403_08063_amd.solver import FUSE_BLOCKED

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


# The last of an odd number of pre-smoothing sweeps with the restriction in its pass: a V-cycle
# against its steps one by one (bitwise), on the finest level and, from 128 on, on a correction
# level that starts from 0; nu1 = 2 keeps the separate restriction.
@pytest.mark.parametrize("B,order,nu1", [(64, 2, 1), (64, 1, 3), (72, 0, 3), (72, 2, 2), (128, 2, 1), (128, 2, 3)])
def test_blocks_restriction_in_the_last_sweep(B, order, nu1):
    say(f"blocks restriction in sweep B={B} order={order} nu1={nu1}")
    rb = RefinedBlocks(B, order, nu1=nu1, nu2=1, coarse_iters=4, device=DEV)
    f, u0 = _blocks_state(rb, 3 * B + nu1)
    want = u0.clone()
    rhs, its = [f], [want]
    for l in range(rb.levels - 1):
        for _ in range(nu1):
            rb.smooth(l, rhs[l], its[l], 1)
        rhs.append(rb.restrict_residual(l, rhs[l], its[l], rb.zeros(l + 1)))
        its.append(rb.zeros(l + 1))
    for _ in range(4):
        rb.smooth(rb.levels - 1, rhs[-1], its[-1], 1)
    for l in range(rb.levels - 2, -1, -1):
        rb.prolong_correct(l, its[l + 1], its[l])
        rb.smooth(l, rhs[l], its[l], 1)
    got = rb.vcycle(f, u0.clone())
    inner = (slice(None),) + (slice(1, -1),) * 3
    # the coarsest iterations of 4^3 levels in one launch round differently: 1e-13
    scale = want[inner].abs().max()
    assert (got[inner] - want[inner]).abs().max() <= (1e-13 * scale if rb.level_B(rb.levels - 1) == 4 else 0.0)
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


def _fv_state(N, seed):
    u, _ = inputs.fv_harmonic(N)
    u[(slice(1, -1),) * 3] = np.random.default_rng(seed).uniform(-1.0, 1.0, (N,) * 3)
    return torch.from_numpy(inputs.fv_uniform(N, seed + 1, 10.0)).to(DEV), torch.from_numpy(u).to(DEV)


# Passes of two and three Jacobi sweeps with what stands around them (correction, restriction,
# zero start) for every split of nu into passes, on levels that march (256, 128), fit LDS boxes
# (64 .. 16) or lie in the one-launch tail: the oracle's operations in its order, so bitwise.
@pytest.mark.parametrize("N,nu1,nu2", [(256, 2, 3), (128, 2, 2), (128, 1, 4), (128, 5, 1), (64, 2, 3), (64, 4, 2),
                                       (32, 3, 5), (32, 0, 2), (16, 2, 0), (16, 7, 1)])
def test_fv_cycle_with_sweeps_sharing_passes(oracle, N, nu1, nu2):
    say(f"fv cycle N={N} nu=({nu1},{nu2})")
    f, u = _fv_state(N, N + 10 * nu1 + nu2)
    L = max(1, N.bit_length() - 2)
    mg = FVMultigrid(N, L, nu1=nu1, nu2=nu2, device=DEV)
    fo, want = host(f), host(u).copy()
    for _ in range(2):
        mg.vcycle(f, u)
        oracle.fv_vcycle(fo, want, L, nu1=nu1, nu2=nu2)
    got = host(u)
    assert np.array_equal(got, want), relmax(got, want)
    mg.close()


# The norm riding on the next cycle's pre-smoothing (nu1 = 2, 3): whether the tolerance or the
# limit ends the solve, the iterate is that of as many V-cycles (bitwise) and the norm that of
# its residual (another order of at most 2e6 squares: 1e-12).
@pytest.mark.parametrize("N", [32, 128])
@pytest.mark.parametrize("nu1", [1, 2, 3])
def test_fv_norm_rides_on_the_next_cycle(N, nu1):
    say(f"fv riding norm N={N} nu1={nu1}")
    f, u0 = _fv_state(N, 5 * N + nu1)
    mg = FVMultigrid(N, nu1=nu1, nu2=2, max_cycles=4, device=DEV)
    its = [u0.clone()]
    for _ in range(4):
        its.append(mg.vcycle(f, its[-1].clone()))
    _, end = mg.solve(f, u0.clone(), tol=0.0)
    norms = []
    for k in range(1, 5):
        one = FVMultigrid(N, nu1=nu1, nu2=2, max_cycles=k, device=DEV)
        got, info = one.solve(f, u0.clone(), tol=0.0)
        assert info.cycles == k and torch.equal(got, its[k])
        norms.append(info.relres)
        one.close()
    assert end.cycles == 4 and abs(end.relres - norms[3]) <= 1e-12 * norms[3]
    got, info = mg.solve(f, u0.clone(), tol=0.5 * (norms[1] + norms[2]))
    assert info.converged and info.cycles == 3 and torch.equal(got, its[3])
    assert abs(info.relres - norms[2]) <= 1e-12 * norms[2]
    mg.close()


def _plain(dim, n):
    return FUSE_BLOCKED if dim == 3 and n > 65 else False


# Every fused path (2D strips, 3D boxes and marching tiles, the LDS tail, restriction,
# prolongation, zero start) against the per-step kernels: bitwise.  Where 3D levels march, the
# blocked restriction sums in an order of its own; they are compared with the blocked kernels
# one by one, which the other flags leave bitwise unchanged.  Sizes: less than a tile, one
# node over a tile or chunk, coarsest levels that are no power of two, the tail alone.
@pytest.mark.parametrize("dim,n,variable", [(2, 5, False), (2, 21, True), (2, 65, False), (2, 129, True),
                                            (2, 241, False), (2, 513, True), (2, 1281, False), (3, 9, False),
                                            (3, 13, True), (3, 25, False), (3, 33, True), (3, 49, False),
                                            (3, 65, True), (3, 97, False), (3, 81, True), (3, 161, False)])
def test_cycle_on_fused_paths_is_bitwise(dim, n, variable):
    for nu1, nu2 in ((1, 1), (2, 2), (3, 1), (1, 4), (0, 2), (2, 0)):
        say(f"cycle dim={dim} n={n} variable={variable} nu=({nu1},{nu2})")
        g = torch.Generator(device=DEV).manual_seed(n + nu1)
        f = torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g) - 0.5
        u0 = torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g) - 0.5
        mg = Multigrid(dim, n, nu1=nu1, nu2=nu2, variable=variable, device=DEV)
        if variable:
            mg.set_coefficients(torch.exp(torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g)))
        out = []
        for flags in (True, _plain(dim, n)):
            mg.set_fusion(flags)
            u = u0.clone()
            for _ in range(2):
                mg.vcycle(f, u)
            out.append(u)
        assert torch.equal(out[0], out[1])
        mg.close()


# Solves, whose norms overlap the next cycle or ride on the last pass, against the per-step
# kernels: the same cycles and, in FP64, the same iterate (bitwise) and its norm in another order
# (up to 1e6 squares: 1e-12).  With FP32 corrections the scale that a norm sets may round another
# way, 6e-8 of a correction, which a cycle that reduces the residual by 20 makes 1e-6 of it, some
# ten cycles 1e-5: 1e-3 for the norm, and both iterates within 1e-8.
@pytest.mark.parametrize("dim,n", [(2, 65), (2, 257), (2, 1025), (3, 33), (3, 65), (3, 97)])
@pytest.mark.parametrize("precision", ["f64", "f32_ir"])
@pytest.mark.parametrize("variable", [False, True])
def test_solve_on_fused_paths(dim, n, precision, variable):
    say(f"solve dim={dim} n={n} {precision} variable={variable}")
    g = torch.Generator(device=DEV).manual_seed(n)
    f = torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g) - 0.5
    mg = Multigrid(dim, n, precision=precision, variable=variable, device=DEV)
    if variable:
        mg.set_coefficients(torch.exp(torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g)))
    res = []
    for flags in (True, _plain(dim, n)):
        mg.set_fusion(flags)
        u, info = mg.solve(f, tol=1e-9)
        res.append((u.clone(), info))
    (a, ia), (b, ib) = res
    assert ia.cycles == ib.cycles and ia.converged
    assert abs(ia.relres - ib.relres) <= (1e-12 if precision == "f64" else 1e-3) * ib.relres
    if precision == "f64":
        assert torch.equal(a, b)
    else:
        assert (a - b).abs().max() <= 1e-8 * b.abs().max()
    mg.close()


# Coarsest inverses: one unknown, sizes on both sides of the 128 unknowns that one workgroup's
# LDS takes (2D 13^2, 3D 7^3), the largest.  The residual of the direct solve is rounding
# amplified by the condition number (at most 4 / sin^2(pi h / 2) times the range of k, 5e3):
# 1e-11 of the right-hand side.
@pytest.mark.parametrize("dim,nc", [(2, 3), (3, 3), (2, 5), (3, 5), (2, 13), (2, 14), (3, 7), (3, 8), (2, 33), (3, 12)])
@pytest.mark.parametrize("variable", [False, True])
def test_coarsest_inverse_sizes(dim, nc, variable):
    say(f"coarsest inverse dim={dim} n={nc} variable={variable}")
    g = torch.Generator(device=DEV).manual_seed(nc)
    n = 2 * nc - 1
    mg = Multigrid(dim, n, levels=2, variable=variable, device=DEV)
    if variable:
        mg.set_coefficients(torch.exp(torch.rand((n,) * dim, dtype=torch.float64, device=DEV, generator=g)))
    f = torch.rand((nc,) * dim, dtype=torch.float64, device=DEV, generator=g) - 0.5
    u = mg.zeros(1)
    mg.coarsest_solve(f, u)
    inner = (slice(1, -1),) * dim
    r = mg.residual(1, f, u)[inner]
    assert r.norm() <= 1e-11 * f[inner].norm()
    mg.close()


# Galerkin levels from the smallest on, rows and planes of 17, 33 and 65 nodes, uneven sweep
# counts: V-cycles against the oracle's sparse
# products (rounding only: 1e-12 of the magnitude).
@pytest.mark.parametrize("n,levels,nu", [(5, 2, (2, 2)), (9, 3, (1, 2)), (9, 3, (2, 1)), (17, 4, (2, 2)),
                                         (33, 5, (3, 2)), (65, 6, (2, 2))])
def test_galerkin_cycle_at_edge_sizes(n, levels, nu):
    from oracle import galerkin as og
    say(f"galerkin cycle n={n} levels={levels} nu={nu}")
    k = inputs.lognormal_k(3, n, seed=4)
    f = inputs.uniform_interior(3, n, seed=9)
    mg = GalerkinMultigrid(torch.from_numpy(np.ascontiguousarray(k)).to(DEV), levels, nu1=nu[0], nu2=nu[1])
    u = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
    A = og.hierarchy(k, levels)
    uo = np.zeros((n - 2) ** 3)
    for _ in range(2):
        mg.vcycle(torch.from_numpy(np.ascontiguousarray(f)).to(DEV), u)
        uo = og.vcycle(A, og.interior(f), uo, n, nu[0], nu[1])
    want = og.embed(uo, n)
    assert np.abs(host(u) - want).max() <= 1e-12 * np.abs(want).max()
    mg.close()
