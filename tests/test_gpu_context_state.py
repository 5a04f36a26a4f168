"""What a call on a context leaves behind for the next one, and what it leaves running."""
import pytest
import torch

from paper_2403_08063_amd import FVMultigrid, GalerkinMultigrid, Multigrid, RefinedBlocks
from paper_2403_08063_amd.solver import FUSE_ALL, FUSE_TAIL, solve_noalloc

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def say(*a):
    print(*a, flush=True)


def rand(shape, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.rand(shape, dtype=torch.float64, device=DEV, generator=g) - 0.5


# A single step on a coarse level with Dirichlet data of its own, then a V-cycle, whose corrections
# have zero Dirichlet data: bitwise that of a context without the step.  Levels that march, fit LDS
# boxes and lie in the tail; one and two passes (the result in either buffer).
@pytest.mark.parametrize("N,level,sweeps", [(256, 1, 1), (128, 1, 3), (64, 1, 2), (64, 2, 4), (32, 2, 1)])
def test_fv_cycle_after_a_coarse_step(N, level, sweeps):
    say(f"fv coarse step N={N} level={level} sweeps={sweeps}")
    a, b = FVMultigrid(N, device=DEV), FVMultigrid(N, device=DEV)
    f, u = rand((N + 2,) * 3, N), rand((N + 2,) * 3, N + 1)
    a.jacobi(level, rand(a.zeros(level).shape, 2), rand(a.zeros(level).shape, 3), sweeps)
    assert torch.equal(a.vcycle(f, u.clone()), b.vcycle(f, u.clone()))
    a.close()
    b.close()


def test_fv_cycle_after_a_coarsest_solve():
    # a coarsest level of more than 16^3 cells is iterated by sweeps, here an odd number of passes
    a, b = [FVMultigrid(64, 2, coarse_iters=7, device=DEV) for _ in range(2)]
    f, u = rand((66,) * 3, 4), rand((66,) * 3, 5)
    a.coarse_solve(rand((34,) * 3, 6), rand((34,) * 3, 7))
    assert torch.equal(a.vcycle(f, u.clone()), b.vcycle(f, u.clone()))
    a.close()
    b.close()


# The same for the refined layout: levels of boxes, of passes of two sweeps, the coarsest.
@pytest.mark.parametrize("B,level,sweeps", [(16, 1, 1), (16, 1, 2), (16, 2, 3), (128, 1, 2), (12, 1, 1)])
def test_blocks_cycle_after_a_coarse_step(B, level, sweeps):
    say(f"blocks coarse step B={B} level={level} sweeps={sweeps}")
    a, b = [RefinedBlocks(B, 2, coarse_iters=5, device=DEV) for _ in range(2)]
    f, u = rand(a.zeros(0).shape, B), rand(a.zeros(0).shape, B + 1)
    a.smooth(level, rand(a.zeros(level).shape, 2), rand(a.zeros(level).shape, 3), sweeps)
    inner = (slice(None),) + (slice(1, -1),) * 3
    assert torch.equal(a.vcycle(f, u.clone())[inner], b.vcycle(f, u.clone())[inner])
    a.close()
    b.close()


# The allocation-free solve promises the results of the context solve, residual included, also
# where the norm is a sum over many workgroups' parts (2D: 4 of them at 65, hundreds at 513).
@pytest.mark.parametrize("n", [65, 129, 241, 513])
@pytest.mark.parametrize("variable", [False, True])
def test_noalloc_norms_equal_the_context_solve(n, variable):
    say(f"noalloc norms n={n} variable={variable}")
    f = rand((n, n), n)
    k = torch.exp(rand((n, n), n + 1)) if variable else None
    mg = Multigrid(2, n, variable=variable, device=DEV)
    if variable:
        mg.set_coefficients(k)
    for tol in (1e-2, 1e-6, 1e-10):
        a, ia = mg.solve(f, tol=tol)
        b, ib = solve_noalloc(f, torch.zeros_like(f), k=k, tol=tol)
        assert torch.equal(a, b) and (ia.cycles, ia.relres) == (ib.cycles, ib.relres)
    mg.close()


# A solve that ends by its tolerance after work was enqueued ahead (the first cycle's contraction is
# not predicted) returns with an idle stream: f, u and the workspace are the caller's again.
@pytest.mark.parametrize("dim,n,precision", [(2, 65, "f64"), (2, 2049, "f64"), (2, 2049, "f32_ir"), (3, 65, "f64"),
                                             (3, 65, "f32_ir"), (3, 257, "f64")])
def test_solve_returns_with_an_idle_stream(dim, n, precision):
    say(f"idle stream dim={dim} n={n} {precision}")
    mg = Multigrid(dim, n, precision=precision, device=DEV)
    f = rand((n,) * dim, n)
    for _ in range(2):
        u, info = mg.solve(f, mg.zeros(), tol=0.24)
        assert torch.cuda.current_stream(DEV).query()
        assert info.cycles == 1
    mg.close()


@pytest.mark.parametrize("N", [64, 256])
def test_fv_solve_returns_with_an_idle_stream(N):
    say(f"fv idle stream N={N}")
    mg = FVMultigrid(N, device=DEV)
    f, u = rand((N + 2,) * 3, N), torch.zeros((N + 2,) * 3, dtype=torch.float64, device=DEV)
    r0 = mg.residual_norm2(f, u) ** 0.5
    for factor, cycles in ((2.0, 0), (0.5, 1)):
        _, info = mg.solve(f, u.zero_(), tol=factor * r0)
        assert torch.cuda.current_stream(DEV).query()
        assert info.converged and info.cycles == cycles
    mg.close()


# Where the norm is a pass of its own and where it rides on the next cycle, by the contraction so far
# and the tolerance: the solve ends at the first iterate within it, bitwise that of as many V-cycles.
@pytest.mark.parametrize("N,nu1", [(32, 3), (128, 2)])
def test_fv_solve_ends_at_the_first_iterate_within_the_tolerance(N, nu1):
    say(f"fv tolerances N={N} nu1={nu1}")
    mg = FVMultigrid(N, nu1=nu1, nu2=2, max_cycles=5, device=DEV)
    f = rand((N + 2,) * 3, N)
    its, norms = [torch.zeros((N + 2,) * 3, dtype=torch.float64, device=DEV)], []
    for k in range(6):
        norms.append(mg.residual_norm2(f, its[k]) ** 0.5)
        its.append(mg.vcycle(f, its[k].clone()))
    for q in range(1, 22):  # between the norms and, with a little room, on either side of each
        tol = norms[0] * (norms[5] / norms[0]) ** (q / 20.0) * 1.02
        k = next((i for i in range(6) if norms[i] <= tol), 5)
        u, info = mg.solve(f, its[0].clone(), tol=tol)
        assert info.cycles == k and torch.equal(u, its[k])
        assert abs(info.relres - norms[k]) <= 1e-12 * norms[k]
    mg.close()


def test_blocks_solve_ends_at_the_first_iterate_within_the_tolerance():
    rb = RefinedBlocks(64, 2, nu1=3, nu2=2, coarse_iters=8, max_cycles=4, device=DEV)
    f = rand(rb.zeros(0).shape, 64)
    its, norms = [rb.zeros(0)], []
    for k in range(5):
        norms.append(rb.residual_norm2(f, its[k]) ** 0.5)
        its.append(rb.vcycle(f, its[k].clone()))
    assert all(b < a for a, b in zip(norms, norms[1:]))
    inner = (slice(None),) + (slice(1, -1),) * 3
    for q in range(-1, 13):
        tol = norms[0] * (norms[4] / norms[0]) ** (q / 11.0) * 1.02
        k = next((i for i in range(5) if norms[i] <= tol), 4)
        u, info = rb.mg_solve(f, its[0].clone(), tol)
        assert info.cycles == k and torch.equal(u[inner], its[k][inner])
        assert abs(info.relres - norms[k]) <= 1e-11 * norms[k]
    rb.close()


# A context built while a stream is captured, as a program that captures its whole setup does: every
# call of it but the ones that read norms can be recorded.  Three replays, with eager work and a
# synchronisation between them, each against the eager cycle.
@pytest.mark.parametrize("make,shape", [
    (lambda: Multigrid(3, 65, device=DEV), (65,) * 3),
    (lambda: Multigrid(2, 257, device=DEV), (257,) * 2),
    (lambda: FVMultigrid(32, device=DEV), (34,) * 3),
])
def test_context_built_under_capture(make, shape):
    say(f"capture {shape}")
    f, u0 = rand(shape, 1), rand(shape, 2)
    eager = make()
    want = eager.vcycle(f, u0.clone())
    u = u0.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mg = make()
        mg.vcycle(f, u)
    for _ in range(3):
        u.copy_(u0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(u, want)
        assert torch.equal(eager.vcycle(f, u0.clone()), want)
    eager.close()
    mg.close()


# More contexts than idle norm buffers are kept, of all four kinds, read norms, end in any order and
# are followed by others: each reads its own.
def test_norm_buffers_pass_between_contexts():
    f, g = rand((33,) * 3, 1), rand((18,) * 3, 2)
    z, zg = torch.zeros_like(f), torch.zeros_like(g)
    k = torch.exp(rand((33,) * 3, 3))
    want = float((f[1:-1, 1:-1, 1:-1] ** 2).sum()), float((g[1:-1, 1:-1, 1:-1] ** 2).sum())
    for _ in range(3):
        vertex = [Multigrid(3, 33, device=DEV) for _ in range(20)]
        cells = [FVMultigrid(16, device=DEV) for _ in range(5)]
        gal, blk = GalerkinMultigrid(k), RefinedBlocks(8, device=DEV)
        fb = rand(blk.zeros(0).shape, 4)
        for a in vertex + cells:
            s, w = (a.residual_norm2(f, z), want[0]) if isinstance(a, Multigrid) else (a.residual_norm2(g, zg), want[1])
            assert abs(s - w) <= 1e-12 * w
        assert gal.solve(f, tol=1e-6)[1].converged
        w = float((fb[:, 1:-1, 1:-1, 1:-1] ** 2).sum())
        assert abs(blk.residual_norm2(fb, blk.zeros(0)) - w) <= 1e-12 * w
        for a in vertex[::2] + [gal] + cells + [blk] + vertex[1::2]:
            a.close()


# The tail's coarsest solve by the workgroup (more than 64 unknowns), behind levels of one wave (2D
# 41: 21 and 11 nodes a side) and of the workgroup, and by one wave (the last): bitwise the per-level
# kernels.
@pytest.mark.parametrize("dim,n,levels", [(2, 41, 3), (2, 121, 3), (3, 29, 3), (3, 33, 3), (2, 37, 3)])
@pytest.mark.parametrize("variable", [False, True])
@pytest.mark.parametrize("precision", ["f64", "f32_ir"])
def test_tail_with_a_large_coarsest_level(dim, n, levels, variable, precision):
    say(f"tail dim={dim} n={n} levels={levels} variable={variable} {precision}")
    mg = Multigrid(dim, n, levels=levels, variable=variable, precision=precision, device=DEV)
    if variable:
        mg.set_coefficients(torch.exp(rand((n,) * dim, 1)))
    f, u0 = rand((n,) * dim, 2), rand((n,) * dim, 3)
    out = []
    for flags in (FUSE_ALL, FUSE_ALL & ~FUSE_TAIL):
        mg.set_fusion(flags)
        u = u0.clone()
        for _ in range(2):
            mg.vcycle(f, u)
        out.append(u)
    assert torch.equal(out[0], out[1])
    mg.close()


# Coarsest inverses of as many unknowns as one wave and four waves take, and one row more: 4, 8, 9 and
# 16, 25.  The residual is rounding amplified by the condition number (at most 4 / sin^2(pi h / 2) times
# the range of k, 5e2): 1e-12 of the right-hand side.
@pytest.mark.parametrize("dim,nc", [(2, 4), (3, 4), (2, 5), (2, 6), (2, 7)])
@pytest.mark.parametrize("variable", [False, True])
def test_coarsest_inverse_of_few_unknowns(dim, nc, variable):
    say(f"coarsest inverse dim={dim} n={nc} variable={variable}")
    n = 2 * nc - 1
    mg = Multigrid(dim, n, levels=2, variable=variable, device=DEV)
    if variable:
        mg.set_coefficients(torch.exp(rand((n,) * dim, nc)))
    f, u = rand((nc,) * dim, 2), mg.zeros(1)
    mg.coarsest_solve(f, u)
    inner = (slice(1, -1),) * dim
    assert mg.residual(1, f, u)[inner].norm() <= 1e-12 * f[inner].norm()
    mg.close()


# mg_smooth by the per-colour kernels or by passes, by sweeps, size, type and coefficient: bitwise the
# same, and neither disturbs the cycles that follow.
@pytest.mark.parametrize("dim,n,level", [(2, 65, 0), (2, 65, 1), (2, 1025, 0), (3, 33, 0), (3, 65, 0), (3, 65, 1),
                                         (3, 113, 1)])
@pytest.mark.parametrize("variable", [False, True])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_smooth_in_place_and_by_passes(dim, n, level, variable, dtype):
    say(f"smooth dim={dim} n={n} level={level} variable={variable} {dtype}")
    mg, fresh = [Multigrid(dim, n, variable=variable, precision="f32_ir", device=DEV) for _ in range(2)]
    if variable:
        for a in (mg, fresh):
            a.set_coefficients(torch.exp(rand((n,) * dim, 1)))
    shape = mg.zeros(level).shape
    f, u0 = rand(shape, 2).to(dtype), rand(shape, 3).to(dtype)
    for sweeps in (1, 2, 3, 4):
        out = []
        for flags in (True, False):
            mg.set_fusion(flags)
            out.append(mg.smooth(level, f, u0.clone(), sweeps))
        assert torch.equal(out[0], out[1]) and not torch.equal(out[0], u0)
    mg.set_fusion(True)
    f, u0 = rand((n,) * dim, 4), rand((n,) * dim, 5)
    assert torch.equal(mg.vcycle(f, u0.clone()), fresh.vcycle(f, u0.clone()))
    mg.close()
    fresh.close()


@pytest.mark.parametrize("N", [8, 16, 64, 128, 256])
def test_fv_two_sweeps_in_a_call(N):
    say(f"fv two sweeps N={N}")
    mg = FVMultigrid(N, device=DEV)
    f, u = rand((N + 2,) * 3, N), rand((N + 2,) * 3, N + 1)
    want = mg.jacobi(0, f, mg.jacobi(0, f, u.clone(), 1), 1)
    assert torch.equal(mg.jacobi(0, f, u.clone(), 2), want)
    mg.close()
