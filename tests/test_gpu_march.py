"""The fused smoothing passes of the multigrid levels against the oracle: full
rows and tiles in x, rows and planes that the boxes do not divide evenly, one to
three components, from a zero guess and from an iterate, as stop levels and
with relaxed coarsest levels.

A fixed number of cycles on random data, so every pass's rounding is compared
before the iteration contracts it: a cycle repeats the oracle's operations up to
the order of the neighbour sums, some 1e-16 of x per half-sweep, so 1e-11 of x
leaves four digits for the correction's condition.
"""
import numpy as np
import pytest

from tests.test_gpu_parity import TOL, assert_close, host, plain_ctx, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    return torch


@pytest.fixture(scope="module")
def hp():
    from paper_2503_22695_amd import hipib
    hipib.lib()
    return hipib


# (n, op, components, dt, krylov, coarse_sweeps): Helmholtz stops descending on the
# first level with 1 / dt >= 0.06 n_l^2
CASES = [(48, "poisson", 1, 1e-3, 1, 0), (64, "poisson", 3, 1e-3, 0, 0), (96, "poisson", 1, 1e-3, 0, 0),
         (128, "poisson", 1, 1e-3, 1, 0), (192, "poisson", 1, 1e-3, 1, 0), (32, "poisson", 1, 1e-3, 1, 4),
         (24, "poisson", 2, 1e-3, 0, 4), (24, "helmholtz", 3, 1e-3, 1, 0), (64, "helmholtz", 2, 1e-3, 1, 0),
         (128, "helmholtz", 3, 5e-4, 1, 0), (96, "helmholtz", 3, 1e-2, 1, 0), (128, "helmholtz", 1, 5e-3, 1, 0),
         (48, "helmholtz", 2, 5e-2, 1, 0)]


@pytest.mark.parametrize("n,op,ncomp,dt,krylov,sweeps", CASES)
def test_fused_cycles(torch_dev, hp, ref, n, op, ncomp, dt, krylov, sweeps):
    say("fused cycles", n, op, ncomp, dt, krylov, sweeps)
    rng = np.random.default_rng(1000 + n)
    b = rng.standard_normal((ncomp, n, n, n))
    b -= b.mean(axis=(1, 2, 3), keepdims=True)
    x0 = 1e-3 * rng.standard_normal(b.shape)
    poisson = op == "poisson"
    ctx = plain_ctx(hp, n, dt=dt, mg_fixed_cycles=2, mg_krylov=krylov, mg_coarse_sweeps=sweeps)
    xd = to_dev(torch_dev, x0)
    _, rr = ctx.mg_solve(hp.OP_POISSON if poisson else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    fl = ref.fluid(n, dt=dt, fixed_cycles=2, krylov=krylov if ncomp == 1 else 0, coarse_sweeps=sweeps)
    for d in range(ncomp):
        xr, _, rrr = ref.mg_solve(fl, 0.0 if poisson else 1.0 / dt, 1.0 if poisson else 0.01, poisson, b[d], x0[d])
        assert_close(f"x[{d}]", host(xd)[d], xr, TOL)
        # the residual norm that the last pass sums: b - A x rounds to some eps |b|
        assert abs(rr[d] - rrr) <= 1e-6 * rrr + 1e-13, (rr[d], rrr)


@pytest.mark.parametrize("n,op,ncomp,mixed", [(24, "poisson", 1, 0), (32, "poisson", 1, 0), (24, "helmholtz", 3, 0),
                                              (32, "helmholtz", 2, 0), (24, "poisson", 1, 1), (32, "poisson", 1, 1)])
def test_exact_level(torch_dev, hp, ref, n, op, ncomp, mixed):
    """The exact solve of a 24^3 or 32^3 level (n not and a multiple of the
    matrix tiles' 16) as the only level: one plain cycle in FP64 returns the
    solution, three of the FP32 form with FP64 residuals between them do (each
    leaves some 1e-6 of the error before it)."""
    say("exact level", n, op, ncomp, mixed)
    rng = np.random.default_rng(7 * n + ncomp)
    b = rng.standard_normal((ncomp, n, n, n))
    b -= b.mean(axis=(1, 2, 3), keepdims=True)
    poisson, dt = op == "poisson", 10.0       # (Helmholtz: viscous enough not to stop above the exact level)
    ctx = plain_ctx(hp, n, dt=dt, mg_fixed_cycles=3 if mixed else 1, mg_krylov=0,
                    precision=hp.MIXED if mixed else hp.FP64)
    xd = to_dev(torch_dev, np.zeros_like(b))
    ctx.mg_solve(hp.OP_POISSON if poisson else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    for d in range(ncomp):
        e = 4.0 * n * n * np.sin(np.pi * np.arange(n) / n) ** 2
        lam = (0.0 if poisson else 1.0 / dt) + (1.0 if poisson else 0.01) * (e[:, None, None] + e[:, None] + e)
        lam[0, 0, 0] = np.inf if poisson else lam[0, 0, 0]
        assert_close(f"x[{d}]", host(xd)[d], np.real(np.fft.ifftn(np.fft.fftn(b[d]) / lam)), TOL)


@pytest.mark.parametrize("n,mixed", [(48, 0), (64, 0), (96, 1), (128, 0), (192, 0)])
def test_open_iterations_bitwise(torch_dev, hp, n, mixed):
    """Conjugate gradients enqueued one iteration at a time (a context's first
    solve, whose length it does not know) and all together (its second, where
    an iteration leaves its steps of r and x to the next one's passes): the same
    solution to the bit, also where fewer or more iterations are enqueued than
    needed."""
    torch = torch_dev
    say("open iterations", n, mixed)
    rng = np.random.default_rng(n)
    b = rng.standard_normal((n, n, n))
    b -= b.mean()
    easy = np.cos(2 * np.pi * np.arange(n) / n) * np.ones((n, n, 1))   # an eigenvector: few iterations
    ctx = plain_ctx(hp, n, precision=hp.MIXED if mixed else hp.FP64)
    out = {}
    for name, rhs in (("first", b), ("again", b), ("easy", easy), ("short", b), ("easy after", easy)):
        x = torch.zeros((n, n, n), dtype=torch.float64, device="cuda")
        cyc, rr = ctx.mg_solve(hp.OP_POISSON, to_dev(torch, rhs), x)
        assert rr[0] <= 1e-10
        out[name] = (int(cyc[0]), host(x))
    for one, other in (("first", "again"), ("first", "short"), ("easy", "easy after")):
        assert out[one][0] == out[other][0]
        assert np.array_equal(out[one][1], out[other][1]), (one, other)


@pytest.mark.parametrize("n,mixed,over", [
    (48, 0, {}), (64, 0, {}), (96, 1, {}), (128, 0, {}), (192, 0, {}),
    (32, 0, {"mg_coarse_sweeps": 4}), (64, 0, {"mg_coarse_sweeps": 4}), (96, 1, {"mg_coarse_sweeps": 4}),
    (48, 0, {"mg_pre": 1, "mg_post": 1}), (24, 0, {}),
    (64, 0, {"mg_fixed_cycles": 3}), (64, 0, {"mg_max_cycles": 3}), (96, 1, {"mg_max_cycles": 3}),
    (64, 0, {"mg_max_cycles": 3, "mg_coarse_sweeps": 4})])
def test_batches_return_the_same(torch_dev, hp, n, mixed, over):
    """What a conjugate-gradient solve returns (solution, cycles, residual norm, or
    that it did not converge) has the same bits however its iterations were
    enqueued: one at a time in a context's first solve, all together after a
    like one, in a batch too short after an easier one, too long after a harder one (it
    stops at an iteration that others follow); exact and relaxed coarsest levels,
    stops by the tolerance, by a fixed number of cycles and by the limit."""
    torch = torch_dev
    say("batches", n, mixed, over)
    rng = np.random.default_rng(3 * n)
    b = rng.standard_normal((n, n, n))
    b -= b.mean()
    easy = np.cos(2 * np.pi * np.arange(n) / n) * np.ones((n, n, 1))   # an eigenvector: few iterations
    ctx = plain_ctx(hp, n, precision=hp.MIXED if mixed else hp.FP64, **over)
    out = []
    for rhs in (easy, easy, b, b, easy):
        x = torch.zeros((n, n, n), dtype=torch.float64, device="cuda")
        try:
            cyc, rr = ctx.mg_solve(hp.OP_POISSON, to_dev(torch, rhs), x)
            out.append((int(cyc[0]), float(rr[0]), host(x)))
        except hp.HipIBError as e:
            assert over.get("mg_max_cycles") and e.status == 4   # HIPIB_E_NOCONV
            out.append((-1, 0.0, host(x)))
    say("cycles", [o[0] for o in out])
    for one, other in ((0, 1), (0, 4), (2, 3)):
        assert out[one][:2] == out[other][:2], (one, other, out[one][:2], out[other][:2])
        assert np.array_equal(out[one][2], out[other][2]), (one, other)


@pytest.mark.parametrize("n,sigma", [(48, 0.1), (96, 0.1), (48, 1e4), (96, 645.12)])
def test_norm_of_a_converged_cycle(torch_dev, hp, n, sigma):
    """The residual norm that the last fused pass of a cycle sums, where x is as
    converged as rounding lets it be, against that of the pass that starts a
    solve (a second solve from x that has nothing to do): both colours' rounding
    is in it.  Descending cycles (sigma = 0.1) and over-relaxed ones on the
    finest level.

    Both add the terms of the same formula.  With smooth data one colour's alone
    give 0.67 to 0.71 of the norm (simulated in numpy, with and without fused
    multiply-adds), and the rounding of another order of a cell's neighbours 0.93 to
    1.01: the bound is half way."""
    torch = torch_dev
    say("norm of a converged cycle", n, sigma)
    t = 2 * np.pi * np.arange(n) / n
    b = np.cos(t)[:, None, None] * np.cos(2 * t)[:, None] + np.sin(t)
    bd = to_dev(torch, b)
    xd = torch.zeros((n, n, n), dtype=torch.float64, device="cuda")
    _, last = plain_ctx(hp, n, dt=1.0 / sigma, mg_fixed_cycles=25).mg_solve(hp.OP_HELMHOLTZ, bd, xd)
    cyc, start = plain_ctx(hp, n, dt=1.0 / sigma, mg_rtol=1e-6).mg_solve(hp.OP_HELMHOLTZ, bd, xd)
    assert cyc[0] == 0
    assert abs(last[0] / start[0] - 1.0) <= 0.15, (last[0], start[0])


@pytest.mark.parametrize("op,ncomp,dt", [("poisson", 1, 1e-3), ("helmholtz", 3, 1e-3), ("helmholtz", 3, 2e-4)])
def test_fused_cycles_256(torch_dev, hp, ref, op, ncomp, dt):
    """The boxes of 256^3 (a pass beyond the last-level cache), as test_fused_cycles;
    of three components the last one is compared."""
    n = 256
    say("fused cycles", n, op, ncomp, dt)
    rng = np.random.default_rng(n)
    b = rng.standard_normal((ncomp, n, n, n))
    b -= b.mean(axis=(1, 2, 3), keepdims=True)
    poisson = op == "poisson"
    ctx = plain_ctx(hp, n, dt=dt, mg_fixed_cycles=2)
    xd = to_dev(torch_dev, np.zeros_like(b))
    _, rr = ctx.mg_solve(hp.OP_POISSON if poisson else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    fl = ref.fluid(n, dt=dt, fixed_cycles=2)
    xr, _, rrr = ref.mg_solve(fl, 0.0 if poisson else 1.0 / dt, 1.0 if poisson else 0.01, poisson, b[-1])
    assert_close("x", host(xd)[-1], xr, TOL)
    assert abs(rr[-1] - rrr) <= 1e-6 * rrr + 1e-13, (rr, rrr)


@pytest.mark.parametrize("n,op,ncomp,dt", [(48, "poisson", 1, 1e-3), (64, "poisson", 3, 1e-3), (128, "poisson", 1, 1e-3),
                                           (192, "poisson", 1, 1e-3), (128, "helmholtz", 3, 5e-4),
                                           (96, "helmholtz", 3, 1e-2), (128, "helmholtz", 1, 5e-3)])
def test_fused_cycle_fp32(torch_dev, hp, ref, n, op, ncomp, dt):
    """One FP32 cycle of the FP64 residual against the oracle's FP64 cycle (the same
    one, the smoother being linear).  Some ten operations of four roundings a level
    and five levels at 6e-8 each: 1.2e-5 of the correction, so 2e-5."""
    say("fused cycle, FP32", n, op, ncomp, dt)
    rng = np.random.default_rng(2000 + n)
    b = rng.standard_normal((ncomp, n, n, n))
    b -= b.mean(axis=(1, 2, 3), keepdims=True)
    x0 = 1e-3 * rng.standard_normal(b.shape)
    x0 -= x0.mean(axis=(1, 2, 3), keepdims=True)
    poisson = op == "poisson"
    ctx = plain_ctx(hp, n, dt=dt, mg_fixed_cycles=1, mg_krylov=0, precision=hp.MIXED)
    xd = to_dev(torch_dev, x0)
    ctx.mg_solve(hp.OP_POISSON if poisson else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    fl = ref.fluid(n, dt=dt, fixed_cycles=1, krylov=0)
    for d in range(ncomp):
        xr, _, _ = ref.mg_solve(fl, 0.0 if poisson else 1.0 / dt, 1.0 if poisson else 0.01, poisson, b[d], x0[d])
        assert_close(f"correction[{d}]", host(xd)[d] - x0[d], xr - x0[d], 2e-5)
