"""The separate smoothing, residual and transfer kernels of the multigrid levels
against the oracle: every smoothing count other than two before and two after the
coarse-grid correction (which runs in fused passes), none on one side among them.

As for the fused passes, a fixed number of cycles on random data and 1e-11 of x: a
cycle repeats the oracle's operations up to the order of the neighbour sums.  The
FP32 cycles are compared where they have converged.
"""
import numpy as np
import pytest

from tests.test_gpu_parity import TOL, assert_close, host, plain_ctx, rel, say, to_dev

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


# (n, op, components, dt, krylov, coarse_sweeps, pre, post): Helmholtz stops descending on
# the first level with 1 / dt >= 0.06 n_l^2 (the second one at 128^3 with 4e-3)
CASES = [(48, "poisson", 1, 1e-3, 1, 0, 1, 1), (64, "poisson", 1, 1e-3, 1, 0, 3, 2), (64, "poisson", 1, 1e-3, 1, 4, 1, 3),
         (64, "poisson", 3, 1e-3, 0, 0, 2, 1), (48, "poisson", 1, 1e-3, 0, 0, 0, 2), (48, "poisson", 2, 1e-3, 0, 4, 2, 0),
         (96, "poisson", 1, 1e-3, 1, 0, 2, 0), (64, "helmholtz", 3, 1e-3, 1, 0, 1, 1), (128, "helmholtz", 2, 4e-3, 1, 0, 3, 1),
         (96, "helmholtz", 3, 1e-2, 1, 0, 3, 3), (48, "helmholtz", 1, 5e-2, 1, 0, 0, 1)]


def problem(n, op, ncomp, dt):
    rng = np.random.default_rng(500 + n + ncomp)
    b = rng.standard_normal((ncomp, n, n, n))
    b -= b.mean(axis=(1, 2, 3), keepdims=True)
    return b, 1e-3 * rng.standard_normal(b.shape), (0.0, 1.0, True) if op == "poisson" else (1.0 / dt, 0.01, False)


@pytest.mark.parametrize("n,op,ncomp,dt,krylov,sweeps,pre,post", CASES)
def test_separate_cycles(torch_dev, hp, ref, n, op, ncomp, dt, krylov, sweeps, pre, post):
    say("separate cycles", n, op, ncomp, dt, krylov, sweeps, pre, post)
    b, x0, coef = problem(n, op, ncomp, dt)
    ctx = plain_ctx(hp, n, dt=dt, mg_fixed_cycles=2, mg_krylov=krylov, mg_coarse_sweeps=sweeps, mg_pre=pre, mg_post=post)
    xd = to_dev(torch_dev, x0)
    _, rr = ctx.mg_solve(hp.OP_POISSON if coef[2] else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    fl = ref.fluid(n, dt=dt, fixed_cycles=2, krylov=krylov if ncomp == 1 else 0, coarse_sweeps=sweeps, pre=pre, post=post)
    for d in range(ncomp):
        xr, _, rrr = ref.mg_solve(fl, *coef, b[d], x0[d])
        assert_close(f"x[{d}]", host(xd)[d], xr, TOL)
        assert abs(rr[d] - rrr) <= 1e-6 * rrr + 1e-13, (rr[d], rrr)


@pytest.mark.parametrize("n,op,ncomp,dt,pre,post", [(64, "poisson", 1, 1e-3, 1, 1), (64, "poisson", 1, 1e-3, 3, 0),
                                                    (96, "helmholtz", 3, 1e-2, 3, 1), (64, "helmholtz", 2, 1e-3, 1, 2)])
def test_separate_cycles_mixed(torch_dev, hp, ref, n, op, ncomp, dt, pre, post):
    """To the default tolerance of 1e-10, against the oracle's solution to the same one:
    1e-8 as for the mixed solves with the default counts."""
    say("separate cycles, mixed", n, op, ncomp, dt, pre, post)
    b, x0, coef = problem(n, op, ncomp, dt)
    ctx = plain_ctx(hp, n, dt=dt, mg_pre=pre, mg_post=post, precision=hp.MIXED)
    xd = to_dev(torch_dev, x0)
    _, rr = ctx.mg_solve(hp.OP_POISSON if coef[2] else hp.OP_HELMHOLTZ, to_dev(torch_dev, b), xd)
    fl = ref.fluid(n, dt=dt, pre=pre, post=post)
    for d in range(ncomp):
        assert rr[d] <= 1e-10
        assert rel(host(xd)[d], ref.mg_solve(fl, *coef, b[d], x0[d])[0]) <= 1e-8
