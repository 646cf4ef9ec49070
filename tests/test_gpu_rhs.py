"""The fluid right-hand side in columns against the oracle: columns of one to eight
cells, tiles wider than the grid, rows that fill eight slabs of tiles
and rows that do not, with and without convection.

Random data, one fluid step: the right-hand side repeats the oracle's operations
(a wrong neighbour shows in the first digit), the solves stop at the same
iterates; the tolerance is that of the same comparison on smaller grids.
"""
import numpy as np
import pytest

from tests.test_gpu_parity import assert_close, host, plain_ctx, say, to_dev

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


@pytest.mark.parametrize("n,convection", [(12, 1), (48, 1), (64, 1), (96, 1), (128, 1), (96, 0)])
def test_rhs_columns(torch_dev, hp, ref, n, convection):
    torch = torch_dev
    say("rhs columns", n, convection)
    rng = np.random.default_rng(n + convection)
    u = 0.1 * rng.standard_normal((3, n, n, n))
    f = rng.standard_normal((3, n, n, n))
    p = np.zeros((n, n, n))
    ctx = plain_ctx(hp, n, convection=convection)
    ud, pd = to_dev(torch, u), to_dev(torch, p)
    ctx.ns_step(to_dev(torch, f), ud, pd)
    cyc, _ = ctx.step_stats()
    ur, pr, st = ref.ns_step(ref.fluid(n, convection=convection), f, u, p)
    assert list(cyc[0]) == list(st.cycles)
    assert_close("u", host(ud), ur)
    assert_close("p", host(pd), pr)
