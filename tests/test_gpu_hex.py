"""The hexahedral element kernels, eight lanes to an element, against the oracle:
meshes that leave lanes of a wavefront without an element, elements in grid order
(neighbours in a wavefront share a face, along each of the three axes) and in
random order, and materials that change from element to element.

Tolerances are those of the same comparisons on the workloads' meshes.
"""
import dataclasses

import numpy as np
import pytest

from paper_2503_22695_amd import inputs
from tests.test_gpu_adjoint import assert_rel, deformed
from tests.test_gpu_parity import assert_close, host, say, to_dev

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


@pytest.mark.parametrize("n_el,order,mixed", [(1, "x", 0), (3, "x", 1), (3, "y", 0), (3, "z", 1), (5, "random", 1),
                                              (9, "x", 1)])
def test_hex_elements(torch_dev, hp, ref, n_el, order, mixed):
    torch = torch_dev
    say("hex elements", n_el, order, mixed)
    base = inputs.ho_block(n=32, n_el=n_el)
    grid = np.arange(n_el ** 3).reshape(n_el, n_el, n_el)   # [z][y][x]
    pick = {"x": grid.ravel(), "y": grid.transpose(0, 2, 1).ravel(), "z": grid.transpose(1, 2, 0).ravel(),
            "random": np.random.default_rng(n_el).permutation(n_el ** 3)}[order]
    ho = base.materials[0]
    nh = inputs.neo_hookean_block().materials[0]
    mat = (np.arange(n_el ** 3) // 3 % 2 if mixed else np.zeros(n_el ** 3)).astype(np.int32)
    prob = dataclasses.replace(base, conn=np.ascontiguousarray(base.conn[pick]), fibre=base.fibre[pick], mat_id=mat,
                               materials=[ho, nh])
    ctx = hp.context_for_problem(prob)
    mesh = ref.MeshBuffers.from_problem(prob)
    x = deformed(prob, 17, 0.05)
    xd = to_dev(torch, x)
    V = np.random.default_rng(23).standard_normal(x.shape)
    assert_close("F", host(ctx.fe_force(xd, 0.0)), ref.fe_force(mesh, x)[0])
    assert_close("HV", host(ctx.fe_hvp(xd, to_dev(torch, V))), ref.fe_hvp(mesh, x, V), 1e-10)
    dth = torch.zeros((hp.MAX_MATERIALS, 4), dtype=torch.float64, device="cuda")
    ctx.fe_param_vjp(xd, to_dev(torch, V), dth)
    want = ref.fe_param_vjp(mesh, x, V)
    assert_rel("dtheta", host(dth)[0], want[0], 1e-10)
    assert float(dth[1:].abs().max()) == 0.0
