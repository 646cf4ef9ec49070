"""Binning, spreading and interpolation against the oracle where tiles are many,
empty, sparse and crowded: one and several rounds of the scan over the tiles, a
number of tiles that is no multiple of four, tiles of at most 64 nodes, of more,
and of more than one work item, and more work items than workgroups.

Tolerances are those of the same comparison on smaller node sets.
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


# (n, nodes spread evenly, nodes in one tile's corner, deterministic): 27, 512, 13824 tiles
@pytest.mark.parametrize("n,even,crowd,det", [(12, 500, 300, 0), (64, 3000, 64, 0), (64, 3000, 65, 1), (192, 40000, 700, 0),
                                              (192, 1, 0, 0)])
def test_bins(torch_dev, hp, ref, n, even, crowd, det):
    torch = torch_dev
    say("bins", n, even, crowd, det)
    rng = np.random.default_rng(n + crowd)
    X = np.concatenate([rng.uniform(-0.3, 1.3, (even, 3)), rng.uniform(0.05, 0.05 + 2.0 / n, (crowd, 3))])
    X = X[rng.permutation(len(X))]
    F = rng.standard_normal(X.shape)
    u = rng.standard_normal((3, n, n, n))
    ctx = plain_ctx(hp, n, deterministic=det)
    ctx.set_mesh(X, np.zeros((0, 8)), np.zeros((0, 3)), np.zeros(0))
    Xd = to_dev(torch, X)
    for _ in range(2):   # the second binning finds the counts that the first one left
        f = torch.zeros((3, n, n, n), dtype=torch.float64, device="cuda")
        ctx.spread(Xd, to_dev(torch, F), f)
        assert_close("f", host(f), ref.spread(n, X, F))
        assert_close("U", host(ctx.interpolate(Xd, to_dev(torch, u))), ref.interpolate(X, u))


@pytest.mark.parametrize("n,mixed,det", [(64, 0, 0), (64, 0, 1), (12, 0, 0), (64, 1, 0)])
def test_interpolation_order(torch_dev, hp, n, mixed, det):
    """A node's interpolated velocity has the same bits whatever the order of the
    nodes and whichever others share its tile: a tile of 300 nodes (a full work
    item and one of 44), sparse tiles, several orders, and part of the nodes
    alone, so that the crowded tile is sparse."""
    torch = torch_dev
    say("interpolation order", n, mixed, det)
    rng = np.random.default_rng(17 + n)
    X = np.concatenate([rng.uniform(-0.3, 1.3, (400, 3)), rng.uniform(0.05, 0.05 + 2.0 / n, (300, 3))])
    u = to_dev(torch, rng.standard_normal((3, n, n, n)))

    def interpolate(nodes):
        ctx = plain_ctx(hp, n, deterministic=det, precision=hp.MIXED if mixed else hp.FP64)
        ctx.set_mesh(X[nodes], np.zeros((0, 8)), np.zeros((0, 3)), np.zeros(0))
        return host(ctx.interpolate(to_dev(torch, X[nodes]), u))

    U = interpolate(np.arange(len(X)))
    for nodes in [rng.permutation(len(X)) for _ in range(4)] + [np.arange(len(X))[::-1], np.arange(0, len(X), 7)]:
        assert np.array_equal(interpolate(nodes), U[nodes])
