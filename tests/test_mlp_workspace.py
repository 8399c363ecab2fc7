"""Workspace of the network field: what its layout holds, on the host; and that nothing of what
the workspace held before a forward reaches a gradient, on the GPU."""

import numpy as np
import pytest
import torch

import paper_2509_14442_amd._lib as L

BLOCK = 64 * 64 + 64  # one layer's partial gradient


@pytest.mark.parametrize("depth", [1, 4, 8])
@pytest.mark.parametrize("n", [1, 100, 129, 128 ** 3])
def test_workspace_holds_the_activations_once(n, depth):
    """Activations, the 127 rows a backward block may load past them, transposed weights, at most
    512 blocks of partial gradients, inputs; each part rounded up to 256 bytes."""
    blocks = min(max((n + 63) // 64, 1), 512)
    floats = (depth * n + 127) * 64 + depth * 64 * 64 + (depth + 1) * blocks * BLOCK + 4 * n
    size = L.load().rbos_mlp_workspace_bytes(64, depth, n)
    assert 4 * floats <= size <= 4 * floats + 4 * 256


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [0x7F800001, 0x7FC00000, 0x7F800000, -0x00800000])  # NaNs, infinities
@pytest.mark.parametrize("depth,n", [(1, 1), (1, 129), (4, 65), (8, 200)])
def test_stale_workspace_does_not_reach_the_gradient(depth, n, bits):
    """The same gradient, bit for bit, from a workspace of zeros and one full of what is no number."""
    from paper_2509_14442_amd import api

    g = torch.Generator().manual_seed(depth)
    theta = (0.3 * torch.randn(api.MLP.param_count(64, depth), generator=g)).cuda()
    m = api.MLP(theta, 64, depth, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0))
    x, lam = torch.rand((n, 3), generator=g).cuda(), torch.randn((n, 5), generator=g).cuda()
    out = []
    for fill in (0, bits):
        m.forward(x)
        ws = next(iter(m._ws.values()))
        ws[:ws.numel() // 4 * 4].view(torch.int32).fill_(fill)
        m.forward(x)
        out.append(m.backward(lam, x).cpu().numpy())
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])
