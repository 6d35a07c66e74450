"""Tiled score kernels with their top-k (marked `gpu`): widths around the expert tiles,
one stage of K to several turns of the ring, a ragged last token block.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08782_amd import moe

from parity import GATE_TOL, close, np32, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    moe.load_library()
    yield


@pytest.mark.parametrize("T,d,E,k", [(8192, 64, 33, 2), (8161, 192, 64, 6), (8193, 320, 65, 3),
                                     (8130, 448, 100, 8), (8192, 2048, 128, 8),
                                     (8200, 704, 128, 16), (8192, 576, 129, 4), (8129, 64, 256, 8)])
@pytest.mark.parametrize("want", [True, False])
def test_tiled_scores_and_their_topk(T, d, E, k, want):
    say("[score-edge]", T, d, E, k, want)
    g = torch.Generator().manual_seed(T + d + E)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16)
    w = (torch.randn(E, d, generator=g) * 0.05).to(torch.bfloat16)
    bias = torch.randn(E, generator=g) * 0.3
    xc, wc, bc = x.cuda(), w.cuda(), bias.cuda()
    logits, idx, gate = moe.moe_route_topk(xc, wc, bc, k, renorm=True)
    ref = np32(x).astype(np.float64) @ np32(w).astype(np.float64).T + np32(bias)
    mag = np.abs(np32(x)).astype(np.float64) @ np.abs(np32(w)).astype(np.float64).T
    got = logits.cpu().numpy()
    # an fp32 sum of d exact products in any order, 2 u per addition, and the bias
    bound = (2 * d + 8) * 2.0 ** -24 * (mag + np.abs(np32(bias))) + 1e-30
    assert np.all(np.abs(got - ref) <= bound)
    ridx, rgate = oracle.topk(got, k, renorm=True)
    if not want:
        _, idx, gate = moe.moe_route_topk(xc, wc, bc, k, renorm=True, want_logits=False)
    np.testing.assert_array_equal(idx.cpu().numpy(), ridx)
    close(np32(gate), rgate, GATE_TOL, "gates")
