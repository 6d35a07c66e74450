"""Edges of the vector quantization (marked `gpu`): every E4M3 decision boundary and its
neighbours, at scales over the whole exponent range, both row layouts; rows with
infinities and NaN as the element-by-element kernel (misaligned rows) gives them.
"""
import numpy as np
import pytest
import torch

from oracle import quant as oq
from paper_2607_08782_amd import moe

from parity import np32, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    moe.load_library()
    yield


def _boundaries() -> np.ndarray:
    grid = oq.e4m3_decode(np.arange(0x7F))
    mid = ((grid[1:] + grid[:-1]) / 2).astype(np.float32)
    pts = np.concatenate([grid.astype(np.float32), mid])
    pts = np.concatenate([pts, np.nextafter(pts, np.float32(np.inf)), np.nextafter(pts, np.float32(0))])
    pts = np.minimum(pts, np.float32(448.0))
    return np.concatenate([pts, -pts])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols", [(40, 1024), (1100, 1024), (1031, 520), (1024, 4096),
                                       (1025, 4104), (1030, 8)])
def test_codes_at_every_boundary_and_scale(dtype, rows, cols):
    say("[quant-edge]", dtype, rows, cols)
    rng = np.random.RandomState(rows + cols)
    b = _boundaries()
    v = rng.choice(b, size=(rows, cols)).astype(np.float32)
    v[:, 0] = 448.0                                  # scale 1 before the row's factor
    # powers of two keep the boundaries exact; the fast rows' range ends inside them
    e = rng.randint(-118, 119, size=(rows, 1))
    e[::3] = 0
    v = np.ldexp(v, e)
    odd = rng.rand(rows) < 0.5                       # a scale that is not a power of two
    v[odd] *= rng.uniform(0.5, 1.0, size=(int(odd.sum()), 1)).astype(np.float32)
    x = torch.from_numpy(v.astype(np.float32)).to(dtype)
    q, s = moe.moe_quantize_e4m3(x.cuda())
    rq, rs = oq.quantize_rows(np32(x))
    np.testing.assert_array_equal(s.cpu().numpy(), rs)
    np.testing.assert_array_equal(q.cpu().numpy(), rq)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows", [20, 1056])
def test_rows_that_are_not_finite_match_the_element_kernel(dtype, rows):
    say("[quant-nonfinite]", dtype, rows)
    g = torch.Generator().manual_seed(rows)
    x = torch.randn(rows, 264, generator=g)
    x[1, 7] = float("inf")
    x[2, 9] = -float("inf")
    x[3, 11] = float("nan")
    x[4] = float("nan")
    x[5, ::2] = float("nan")
    x[6] = -0.0
    x[7] = 1e-40                                     # subnormal rows
    x = x.to(dtype)
    flat = torch.empty(rows * 264 + 1, dtype=dtype, device="cuda")
    un = flat[1:].view(rows, 264)
    un.copy_(x)
    q, s = moe.moe_quantize_e4m3(x.cuda())
    rq, rs = moe.moe_quantize_e4m3(un)
    assert torch.equal(s.view(torch.int32), rs.view(torch.int32))
    assert torch.equal(q, rq)
