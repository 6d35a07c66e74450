"""Rows that are not finite stay among themselves (marked `gpu`): in every path of the
expert FFN a row of infinities or NaN leaves the bits of all other rows as they were
(tiles, their split K, strips, streaming, fp32), and the combine drops the rows that it
loads only to fill a batch of loads."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08782_amd import moe

from parity import np32, say

pytestmark = pytest.mark.gpu
SMALL, LARGE = moe.MOE_FFN_SMALL_GROUPS, moe.MOE_FFN_LARGE_GROUPS


@pytest.mark.parametrize("path,sizes,d,f,hint,dtype", [
    ("tiles", [300, 700], 128, 192, LARGE, torch.bfloat16),
    ("tiles with split K", [300], 2048, 128, LARGE, torch.bfloat16),
    ("strips", [70, 5, 130], 256, 128, SMALL, torch.bfloat16),
    ("streaming", [70, 5, 130], 4160, 4160, SMALL, torch.bfloat16),
    ("fp32, K over four waves", [70, 5, 130], 65, 130, 0, torch.float32),
    ("fp32, whole-K waves", [2000, 2100], 40, 2048, 0, torch.float32),
])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_ffn_rows_beside_rows_that_are_not_finite(path, sizes, d, f, hint, dtype, bad):
    say("[nonfinite]", path, bad)
    gen = torch.Generator().manual_seed(d)
    N = sum(sizes)
    x = torch.randn((N, d), generator=gen).to(dtype)
    wt = moe.WeightTable([(torch.randn((2 * f, d), generator=gen) * d ** -0.5).to(dtype).cuda() for _ in sizes],
                         [(torch.randn((d, f), generator=gen) * f ** -0.5).to(dtype).cuda() for _ in sizes])
    off = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).cuda()
    want = moe.moe_grouped_ffn(x.cuda(), off, wt, products=3 | hint)
    rows = [0, sizes[0] - 1, N - 1, N // 2]
    x[rows] = bad
    got = moe.moe_grouped_ffn(x.cuda(), off, wt, products=3 | hint)
    torch.cuda.synchronize()
    keep = torch.ones(N, dtype=torch.bool)
    keep[rows] = False
    assert torch.isfinite(want).all()
    assert torch.equal(got[keep.cuda()], want[keep.cuda()])
    assert not torch.isfinite(got[rows].float()).any()


@pytest.mark.parametrize("d,k", [(2048, 9), (512, 4), (520, 9), (256, 2), (7, 3)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_combine_drops_what_it_loads_for_nothing(d, k, dtype):
    """y_perm's first rows, which fill a batch of loads, are not finite and belong to one
    token; values and gates make every other sum exact."""
    say("[nonfinite] combine d=%d k=%d" % (d, k), dtype)
    T = 60
    rng = np.random.default_rng(d + k)
    here = rng.random((T, k)) < rng.random((T, 1))
    here[0], here[1], here[2] = False, False, True
    here[0, 0] = True
    N = int(here.sum())
    token_row = np.full((T, k), -1, np.int32)
    order = rng.permutation(N - 1).astype(np.int32) + 1
    token_row[here] = np.concatenate([[0], order])                # token 0 alone has row 0
    gate = rng.choice(np.array([0.25, 0.5, 1.0], np.float32), size=(T, k)).astype(np.float32)
    y_perm = rng.integers(-2, 3, size=(N, d)).astype(np.float32)
    y_perm[0, ::2], y_perm[0, 1::2] = np.nan, np.inf
    got = moe.moe_combine(torch.from_numpy(y_perm).to(dtype).cuda(), torch.from_numpy(token_row).cuda(),
                          torch.from_numpy(gate).cuda(), None, T=T, d=d)
    torch.cuda.synchronize()
    ref = oracle.combine(np.nan_to_num(y_perm, posinf=0.0), token_row, gate, None, T, d, k)
    np.testing.assert_array_equal(np32(got[1:T]), ref[1:].astype(np.float32))
    assert not torch.isfinite(got[0].float()).any()
