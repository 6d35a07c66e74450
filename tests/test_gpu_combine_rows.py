"""Combine over many tokens (marked `gpu`): a wave per token and the other widths, every
number of local rows from none to k (one, two, up to four and up to eight rows loaded
together), in bf16 and fp32.
Values are small integers and gates powers of two, so every sum is exact and the output
equals the oracle's bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08782_amd import moe

from parity import np32, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,d,dtype", [(8192, 3, 2048, "bf16"), (8191, 8, 2048, "bf16"),
                                         (8195, 16, 2048, "bf16"), (4097, 2, 4096, "bf16"),
                                         (8193, 1, 2048, "bf16"), (2731, 5, 6144, "bf16"),
                                         (8192, 4, 1024, "f32"), (33, 6, 512, "bf16"),
                                         (50, 9, 256, "f32"), (70, 4, 520, "bf16")])
def test_combine_exact(T, k, d, dtype):
    say("[combine rows]", T, k, d, dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(T + 7 * k + d)
    here = rng.random((T, k)) < rng.random((T, 1))
    here[:3] = False
    here[3:6] = True
    N = int(here.sum())
    token_row = np.full((T, k), -1, np.int32)
    token_row[here] = rng.permutation(N).astype(np.int32)
    gate = rng.choice(np.array([0.25, 0.5, 1.0], np.float32), size=(T, k)).astype(np.float32)
    y_perm = rng.integers(-2, 3, size=(N, d)).astype(np.float32)
    y_shared = rng.integers(-2, 3, size=(T, d)).astype(np.float32)
    got = moe.moe_combine(torch.from_numpy(y_perm).to(dt).cuda(), torch.from_numpy(token_row).cuda(),
                          torch.from_numpy(gate).cuda(), torch.from_numpy(y_shared).to(dt).cuda(),
                          T=T, d=d)
    torch.cuda.synchronize()
    ref = oracle.combine(y_perm, token_row, gate, y_shared, T, d, k)
    np.testing.assert_array_equal(np32(got[:T]), ref.astype(np.float32))
