"""SiLU of the gate/up epilogues over its whole range (marked `gpu`): each path that
applies it, one gate value per row (on both sides of the switch to a plain division at
87), up values that are powers of two and W2 the identity, so y holds bf16(SiLU(a) * 2^s)
itself.

Down to the smallest result: for a in (-88.7, -87.3) 1 + exp(-a) lies above 2^126, whose
reciprocal is subnormal, and SiLU(a) is still a normal number.  Tolerance: the bf16
rounding (8 bits, 2^-8) and exp in fp32 (its argument, up to 128 in powers of two, is
rounded to 2^-18: 2^-18.5 of the result).
"""
import numpy as np
import pytest
import torch

from paper_2607_08782_amd import moe

from parity import np32, say

pytestmark = pytest.mark.gpu
SMALL, LARGE = moe.MOE_FFN_SMALL_GROUPS, moe.MOE_FFN_LARGE_GROUPS


@pytest.mark.parametrize("path,rows,d,hint", [
    ("tiles", 300, 64, LARGE),
    ("tiles with split K", 300, 4096, LARGE),
    ("strips", 200, 64, SMALL),
    ("split-K streaming", 200, 4160, SMALL),
])
def test_silu_down_to_its_smallest_results(path, rows, d, hint):
    say("[silu]", path, "rows=%d d=%d" % (rows, d))
    f = 64
    a = np.concatenate([np.linspace(-88.5, -86, 40), -np.geomspace(1e-3, 86, 70),
                        np.geomspace(1e-3, 86, 30), [-100.0, -89.0, -87.0, 0.0, 86.5, 87.0, 500.0, 1e30]])
    a = np.resize(a, rows)
    x = torch.zeros((rows, d))
    x[:, 0] = torch.from_numpy(a)
    x[:, 1] = 1.0
    x = x.bfloat16()
    up = np.resize(np.array([0, 7, 60, 100]), f)
    w13 = torch.zeros((2 * f, d))
    w13[:f, 0] = 1.0
    w13[f:, 1] = torch.from_numpy(2.0 ** up).float()
    w2 = torch.zeros((d, f))
    w2[:f] = torch.eye(f)
    wt = moe.WeightTable([w13.bfloat16().cuda()], [w2.bfloat16().cuda()])
    off = torch.tensor([0, rows], dtype=torch.int32).cuda()
    y = moe.moe_grouped_ffn(x.cuda(), off, wt, products=3 | hint)
    torch.cuda.synchronize()
    got = np32(y)[:, :f].astype(np.float64)
    av = np32(x)[:, 0].astype(np.float64)[:, None]
    with np.errstate(over="ignore"):
        ref = av / (1.0 + np.exp(-av)) * 2.0 ** up
    ref = np.where(av < -88.7, 0.0, ref)               # exp(-a) above the fp32 range
    # results that bf16 holds as normal numbers, products of them included
    seen = ((np.abs(ref) > 2.0 ** -100) | (av < -88.7)) & (np.abs(ref) < 2.0 ** 127)
    bad = np.abs(got - ref) > (2.0 ** -8 + 2.0 ** -17) * np.abs(ref)
    assert not (bad & seen).any(), (av[(bad & seen).any(1)][:5], got[bad & seen][:5], ref[bad & seen][:5])
    assert ((np.abs(ref) > 2.0 ** -100) & (av < -87.4)).sum() > 50
