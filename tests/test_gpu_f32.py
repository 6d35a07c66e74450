"""The fp32 matrix-core kernels at the edges of their tiles: the grouped FFN
(32- and 64-row tiles, 16-, 32- and 64-column tiles, K in 16-wide blocks split
over four waves, 16-byte and 4-byte loads) and the gate scores (16 tokens x 16
experts per wave, 1 to 16 expert tiles), against the oracle in float64.

Tolerance: a sum of n fp32 products differs from the exact one by at most about
n u sum|terms| (u = 2^-24); the terms here are random signs, so the errors stay
near sqrt(n) u max|ref|, below 1e-5 max|ref| for every n used.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08782_amd import moe

from parity import LOGIT_TOL, OUT_TOL, close, np32, say

pytestmark = pytest.mark.gpu


def _placed(t, shift):
    """t on the GPU, `shift` elements past a 16-byte boundary."""
    buf = torch.zeros(t.numel() + 4, dtype=t.dtype, device="cuda")
    view = buf[shift:shift + t.numel()].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("sizes,d,f,shift,gather", [
    ([1, 0, 31, 32, 33], 16, 16, 0, False),        # one K block, 16-column tiles
    ([17, 64, 5], 72, 40, 0, True),                # K tail of 8, column tail
    ([17, 64, 5], 73, 41, 0, False),               # rows not 16-byte multiples
    ([40, 3], 64, 64, 1, True),                    # misaligned input rows
    ([200, 90, 0, 333], 132, 516, 0, True),        # 32 x 32 tiles, K split over waves
    ([1000, 70, 1100], 20, 2051, 0, False),        # 64 x 64 tiles of whole-K waves (gate/up)
    ([700, 65, 800], 2052, 36, 0, True),           # ... and of the down product
    ([1], 1, 1, 0, False),
    ([33, 2], 3, 2, 1, False),                     # rows shorter than a load
    ([5, 40], 4, 5, 3, True),
    ([70], 6, 19, 2, False),                       # a K tail in every quarter's last block
    ([31, 600], 65, 130, 1, True),
])
def test_f32_ffn_tile_edges(sizes, d, f, shift, gather):
    say("[f32 ffn]", sizes, "d=%d f=%d shift=%d gather=%s" % (d, f, shift, gather))
    gen = torch.Generator().manual_seed(d * 7 + f)
    N, T = sum(sizes), 50
    x = torch.randn((T if gather else N, d), generator=gen)
    w13 = [torch.randn((2 * f, d), generator=gen) * d ** -0.5 for _ in sizes]
    w2 = [torch.randn((d, f), generator=gen) * f ** -0.5 for _ in sizes]
    tok = torch.randint(0, T, (N + 2,), generator=gen, dtype=torch.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    wt = moe.WeightTable([w.cuda() for w in w13], [w.cuda() for w in w2])
    y = torch.full((N + 2, d), 5.0, device="cuda")
    off_dev, xd = torch.tensor(offs).cuda(), _placed(x, shift)
    if gather:
        moe.moe_grouped_ffn_rows(xd, tok.cuda(), off_dev, wt, cap_rows=N + 2, y_perm=y)
    else:
        moe.moe_grouped_ffn(xd, off_dev, wt, cap_rows=N, y_perm=y)
    torch.cuda.synchronize()
    got = np32(y)
    rows = np32(x)[np32(tok).astype(np.int64)[:N]] if gather else np32(x)
    for g, n in enumerate(sizes):
        a = int(offs[g])
        if n:
            ref = oracle.expert_ffn(rows[a:a + n], np32(w13[g]), np32(w2[g]))
            close(got[a:a + n], ref, OUT_TOL["f32"], "group %d" % g)
    assert np.all(got[N:] == 5.0)


@pytest.mark.parametrize("d,f", [(20, 2051), (132, 2304), (2052, 36), (1000, 2048), (17, 2100)])
def test_f32_ffn_bits_are_the_rows_own(d, f):
    """An output row's bits are those of its input row and weights: the same through the
    row map from misaligned token rows, from an aligned packaged copy, in a larger
    workspace, and in a call of a few rows (whole-K waves against K over four waves)."""
    say("[f32 bits] d=%d f=%d" % (d, f))
    gen = torch.Generator().manual_seed(d + f)
    sizes, T = [1000, 70, 1100], 300
    N = sum(sizes)
    x = torch.randn((T, d), generator=gen)
    w13 = [(torch.randn((2 * f, d), generator=gen) * d ** -0.5).cuda() for _ in sizes]
    w2 = [(torch.randn((d, f), generator=gen) * f ** -0.5).cuda() for _ in sizes]
    tok = torch.randint(0, T, (N,), generator=gen, dtype=torch.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    wt, off = moe.WeightTable(w13, w2), torch.tensor(offs).cuda()
    packed = x[tok.long()].contiguous()
    want = moe.moe_grouped_ffn(packed.cuda(), off, wt)
    rows = moe.moe_grouped_ffn_rows(_placed(x, 1), tok.cuda(), off, wt, cap_rows=N)
    wide = torch.zeros((4 * N, d), device="cuda")
    wide[:N] = packed.cuda()
    roomy = moe.moe_grouped_ffn(wide, off, wt)
    misaligned = moe.moe_grouped_ffn(_placed(packed, 3), off, wt)
    for name, y in (("row map", rows), ("capacity", roomy[:N]), ("misaligned", misaligned)):
        assert torch.equal(y, want), name
    for g, n in enumerate(sizes):
        few = packed[offs[g]:offs[g] + 5].contiguous().cuda()
        y = moe.moe_grouped_ffn(few, torch.tensor([0, 5], dtype=torch.int32).cuda(),
                                moe.WeightTable(w13[g:g + 1], w2[g:g + 1]))
        assert torch.equal(y, want[offs[g]:offs[g] + 5]), "a few rows of group %d" % g


@pytest.mark.parametrize("T,E,k,d,shift", [(1, 1, 1, 1, 0), (16, 16, 2, 64, 0), (17, 17, 4, 65, 0),
                                           (33, 33, 8, 130, 0), (50, 100, 8, 516, 0),
                                           (31, 200, 16, 1028, 0), (15, 256, 16, 16, 1)])
def test_f32_scores_tile_edges(T, E, k, d, shift):
    say("[f32 scores] T=%d E=%d k=%d d=%d shift=%d" % (T, E, k, d, shift))
    gen = torch.Generator().manual_seed(T + E)
    x, w = torch.randn((T, d), generator=gen), torch.randn((E, d), generator=gen) * d ** -0.5
    b = torch.randn((E,), generator=gen)
    logits, idx, gate = moe.moe_route_topk(_placed(x, shift), _placed(w, shift), b.cuda(), k)
    torch.cuda.synchronize()
    ref = np32(x).astype(np.float64) @ np32(w).astype(np.float64).T + np32(b)
    close(np32(logits), ref, LOGIT_TOL["f32"], "scores")
    order = np.argsort(-np32(logits), axis=1, kind="stable")[:, :k]
    np.testing.assert_array_equal(idx.cpu().numpy(), order)
