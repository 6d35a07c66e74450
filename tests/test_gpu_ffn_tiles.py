"""The bf16 expert FFN at the edges of its kernels: tiles of 256 rows and their LDS
ring (K of one and two 64-wide steps, column tails, row tiles in blocks of eight; more
tiles than workgroups, so that a tile's last stages load the next tile's first or, with K
= 64, its ring starts again), whole-K strips (32 output columns, 32- and 64-row tiles, K
from 64 to their longest), each against the oracle's expert FFN in float64 on sampled rows.
The tolerance is the parity protocol's: h and y are rounded to bf16 (2^-8 relative
each), sums in fp32."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_08782_amd import moe

from parity import OUT_TOL, close, np32, say

pytestmark = pytest.mark.gpu
LARGE, SMALL = moe.MOE_FFN_LARGE_GROUPS, moe.MOE_FFN_SMALL_GROUPS


@pytest.mark.parametrize("sizes,d,f,hint,gather", [
    ([257, 300], 64, 64, LARGE, False),             # one 64-wide K step
    ([700, 1, 0, 513], 64, 192, LARGE, True),
    ([300, 600], 128, 64, LARGE, True),             # two in the gate/up product, one in the down
    ([256, 512, 1024], 192, 448, LARGE, False),     # exact tiles, column tails
    ([2305], 256, 320, LARGE, False),               # ten row tiles: two blocks of five
    ([4500, 260], 128, 128, LARGE, True),           # 18 row tiles: three blocks of six
    ([300] * 20, 64, 128, LARGE, False),
    # two and three tiles a workgroup, ragged rows and columns
    ([5000 + 37 * i for i in range(16)], 64, 192, LARGE, True),    # the ring starts again, the
    ([5000 + 37 * i for i in range(16)], 64, 64, LARGE, False),    # next tile's rows gathered
    ([5000 + 37 * i for i in range(16)], 128, 320, LARGE, True),   # four stages: chained
    ([4900 + 41 * i for i in range(16)], 192, 128, LARGE, False),
    ([1, 64, 33, 0, 17], 64, 64, SMALL, True),      # strips, one K stage
    ([1, 64, 33, 0, 17], 4096, 128, SMALL, True),   # longest K, both tile heights
    ([128, 129, 256, 65], 192, 2048, SMALL, False),   # several row tiles and tails
    ([200, 3], 4160, 128, SMALL, False),            # gate/up split over workgroups, down a strip
    ([40, 90], 128, 4160, SMALL, True),             # and the reverse
    ([60, 64, 10], 2112, 128, SMALL, False),        # past K = 2048: strips up to 64 rows on average,
    ([100, 70, 80], 2112, 128, SMALL, False),       # split above,
    ([200, 130], 2112, 4096, SMALL, True),          # also with two groups in few strips,
    ([200, 130], 2112, 9856, SMALL, True),          # strips in many
    ([30, 5, 64], 256, 128, 0, False),              # no hint
    ([700, 5, 64, 200], 256, 128, 0, True),
])
def test_bf16_ffn_tile_edges(sizes, d, f, hint, gather):
    say("[bf16 ffn]", sizes, "d=%d f=%d hint=%d gather=%s" % (d, f, hint, gather))
    gen = torch.Generator().manual_seed(d * 31 + f)
    N = sum(sizes)
    T = max(sizes) + 5
    x = torch.randn((T if gather else N, d), generator=gen).bfloat16()
    w13 = [(torch.randn((2 * f, d), generator=gen) * d ** -0.5).bfloat16() for _ in sizes]
    w2 = [(torch.randn((d, f), generator=gen) * f ** -0.5).bfloat16() for _ in sizes]
    tok = torch.cat([torch.randperm(T, generator=gen)[:n] for n in sizes]).to(torch.int32)
    tok = torch.cat([tok, torch.zeros(2, dtype=torch.int32)])
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    wt = moe.WeightTable([w.cuda() for w in w13], [w.cuda() for w in w2])
    y = torch.full((N + 2, d), 5.0, dtype=torch.bfloat16, device="cuda")
    off = torch.tensor(offs).cuda()
    for _ in range(2):
        if gather:
            moe.moe_grouped_ffn_rows(x.cuda(), tok.cuda(), off, wt, cap_rows=N + 2, y_perm=y,
                                     products=3 | hint)
        else:
            moe.moe_grouped_ffn(x.cuda(), off, wt, cap_rows=N, y_perm=y, products=3 | hint)
    torch.cuda.synchronize()
    got = np32(y)
    rows = np32(x)[np32(tok).astype(np.int64)[:N]] if gather else np32(x)
    rng = np.random.default_rng(0)
    for g, n in enumerate(sizes):
        a = int(offs[g])
        if n == 0:
            continue
        # every row of the first and last 16, and some between
        pick = np.unique(np.concatenate([np.arange(min(n, 16)), np.arange(max(0, n - 16), n),
                                         rng.integers(0, n, 24)])) + a
        ref = oracle.expert_ffn(rows[pick], np32(w13[g]), np32(w2[g]))
        close(got[pick], ref, OUT_TOL["bf16"], "group %d" % g)
        assert np.isfinite(got[a:a + n]).all()
    assert np.all(got[N:] == 5.0)


def test_more_tiles_than_a_list_holds():
    """A workgroup lists 256 of its tiles at a time: 260 tiles each, the second list
    included, every row tile and all 64 column tiles of the gate/up product (a column
    tile that is wrong or missing moves its rows of y by an eighth of their size)."""
    sizes, d, f = [200000, 66300], 64, 8192
    say("[bf16 ffn] %d tiles of the gate/up product" % (sum(-(-n // 256) for n in sizes) * (f // 128)))
    N = sum(sizes)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((N, d), generator=gen, device="cuda").bfloat16()
    w13 = [(torch.randn((2 * f, d), generator=gen, device="cuda") * d ** -0.5).bfloat16() for _ in sizes]
    w2 = [(torch.randn((d, f), generator=gen, device="cuda") * f ** -0.5).bfloat16() for _ in sizes]
    off = torch.tensor([0, sizes[0], N], dtype=torch.int32).cuda()
    y = moe.moe_grouped_ffn(x, off, moe.WeightTable(w13, w2), products=3 | LARGE)
    torch.cuda.synchronize()
    a = 0
    for g, n in enumerate(sizes):
        pick = torch.arange(0, n, 61, device="cuda") + a           # four or five of each row tile
        xs = x[pick].double()
        h = torch.nn.functional.silu(xs @ w13[g][:f].double().t()) * (xs @ w13[g][f:].double().t())
        ref = h @ w2[g].double().t()
        rel = (y[pick].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert float(rel.max()) < OUT_TOL["bf16"], (g, float(rel.max()))
        a += n


@pytest.mark.parametrize("sizes,d,f,gather", [
    ([300, 40, 1, 64, 0, 200, 7, 100, 5], 8256, 2048, True),           # the gate/up product
    ([9, 64, 30, 1, 256, 17, 500, 3, 2, 33, 50, 6, 0, 12, 65, 8, 21, 4], 2048, 8256, False),  # down
])
def test_streamed_beside_tiled_groups(sizes, d, f, gather):
    """A long K and more tiles than can be split: the groups of up to 256 rows stream
    beside the tiles of the large one.  Against float64 on every row, the products
    together and one by one, and not the bits of a call that tiles every group."""
    say("[bf16 ffn] mixed", sizes, "d=%d f=%d gather=%s" % (d, f, gather))
    N, T = sum(sizes), max(sizes) + 5
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((T if gather else N, d), generator=gen, device="cuda").bfloat16()
    w13 = [(torch.randn((2 * f, d), generator=gen, device="cuda") * d ** -0.5).bfloat16() for _ in sizes]
    w2 = [(torch.randn((d, f), generator=gen, device="cuda") * f ** -0.5).bfloat16() for _ in sizes]
    tok = torch.randint(0, T, (N + 2,), generator=gen, device="cuda", dtype=torch.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    wt, off = moe.WeightTable(w13, w2), torch.tensor(offs).cuda()
    ws = moe.workspace(moe.moe_grouped_ffn_ws_bytes(moe.MOE_BF16, N + 2, d, f, len(sizes)), "cuda")

    def call(*products):
        y = torch.full((N + 2, d), 5.0, dtype=torch.bfloat16, device="cuda")
        for p in products:
            if gather:
                moe.moe_grouped_ffn_rows(x, tok, off, wt, cap_rows=N + 2, y_perm=y, ws=ws, products=p)
            else:
                moe.moe_grouped_ffn(torch.cat([x, x[:2]]), off, wt, cap_rows=N + 2, y_perm=y, ws=ws,
                                    products=p)
        torch.cuda.synchronize()
        return y

    y = call(3)
    assert torch.equal(y, call(moe.MOE_FFN_GATE_UP, moe.MOE_FFN_DOWN)) and torch.equal(y, call(3))
    assert bool((y[N:] == 5.0).all())
    tiled = call(3 | LARGE)
    rows, small = x[tok[:N].long()] if gather else x, []
    for g, n in enumerate(sizes):
        if n == 0:
            continue
        a = int(offs[g])
        xs = rows[a:a + n].double()
        h = torch.nn.functional.silu(xs @ w13[g][:f].double().t()) * (xs @ w13[g][f:].double().t())
        ref = h @ w2[g].double().t()
        rel = (y[a:a + n].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert float(rel.max()) < OUT_TOL["bf16"], (g, float(rel.max()))
        small += [r for r in range(a, a + n) if n <= 256]
    # over all of them: an order of fp32 sums changes one h in about 10^4 after rounding
    assert not torch.equal(y[small], tiled[small])
