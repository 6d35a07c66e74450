"""moe_route_package against its three parts, bit for bit: batches on both sides of
the one-workgroup packaging launch (1024 tokens), of the top-k taken inside it, and of
each top-k class, with and without co-activation counts, scores handed in, replicas,
row copies, both element types; the parts are checked against the oracle elsewhere."""
import numpy as np
import pytest
import torch

from paper_2607_08782_amd import moe, synth

from parity import say

pytestmark = pytest.mark.gpu

CASES = [
    # T, E, k, d, G, coact, dtype, logits_in, copy
    (1, 8, 2, 256, 2, False, "bf16", False, True),
    (64, 128, 8, 2048, 9, True, "bf16", False, False),
    (65, 16, 4, 512, 3, True, "bf16", False, True),
    (128, 128, 8, 256, 4, False, "bf16", False, False),
    (129, 128, 8, 256, 4, True, "bf16", False, False),      # top-k in a launch of its own
    (256, 64, 6, 256, 8, False, "bf16", False, False),
    (257, 60, 4, 256, 8, False, "bf16", False, False),
    (512, 8, 2, 512, 4, True, "bf16", False, True),
    (300, 200, 16, 256, 5, True, "bf16", False, False),     # E above the LDS co-activation bins
    (63, 256, 16, 256, 5, False, "bf16", False, False),
    (256, 17, 16, 256, 2, False, "bf16", False, False),     # exactly PLAN_IDS assignments
    (1023, 32, 4, 64, 4, False, "bf16", False, False),      # short K: the one-launch router
    (1024, 8, 2, 320, 4, True, "bf16", False, False),
    (1025, 8, 2, 320, 4, True, "bf16", False, True),        # three launches
    (77, 12, 3, 72, 3, True, "f32", False, True),
    (64, 8, 2, 128, 1, False, "f32", True, False),
    (200, 40, 5, 64, 4, False, "bf16", True, False),
    (0, 8, 2, 64, 2, True, "bf16", False, True),
    # K above 2048: short batches' scores in K chunks, summed by either top-k
    (1, 8, 2, 2056, 2, False, "bf16", False, False),
    (64, 8, 2, 4096, 4, False, "bf16", False, True),
    (60, 128, 8, 4104, 9, True, "bf16", False, False),
    (7, 200, 16, 7168, 5, False, "bf16", False, False),
    (300, 60, 4, 14336, 8, False, "bf16", False, False),
    (5, 20, 3, 24576, 4, False, "bf16", False, False),      # as many chunks as there may be
    (2000, 16, 2, 4096, 4, False, "bf16", False, False),    # long: the histogram's launches
    # long batches: the count of all experts per block (up to 32768 tokens, room for it)
    (1088, 128, 8, 256, 9, True, "bf16", False, False),
    (5001, 13, 3, 64, 4, False, "bf16", False, True),
    (2111, 256, 16, 64, 5, True, "bf16", False, False),
    (3000, 200, 5, 64, 3, True, "bf16", False, False),
    (32768, 60, 4, 64, 8, False, "bf16", False, False),
    (32769, 60, 4, 64, 8, False, "bf16", False, False),     # one block more
    (4096, 8, 2, 64, 1, True, "bf16", False, False),        # every expert here: no room
    (1500, 4, 2, 72, 2, True, "f32", True, True),
]


@pytest.mark.parametrize("T,E,k,d", [(64, 8, 2, 2048), (64, 8, 2, 4096), (33, 100, 8, 7168),
                                     (500, 40, 4, 4096), (8200, 64, 6, 256),
                                     (2048, 128, 8, 256), (2049, 128, 8, 256)])
def test_scores_not_asked_for(T, E, k, d):
    """Without a place for the scores the choice and the gates are the same bits, from
    the router alone and in one call, and the scores agree with float64."""
    say("[package] no scores T=%d E=%d k=%d d=%d" % (T, E, k, d))
    cfg = synth.custom_config(dtype="bf16", d=d, E=E, k=k, f=64, G=4, replicas=1, zipf=1.1)
    inp = synth.make_layer(cfg, T, seed=5, device="cuda", experts="none")
    logits, idx, gate = moe.moe_route_topk(inp.X, inp.Wr, inp.bias, k)
    ref = inp.X.double() @ inp.Wr.double().t() + inp.bias.double()
    mag = inp.X.double().abs() @ inp.Wr.double().abs().t() + inp.bias.double().abs()
    # an fp32 sum of d exact products in any order, 2 u per addition, and the bias
    assert bool(((logits.double() - ref).abs() <= (2 * d + 8) * 2.0 ** -24 * mag + 1e-30).all())
    _, idx2, gate2 = moe.moe_route_topk(inp.X, inp.Wr, inp.bias, k, want_logits=False)
    assert torch.equal(idx, idx2) and torch.equal(gate, gate2)
    n_local = int(inp.placement[:, 0].sum())
    cap = T * min(k, n_local)
    i32 = dict(dtype=torch.int32, device="cuda")
    out = {"x_perm": None, "group_offsets": torch.zeros((n_local + 1,), **i32),
           "row_token": torch.zeros((cap,), **i32), "row_gate": torch.zeros((cap,), device="cuda"),
           "token_row": torch.zeros((T, k), **i32), "send_counts": None}
    idx3, gate3 = torch.zeros_like(idx), torch.zeros_like(gate)
    need = moe.moe_route_topk_ws_bytes(moe.MOE_BF16, T, d, E, moe.MOE_RENORM)
    moe.moe_route_package(inp.X, inp.Wr, inp.bias, inp.placement, 0, logits=None, topk_idx=idx3,
                          topk_gate=gate3, ws_route=moe.workspace(need, "cuda"),
                          counts=torch.zeros((E,), **i32), coact=None, out=out,
                          ws_perm=moe.workspace(moe.moe_permute_ws_bytes(T, k, E), "cuda"),
                          cap_rows=cap, copy_rows=False)
    assert torch.equal(idx, idx3) and torch.equal(gate, gate3)


@pytest.mark.parametrize("T,E,k,d,G,coact,dtype,logits_in,copy", CASES)
def test_route_package_equals_its_parts(T, E, k, d, G, coact, dtype, logits_in, copy):
    say("[package] T=%d E=%d k=%d d=%d G=%d" % (T, E, k, d, G), coact, dtype, logits_in, copy)
    cfg = synth.custom_config(dtype=dtype, d=d, E=E, k=k, f=64, G=G, replicas=min(2, G - 1),
                              zipf=1.1)
    inp = synth.make_layer(cfg, T, seed=3, device="cuda", experts="none")
    n_local = int(inp.placement[:, 0].sum())
    cap = T * min(k, n_local)
    handed = torch.randn((T, E), device="cuda") if logits_in else None

    def fresh():
        i32 = dict(dtype=torch.int32, device="cuda")
        return {"logits": handed.clone() if logits_in else torch.zeros((T, E), device="cuda"),
                "idx": torch.zeros((T, k), **i32), "gate": torch.zeros((T, k), device="cuda"),
                "counts": torch.full((E,), -1, **i32),
                "coact": torch.full((E, E), -1, **i32) if coact else None,
                "perm": {"x_perm": torch.zeros((max(cap, 1), d), dtype=inp.X.dtype, device="cuda"),
                         "group_offsets": torch.full((n_local + 1,), -1, **i32),
                         "row_token": torch.full((max(cap, 1),), -1, **i32),
                         "row_gate": torch.zeros((max(cap, 1),), device="cuda"),
                         "token_row": torch.full((T, k), -9, **i32),
                         "send_counts": torch.full((G,), -1, **i32)}}

    code = moe.MOE_BF16 if dtype == "bf16" else moe.MOE_F32
    need = moe.moe_route_topk_ws_bytes(code, T, d, E, moe.MOE_RENORM)
    ws_r = moe.workspace(need, "cuda")
    ws_p = moe.workspace(moe.moe_permute_ws_bytes(T, k, E), "cuda")
    a, b = fresh(), fresh()
    moe.moe_route_topk(None if logits_in else inp.X, inp.Wr, inp.bias, k, logits=a["logits"],
                       logits_in=logits_in, topk_idx=a["idx"], topk_gate=a["gate"], ws=ws_r)
    moe.moe_expert_histogram(a["idx"], E, counts=a["counts"], coact=a["coact"])
    moe.moe_permute(inp.X, a["idx"], a["gate"], a["counts"], inp.placement, 0, E=E, cap_rows=cap,
                    out=a["perm"], ws=ws_p, copy_rows=copy)
    for _ in range(2):                                    # twice into the same buffers
        moe.moe_route_package(inp.X, inp.Wr, inp.bias, inp.placement, 0, logits=b["logits"],
                              topk_idx=b["idx"], topk_gate=b["gate"], ws_route=ws_r,
                              counts=b["counts"], coact=b["coact"], out=b["perm"], ws_perm=ws_p,
                              cap_rows=cap, logits_in=logits_in, copy_rows=copy)
    torch.cuda.synchronize()
    flat = lambda s: {**{n: v for n, v in s.items() if n != "perm"}, **s["perm"]}   # noqa: E731
    fa, fb = flat(a), flat(b)
    for name in fa:
        if fa[name] is not None:
            assert torch.equal(fa[name], fb[name]), name
    if T:
        assert int(fa["counts"].sum()) == T * k
        np.testing.assert_array_equal(np.bincount(fa["idx"].cpu().numpy().ravel(), minlength=E),
                                      fa["counts"].cpu().numpy())
