"""The fused attention kernels at head widths 64, 128 and 256, and every other multiple of 8 up to 128
padded to 64 or 128 in LDS, at the edges of tiles, row blocks and workgroup sizes, with and without the
waves in groups over the memory (query) rows, and the unfused formulation at widths no fused kernel
takes, against the oracle (same tolerance as in the widths' own test: bf16 storage, fp32 accumulation)."""
import math

import numpy as np
import pytest
import torch

import mtf_inputs
import paper_1811_02084_amd as mtf
from helpers import named as to_nt
from oracle import layer as OL
from oracle.layer import B, L, M, H, K, V
from oracle.metrics import m2

pytestmark = pytest.mark.gpu

TOL = 2e-2

CASES = [  # batch, length, heads, d_k, causal, scale (None: 1/sqrt(d_k))
    (1, 8, 1, 8, True, None), (2, 40, 3, 8, False, None), (2, 72, 3, 32, True, None), (1, 136, 2, 56, False, None),
    (2, 64, 2, 64, False, None), (1, 328, 3, 64, True, None), (2, 72, 2, 72, True, None), (1, 264, 2, 96, True, None),
    (2, 136, 3, 120, False, None),
    (4, 200, 32, 64, True, None), (4, 200, 32, 96, True, None),      # 4 waves per workgroup
    (4, 136, 16, 64, True, None), (4, 129, 16, 128, True, None), (4, 136, 16, 72, False, None),  # groups, two row waves
    (5, 200, 16, 64, True, None), (5, 193, 16, 128, False, None), (5, 200, 16, 80, True, None),  # two waves, no groups
    (1, 1, 1, 128, True, None), (2, 31, 3, 128, False, None), (1, 33, 2, 128, True, None), (1, 129, 3, 128, True, None),
    (3, 331, 4, 128, False, None), (1, 1000, 2, 128, True, None), (2, 257, 2, 128, True, -0.05),
    (2, 200, 3, 256, True, None), (5, 200, 16, 256, False, None), (1, 577, 3, 256, True, -0.05),   # groups; none; groups
    (1, 520, 40, 128, True, None), (1, 520, 40, 64, False, None), (1, 520, 60, 64, True, None),
    (4, 384, 32, 64, True, None), (4, 328, 32, 48, False, None), (4, 328, 32, 104, True, None),   # 8 waves
    (2, 104, 2, 64, True, -0.05), (2, 104, 2, 40, True, -0.05), (2, 104, 2, 96, False, -0.05),
]
UNFUSED = [  # widths above 128 other than 256: the two einsums with a row softmax between them, batched products
    (2, 72, 3, 136, True, None), (2, 136, 3, 136, False, None), (1, 200, 2, 264, True, None), (3, 72, 2, 248, False, -0.05),
    (2, 104, 2, 136, True, -0.05), (1, 328, 4, 192, True, None), (1, 8, 1, 520, False, None),
]


@pytest.mark.parametrize("case", CASES + UNFUSED, ids=["-".join(map(str, c)) for c in CASES + UNFUSED])
def test_against_oracle(case):
    b, l, h, dk, causal, scale = case
    print(f"attention core {case}", flush=True)
    mtf.timing_enable(True)
    scale = 1.0 / math.sqrt(dk) if scale is None else scale
    q, k, v, dctx = (mtf_inputs.normal(53, i, (b, l, h, dk)) for i in range(4))
    qn, kn, vn = to_nt(q, (B, L, H, K)), to_nt(k, (B, M, H, K)), to_nt(v, (B, M, H, V))
    ctx_ref, lse_ref = OL.attention_core_fwd(qn, kn, vn, scale, causal)
    ctx, lse = mtf.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale, causal)
    assert m2(ctx.float().cpu().numpy(), ctx_ref.data) <= TOL
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref.data)) <= 1e-3 * max(1.0, np.max(np.abs(lse_ref.data)))
    ctx_s = torch.from_numpy(ctx_ref.data).to(torch.bfloat16)
    lse_s = torch.from_numpy(lse_ref.data).float()
    refs = OL.attention_core_bwd(qn, kn, vn, to_nt(ctx_s, (B, L, H, V)), to_nt(lse_s, (B, H, L)),
                                 to_nt(dctx, (B, L, H, V)), scale, causal)
    gots = mtf.attention_bwd(q.cuda(), k.cuda(), v.cuda(), ctx_s.cuda(), lse_s.cuda(), dctx.cuda(), scale, causal)
    for name, got, ref in zip(("dq", "dk", "dv"), gots, refs):
        assert m2(got.float().cpu().numpy(), ref.data) <= TOL, name
    names = [t["kernel"] for t in mtf.timing_collect()]
    mtf.timing_enable(False)
    assert any("softmax" in n for n in names) == (case in UNFUSED), names


@pytest.mark.parametrize("case", [
    (1, 200, 2, 64, False), (1, 200, 2, 64, True), (1, 200, 2, 96, False), (1, 200, 2, 128, False),   # waves in groups
    (1, 200, 2, 128, True), (2, 200, 3, 256, False), (2, 200, 3, 256, True),
    (5, 200, 32, 64, False), (5, 193, 16, 128, False), (5, 200, 16, 256, False)],                     # no groups
    ids=lambda c: "-".join(map(str, c)))
def test_logits_that_overflow(case):
    """Whole tiles of memory rows whose logits are below the fp32 range (-inf) get no weight, wherever the
    tile falls among the groups; exact powers of two on q and k, so the tolerance is the same."""
    b, l, h, dk, causal = case
    print(f"attention core, overflowing logits {case}", flush=True)
    q, k, v, dctx = (mtf_inputs.normal(57, i, (b, l, h, dk)) for i in range(4))
    q = ((q.float().abs() + 1).bfloat16().float() * 2.0**66).bfloat16()
    k = (k.float() * 2.0**-66).bfloat16()
    for lo, hi in [(32, 64), (96, 128)] if causal else [(0, 64), (96, 128)]:
        k[:, lo:hi] = -(2.0**66)
    scale = 1.0 / dk
    qn, kn, vn = to_nt(q, (B, L, H, K)), to_nt(k, (B, M, H, K)), to_nt(v, (B, M, H, V))
    ctx_ref, lse_ref = OL.attention_core_fwd(qn, kn, vn, scale, causal)
    ctx, lse = mtf.attention_fwd(q.cuda(), k.cuda(), v.cuda(), scale, causal)
    assert m2(ctx.float().cpu().numpy(), ctx_ref.data) <= TOL
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref.data)) <= 1e-3 * max(1.0, np.max(np.abs(lse_ref.data)))
    refs = OL.attention_core_bwd(qn, kn, vn, ctx_ref, lse_ref, to_nt(dctx, (B, L, H, V)), scale, causal)
    gots = mtf.attention_bwd(q.cuda(), k.cuda(), v.cuda(), ctx, lse, dctx.cuda(), scale, causal)
    for name, got, ref in zip(("dq", "dk", "dv"), gots, refs):
        assert m2(got.float().cpu().numpy(), ref.data) <= TOL, name


@pytest.mark.parametrize("length,kernel", [(8, "attn_fwd_kernel<256, 2, false, 1>"), (32, "attn_fwd_kernel<256, 2, false, 1>"),
                                           (33, "attn_fwd_kernel<256, 4, false, 2>")])
def test_one_tile_of_memory_needs_no_groups(length, kernel):
    q = mtf_inputs.normal(58, 0, (1, length, 2, 256)).cuda()
    mtf.timing_enable(True)
    mtf.attention_fwd(q, q, q, 0.1, True)
    names = [t["kernel"] for t in mtf.timing_collect()]
    mtf.timing_enable(False)
    assert names == [kernel]


def test_unfused_widths_remain():
    """A width above 128 other than 256 still runs the two einsums with the row softmax between."""
    q = mtf_inputs.normal(54, 0, (2, 72, 3, 136)).cuda()
    mtf.timing_enable(True)
    mtf.attention_fwd(q, q, q, 0.1, True)
    names = [t["kernel"] for t in mtf.timing_collect()]
    mtf.timing_enable(False)
    assert "softmax_rows_kernel" in names, names
