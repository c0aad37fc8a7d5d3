"""The layer-normalisation gradients and the embedding gradient at the sizes where their passes end
raggedly: rows not a multiple of a workgroup's waves, every chunk count of d_model, blocks of 128 to 1024 ids."""
import pytest
import torch

import paper_1811_02084_amd as mtf

pytestmark = pytest.mark.gpu


def _ints(shape, seed, lo=-8, hi=9):
    return torch.randint(lo, hi, shape, generator=torch.Generator().manual_seed(seed)).float()


@pytest.mark.parametrize("rows,d", [(1, 8), (7, 64), (9, 512), (33, 520), (2049, 1024), (4100, 1032), (1027, 2048), (515, 4096)])
def test_layer_norm_gradients(rows, d):
    """dbias of small integers is exact; dx and dgain within bf16 inputs / fp32 sums of the 64-bit values."""
    print(f"layer norm backward {rows} x {d}", flush=True)
    gen = torch.Generator().manual_seed(rows)
    x, gain = torch.randn((rows, d), generator=gen).bfloat16(), (1 + 0.1 * torch.randn(d, generator=gen)).bfloat16()
    dy = _ints((rows, d), 3, -2, 3).bfloat16()
    _, mean, rstd = mtf.layer_norm_fwd(x.cuda(), gain.cuda(), torch.zeros_like(gain).cuda(), 1e-6)
    dx, dgain, dbias = mtf.layer_norm_bwd(x.cuda(), gain.cuda(), mean, rstd, dy.cuda())
    assert torch.equal(dbias.cpu(), dy.float().sum(0))
    xd, m, r = x.double(), mean.double().cpu()[:, None], rstd.double().cpu()[:, None]
    xh, g = (xd - m) * r, dy.double() * gain.double()
    ref = r * (g - g.mean(1, keepdim=True) - xh * (g * xh).mean(1, keepdim=True))
    # one bf16 rounding (2^-9 of the value), fp32 before it
    assert ((dx.double().cpu() - ref).abs() <= 2.0**-8 * ref.abs() + 1e-5 * r).all()
    terms = (dy.double() * xh).abs().sum(0)
    assert ((dgain.double().cpu() - (dy.double() * xh).sum(0)).abs() <= (rows + 8) * 2.0**-24 * terms + 1e-30).all()


@pytest.mark.parametrize("rows,d,groups", [(4096, 1024, 256), (33, 520, 5), (4096, 2048, 512), (33, 2048, 9)])
def test_layer_norm_backward_reports_its_bytes(rows, d, groups):
    """x, dy in and dx out in bf16, two fp32 statistics per row, the column partials of its workgroups."""
    x = _ints((rows, d), 1).bfloat16().cuda()
    _, mean, rstd = mtf.layer_norm_fwd(x, x[0], x[0], 1e-6)
    mtf.timing_enable(True)
    mtf.layer_norm_bwd(x, x[0], mean, rstd, x)
    got = {t["kernel"]: t["bytes"] for t in mtf.timing_collect()}
    mtf.timing_enable(False)
    assert got["layer_norm_bwd_kernel"] == rows * d * 6 + 8 * rows + groups * 2 * d * 4


@pytest.mark.parametrize("count", [0, 1, 127, 128, 129, 256, 257, 512, 513, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("d", [8, 1024, 1032])
def test_embedding_gradient_exact(count, d):
    """Small integers; a row that no token hits, one that most do, ids outside the stripe."""
    print(f"embedding gradient {count} tokens, width {d}", flush=True)
    ids = torch.randint(0, 40, (count,), generator=torch.Generator().manual_seed(count), dtype=torch.int32)
    ids[::2] = 11
    ids[ids == 13] = 39
    de = _ints((count, d), 5, -2, 3).bfloat16()
    got = mtf.embedding_grad_local(ids.cuda(), de.cuda(), 16, 8).cpu()
    ref = torch.zeros((40, d)).index_add_(0, ids.long(), de.float())[8:24]
    assert torch.equal(got, ref)
