"""fp32 contractions that fold to a matrix product, through LDS tiles: all operand orders, odd sizes at the
edges of tiles and k-chunks, both tile sizes (721 x 1013 outputs take 64 x 64 tiles in every order), batches and
epilogues.  Every output is one chain of fused multiply-adds in ascending k, so it is within K * 2^-24
of sum |a b| of the exact value; small integers are exact."""
import numpy as np
import pytest
import torch

import paper_1811_02084_amd as mtf
from oracle.einsum import einsum, einsum_abs
from helpers import f64, named

pytestmark = pytest.mark.gpu

ORDERS = [("mk", "kn", "mn"), ("km", "kn", "mn"), ("mk", "nk", "mn"), ("km", "nk", "nm"), ("bmk", "bkn", "bmn"),
          ("bmhk", "bnhk", "bhmn"), ("mhk", "hkn", "mn"), ("k", "kn", "n"), ("mk", "k", "m")]
SIZES = [dict(m=1, n=1, k=2, b=2, h=3), dict(m=17, n=15, k=5, b=2, h=3), dict(m=16, n=33, k=127, b=3, h=2),
         dict(m=5, n=64, k=261, b=2, h=2), dict(m=577, n=530, k=37, b=1, h=2), dict(m=130, n=67, k=33, b=17, h=2),
         dict(m=721, n=1013, k=70, b=1, h=1)]


def _rand(dims, sizes, seed, ints=False):
    rng = np.random.default_rng(seed)
    shape = [sizes[d] for d in dims]
    return torch.from_numpy((rng.integers(-2, 3, shape) if ints else rng.standard_normal(shape)).astype(np.float32))


@pytest.mark.parametrize("order", ORDERS, ids=[",".join(o) for o in ORDERS])
@pytest.mark.parametrize("sizes", SIZES, ids=[f"{s['m']}x{s['n']}x{s['k']}" for s in SIZES])
def test_orders(order, sizes):
    da, db, do = order
    print(f"folded fp32 einsum {order} {sizes}", flush=True)
    a, b = _rand(da, sizes, 1), _rand(db, sizes, 2)
    ins = [named(a, da), named(b, db)]
    got = mtf.einsum_local(a.cuda(), da, b.cuda(), db, do)
    ref, ref_abs = einsum(ins, do).data, einsum_abs(ins, do).data
    terms = sizes["k"] * (sizes["h"] if "h" in da and "h" not in do else 1)
    assert np.all(np.abs(f64(got) - ref) <= (terms + 1) * 2.0**-24 * ref_abs)


@pytest.mark.parametrize("sizes", SIZES[1:5] + SIZES[6:], ids=[f"{s['m']}x{s['n']}x{s['k']}" for s in SIZES[1:5] + SIZES[6:]])
@pytest.mark.parametrize("da", ["mk", "km"])
def test_epilogues_exact(sizes, da):
    db, do = "kn", "mn"
    print(f"folded fp32 epilogues {da} {sizes}", flush=True)
    a, b = _rand(da, sizes, 3, True), _rand(db, sizes, 4, True)
    am = a if da == "mk" else a.t()
    ref = am @ b
    aux, bias, old = _rand(do, sizes, 5, True), _rand("n", sizes, 6, True), _rand(do, sizes, 7, True)
    run = lambda **kw: mtf.einsum_local(a.cuda(), da, b.cuda(), db, do, **kw).cpu()
    for dt in (torch.float32, torch.bfloat16):
        assert torch.equal(run(out_dtype=dt, epi=mtf.EPI_RELU), ref.clamp(min=0).to(dt))
        assert torch.equal(run(out_dtype=dt, epi=mtf.EPI_BIAS, aux=bias.cuda()), (ref + bias).to(dt))
        assert torch.equal(run(out_dtype=dt, epi=mtf.EPI_MASK_GT0, aux=aux.cuda()),
                           torch.where(aux > 0, ref, torch.zeros(())).to(dt))
        assert torch.equal(run(alpha=0.5, accumulate=True, out=old.to(dt).cuda()), (0.5 * ref + old).to(dt))
    # an output whose two innermost dims are one column index: the bias runs over the last of them
    n2 = sizes["n"] * 3
    b3, bias3 = _rand("kn", dict(sizes, n=n2), 8, True), _rand("n", dict(n=3), 9, True)
    got = mtf.einsum_local(a.cuda(), da, b3.reshape(sizes["k"], -1, 3).cuda(), "knp", "mnp", epi=mtf.EPI_BIAS_RELU,
                           aux=bias3.cuda())
    assert torch.equal(got.cpu(), ((am @ b3).reshape(sizes["m"], -1, 3) + bias3).clamp(min=0))


@pytest.mark.parametrize("sizes", [dict(m=37, p=5, q=9, k=261), dict(m=721, p=11, q=93, k=70)],
                         ids=["16x16 tiles", "64x64 tiles"])
@pytest.mark.parametrize("da,db", [("mk", "kpq"), ("km", "kpq"), ("mk", "pqk"), ("km", "pqk")])
def test_bits_of_the_generic_kernel(sizes, da, db):
    """One chain of fused multiply-adds in ascending k on either kernel: the same bits.  An output with m between
    the column dims does not fold to a matrix product."""
    print(f"folded against generic {da},{db} {sizes}", flush=True)
    a, b = _rand(da, sizes, 11).cuda(), _rand(db, sizes, 12).cuda()
    aux, bias, old = _rand("mpq", sizes, 13).cuda(), _rand("q", sizes, 14).cuda(), _rand("mpq", sizes, 15).cuda()
    swap = lambda t: t.permute(1, 0, 2).contiguous()   # mpq <-> pmq
    mtf.timing_enable(True)
    mtf.einsum_local(a, da, b, db, "mpq")
    mtf.einsum_local(a, da, b, db, "pmq")
    names = {t["kernel"] for t in mtf.timing_collect()}
    mtf.timing_enable(False)
    assert names == {"einsum_folded_kernel", "einsum_generic_kernel"}
    for dt in (torch.float32, torch.bfloat16):
        for kw, other in ((dict(epi=mtf.EPI_RELU), {}), (dict(epi=mtf.EPI_BIAS, aux=bias), {}),
                          (dict(epi=mtf.EPI_MASK_GT0, aux=aux), dict(aux=swap(aux))),
                          (dict(alpha=0.3, accumulate=True, out=old.to(dt)), dict(out=swap(old).to(dt)))):
            folded = mtf.einsum_local(a, da, b, db, "mpq", out_dtype=dt, **kw)
            generic = mtf.einsum_local(a, da, b, db, "pmq", out_dtype=dt, **{**kw, **other})
            assert torch.equal(folded, swap(generic)), (dt, sorted(kw))
