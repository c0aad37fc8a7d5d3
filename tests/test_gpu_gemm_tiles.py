"""The tile shapes the bf16 GEMM picks for outputs of at most one tile per CU, each with ragged edges in
every direction, all operand layouts and epilogues.  Small integer operands: every product and partial
sum is exact in fp32 (|sum| < 2^24), so the results are compared bit for bit whatever the order."""
import pytest
import torch

import paper_1811_02084_amd as mtf

pytestmark = pytest.mark.gpu

# (m, n, k) -> the tile the rule takes there, as its kernel name starts
TILES = {"TileCfg<64, 64, 1, 1, 4, 128, 8, 2>": [(200, 136, 136), (8, 8, 8), (1, 72, 264)],
         "TileCfg<64, 64, 1, 1, 4, 128, 8, 4>": [(200, 136, 776), (65, 56, 1032)],
         "TileCfg<128, 64, 2, 1, 4, 128, 8, 3>": [(1032, 1544, 904)],
         "TileCfg<128, 128, 2, 2, 2, 64, 8, 4>": [(2056, 1544, 520)],
         "TileCfg<128, 128, 2, 2, 1, 64, 8, 2>": [(2056, 1544, 200)]}
CASES = [(tile, size) for tile, sizes in TILES.items() for size in sizes]


def _ints(shape, seed):
    gen = torch.Generator().manual_seed(seed)
    return torch.randint(-2, 3, shape, generator=gen).to(torch.bfloat16)


def _operands(m, n, k):
    return _ints((m, k), 1), _ints((k, n), 2)


@pytest.mark.parametrize("tile,size", CASES)
@pytest.mark.parametrize("da", ["mk", "km"])
@pytest.mark.parametrize("db", ["kn", "nk"])
def test_layouts(tile, size, da, db):
    m, n, k = size
    if da == "km" and m % 8:
        pytest.skip("an m-contiguous operand needs m divisible by 8 on this path")
    print(f"gemm tile {tile} {size} {da},{db}", flush=True)
    a, b = _operands(m, n, k)
    ref = a.float() @ b.float()
    ag = (a if da == "mk" else a.t().contiguous()).cuda()
    bg = (b if db == "kn" else b.t().contiguous()).cuda()
    mtf.timing_enable(True)
    got = mtf.einsum_local(ag, da, bg, db, "mn", out_dtype=torch.float32)
    names = [t["kernel"] for t in mtf.timing_collect()]
    mtf.timing_enable(False)
    assert len(names) == 1 and tile in names[0], names
    assert torch.equal(got.cpu(), ref)
    got16 = mtf.einsum_local(ag, da, bg, db, "mn", out_dtype=torch.bfloat16)
    assert torch.equal(got16.cpu(), ref.bfloat16())


@pytest.mark.parametrize("tile,size", CASES)
def test_epilogues(tile, size):
    m, n, k = size
    print(f"gemm epilogues {tile} {size}", flush=True)
    a, b = _operands(m, n, k)
    ref = a.float() @ b.float()
    aux, bias, old = _ints((m, n), 3), _ints((n,), 4), _ints((m, n), 5).float()
    run = lambda **kw: mtf.einsum_local(a.cuda(), "mk", b.cuda(), "kn", "mn", **kw).cpu()
    assert torch.equal(run(out_dtype=torch.float32, epi=mtf.EPI_RELU), ref.clamp(min=0))
    for dt in (torch.float32, torch.bfloat16):
        got = run(out_dtype=dt, epi=mtf.EPI_MASK_GT0, aux=aux.cuda())
        assert torch.equal(got, torch.where(aux > 0, ref, torch.zeros(())).to(dt))
        got = run(out_dtype=dt, epi=mtf.EPI_BIAS_RELU, aux=bias.cuda())
        assert torch.equal(got, (ref + bias.float()).clamp(min=0).to(dt))
        got = run(alpha=0.5, accumulate=True, out=old.to(dt).cuda())
        assert torch.equal(got, (0.5 * ref + old).to(dt))


@pytest.mark.parametrize("b,m,n,k", [(12, 808, 144, 1032), (10, 448, 296, 2056)])
@pytest.mark.parametrize("da", ["mk", "km"])
def test_batches_of_few_tiles(b, m, n, k, da):
    """The products of a batch are dealt to the 8 XCDs one by one.  12 of 808x144: 128x64 tiles would be two rounds on
    seven XCDs where 128x128 tiles are one; 10 of 448x296: one round of either, of a shorter stream on
    128x128, since the few tiles of a product on an XCD share little."""
    print(f"gemm batch {b} x {m}x{n}x{k} {da}", flush=True)
    a, w = _ints((b, m, k), 6), _ints((b, k, n), 7)
    ref = torch.stack([x.float() @ y.float() for x, y in zip(a, w)])
    ag = (a if da == "mk" else a.transpose(1, 2).contiguous()).cuda()
    mtf.timing_enable(True)
    got = mtf.einsum_local(ag, "b" + da, w.cuda(), "bkn", "bmn", out_dtype=torch.float32)
    names = [t["kernel"] for t in mtf.timing_collect()]
    mtf.timing_enable(False)
    assert torch.equal(got.cpu(), ref)
    assert len(names) == 1 and "TileCfg<128, 128, " in names[0], names


@pytest.mark.parametrize("size,parts", [((200, 136, 160), 2), ((136, 72, 4096), 4), ((1032, 1544, 1824), 2)])
def test_ranges(size, parts):
    m, n, k = size
    print(f"gemm ranges {size} x {parts}", flush=True)
    a, b = _operands(m, n, k)
    got = mtf.einsum_local_kranges(a.cuda(), "mk", b.cuda(), "kn", "mn", parts)
    for p, g in zip(range(parts), got):
        lo, hi = p * k // parts, (p + 1) * k // parts
        assert torch.equal(g.cpu(), a[:, lo:hi].float() @ b[lo:hi].float())
