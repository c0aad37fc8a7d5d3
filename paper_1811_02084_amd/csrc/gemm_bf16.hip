// Host side of the bf16 MFMA GEMM family: which problems the kernels take, and which tile shape
// runs a given launch.  The kernel template is in gemm_bf16_kernel.h; each tile shape is compiled
// in its own translation unit (gemm_bf16_<shape>.hip).  Every contraction of the Transformer-layer
// path lowers to this kernel (section "Performance Comparison": the einsums are where the
// computation time goes).
#include "gemm_bf16_kernel.h"


namespace mtf {

// The tile loaders keep per-lane byte offsets relative to the tile origin in 32 bits: up to
// (tile rows - 1) * ld * 2 + 2 * k-tile for a k-contiguous operand (256-row tile) and (k-tile - 1) * ld * 2 +
// 2 * tile columns for an mn-contiguous one.  Leading dims beyond this would wrap.
namespace {
bool ld_fits_32bit_offsets(int64_t ld, bool kcontig, int last_krow) {
  const int64_t worst = kcontig ? 255 * ld * 2 + (last_krow + 1) * 2 : last_krow * ld * 2 + 512;
  return ld >= 0 && ld < (INT64_C(1) << 40) && worst <= (int64_t)UINT32_MAX;
}
bool ld_fits_32bit_offsets(const GemmDesc& d, int last_krow) {
  bool fits = ld_fits_32bit_offsets(d.lda, d.a_kcontig, last_krow) && ld_fits_32bit_offsets(d.ldb, d.b_kcontig, last_krow);
  for (int p = 0; p < d.nextra && p < kMaxGroup - 1; ++p)
    fits = fits && ld_fits_32bit_offsets(d.extra[p].lda, d.a_kcontig, last_krow) &&
           ld_fits_32bit_offsets(d.extra[p].ldb, d.b_kcontig, last_krow);
  return fits;
}
}  // namespace

bool gemm_bf16_supported(const GemmDesc& d) {
  if (d.nseg < 1 || d.nseg > kMaxSegments) return false;
  if (!ld_fits_32bit_offsets(d, 63)) return false;
  if (d.M <= 0 || d.N <= 0 || d.M > INT32_MAX || d.N > INT32_MAX) return false;
  if (d.lda % 8 || d.ldb % 8 || d.ldc % 4 || d.N % 8) return false;
  if (!d.a_kcontig && d.M % 8) return false;
  if (d.sA0 % 8 || d.sA1 % 8 || d.sB0 % 8 || d.sB1 % 8 || d.sC0 % 4 || d.sC1 % 4) return false;
  for (int s = 0; s < d.nseg; ++s) {
    if (d.K[s] < 0 || d.K[s] > INT32_MAX) return false;
    if ((d.a_kcontig || d.b_kcontig) && d.K[s] % 8) return false;
    if (!aligned16(d.A[s]) || !aligned16(d.B[s])) return false;
  }
  if (!aligned16(d.C) || (d.epi == MTF_EPI_MASK_GT0 && (!d.aux || !aligned16(d.aux)))) return false;
  if (d.bias && (((uintptr_t)d.bias & 7) || d.nextra > 0)) return false;
  if (d.row_scale && d.nextra > 0) return false;
  if (d.residual && (!aligned16(d.residual) || !d.out_bf16 || d.accumulate || d.nextra > 0 || d.batch0 * d.batch1 != 1))
    return false;
  if (d.batch0 * d.batch1 > 65535) return false;
  if (d.nextra < 0 || d.nextra > kMaxGroup - 1) return false;
  if (d.nextra > 0 && ((1 + d.nextra) * d.nseg > kMaxSlots || d.batch0 * d.batch1 != 1 || d.accumulate ||
                       d.epi != MTF_EPI_NONE))
    return false;
  for (int p = 0; p < d.nextra; ++p) {
    const GemmDesc::Extra& e = d.extra[p];
    if (e.M <= 0 || e.N <= 0 || e.M > INT32_MAX || e.N > INT32_MAX) return false;
    if (e.lda % 8 || e.ldb % 8 || e.ldc % 4 || e.N % 8 || (!d.a_kcontig && e.M % 8)) return false;
    for (int s = 0; s < d.nseg; ++s) {
      if (e.K[s] < 0 || e.K[s] > INT32_MAX) return false;
      if ((d.a_kcontig || d.b_kcontig) && e.K[s] % 8) return false;
      if (!e.A[s] || !e.B[s] || !aligned16(e.A[s]) || !aligned16(e.B[s])) return false;
    }
    if (!e.C || !aligned16(e.C)) return false;
  }
  return true;
}

namespace {
struct Choice {
  double cost;
  int (*launch)(const GemmDesc&, const GemmArgs&, int, hipStream_t);
};

// Tile choice by a cost model in microseconds, fitted to kernel traces of the layer's launches
// and to single launches of [993..8192, 512..8192] outputs with 256..4096 contracted (operands
// from memory): a shape's time is the rounds of tiles on the busiest XCD over the slots an XCD has for
// it, each round a fixed part (prologue and epilogue) plus what the tile takes per 1024 contracted.
// What bounds a tile is mostly its operand stream: these launches take in 7 to 14 TB/s in all (the more, the more
// of it the tiles of an XCD share), so a tile costs about its bytes, (BM + BN) * K * 2, and the widest
// tile that still gives every CU one wins:
//   256x256  31.2 us per 1024 + 5      256x128  17.3 (A along k; else 19.5) + 6
//   128x128, two workgroups per CU: 19.5 for the pair + 2; one per CU in k-groups: 10 + 3.7
//   128x64   7.2 + 4.2                 64x64    4.3 + 4 (one per CU), 8.6 for two sharing a CU + 3.2
// Measured at the edges: 993x1024x1024 (256 tiles of 64x64) 8.5 us against 12.6 on 128x128 (the
// four-wave 128x128 kernel these shapes used before: 13.8), 2048x1024x1024 (256 of 128x64) 11.1
// against 13.3 / 11.9 on 128x128 / 64x64, 4096x1024x4096 (256 of 128x128) 44 against 58 on either side,
// 96x256x256 (8 of 64x64) 4.3 against 6.5.
// The busiest XCD, not the chip: a batch's products are cut into eighths one by one, so 12 of 808x144 make
// 36 tiles of 128x64 (21 = 7 x 3) for each of seven XCDs and none for the eighth: two rounds, 87 us at
// K = 4112 against 51 on 128x128 (2 x 12 tiles).  And up to 8 tiles of a product on an XCD share so little
// of their operands that the XCD takes in 0.95 to 1.2 TB/s: a floor under the shapes with the longest streams
// (10 x 448x296x8192: 128x64 97, 64x64 93, 128x128 83 us).  Over 820 drawn launches the choice is within
// 1 % of the fastest tile on average.
Choice choose_tile(const GemmDesc& d) {
  const int64_t batch = d.batch0 * d.batch1;
  auto busiest = [&](int bm, int bn) {  // tiles on the XCD that gets the most, as the kernel deals them out
    const int64_t first = ceil_div(d.M, bm) * ceil_div(d.N, bn);
    if (d.nextra == 0) return batch * ceil_div(first, 8);
    int64_t tiles[kMaxGroup] = {first}, most = first;
    bool same = true;
    for (int p = 0; p < d.nextra; ++p) {
      tiles[p + 1] = ceil_div(d.extra[p].M, bm) * ceil_div(d.extra[p].N, bn);
      most = std::max(most, tiles[p + 1]);
      same = same && tiles[p + 1] == first;
    }
    const int n = 1 + d.nextra;
    const int64_t eighth = ceil_div(most, 8);  // of the widest problem's grid
    if (same && 8 % n == 0) return eighth * n;
    int64_t sum = 0;
    for (int p = 0; p < n; ++p) sum += std::min(tiles[p], eighth);
    return sum;
  };
  auto per1024 = [&](int bk) {  // the longest problem's contracted length in whole k-tiles, / 1024
    double most = 0;
    for (int p = 0; p < 1 + d.nextra; ++p) {
      double k = 0;
      for (int s = 0; s < d.nseg; ++s) k += (double)(ceil_div(p ? d.extra[p - 1].K[s] : d.K[s], bk) * bk);
      most = std::max(most, k);
    }
    return most / 1024.0;
  };
  auto unshared = [&](int bm, int bn) {
    if (batch == 1 || ceil_div(ceil_div(d.M, bm) * ceil_div(d.N, bn), 8) > 8) return 0.0;
    double k = 0;
    for (int s = 0; s < d.nseg; ++s) k += (double)d.K[s];
    const int64_t rows = std::min<int64_t>(bm, d.M) + std::min<int64_t>(bn, d.N);
    return (double)(busiest(bm, bn) * rows) * k * 2 / 1.1e6 + 3.0;
  };
  auto rounds = [](int64_t tiles, int per_cu) { return (double)ceil_div(tiles, 32 * per_cu); };  // 32 CUs per XCD
  const double k64 = per1024(64), k128 = per1024(128);
  const int64_t small_tiles = busiest(128, 128), tiny_tiles = busiest(64, 64);
  const double pair_rate = batch == 1 ? std::min(19.5, 15.2 + 0.5 * (double)(small_tiles - 33)) : 19.5;
  const Choice choices[] = {
      {rounds(busiest(256, 256), 1) * (31.2 * k64 + 5.0), launch_large},
      {rounds(busiest(256, 128), 1) * ((d.a_kcontig ? 17.3 : 19.5) * k64 + 6.0), launch_split},
      // two small tiles share a CU and cover each other (and take less time while few CUs have two: 34 on
      // an XCD, 15.2 per 1024); with at most one per CU, k-groups do that
      // (from 448 contracted on: below, their exchange costs more: 4096x1024x256 9.7 us against 8.8)
      small_tiles > 32 ? Choice{rounds(small_tiles, 2) * (pair_rate * k64 + 2.0), launch_small}
                       : Choice{10.0 * k64 + 3.7, k64 > 448 / 1024.0 ? launch_pair : launch_small},
      {std::max(rounds(busiest(128, 64), 1) * (7.2 * k128 + 4.2), unshared(128, 64)), launch_narrow},
      // 64x64 with a deep ring and the CU to itself, or two with a shallow one: the deep ring pays
      // from about 6 k-tiles on (993x1024: K = 512 7.2 against 7.0 us, K = 1024 8.5 against 9.2)
      {std::max(rounds(tiny_tiles, 1) * (4.3 * k128 + 4.0), unshared(64, 64)), k128 >= 0.75 ? launch_tiny_deep : launch_tiny},
      {std::max(rounds(tiny_tiles, 2) * (8.6 * k128 + 3.2), unshared(64, 64)), launch_tiny},
  };
  // the k-tiles of 128 need twice the reach in the loaders' 32-bit offsets
  const bool reach128 = ld_fits_32bit_offsets(d, 127);
  const Choice* best = &choices[0];
  for (int i = 1; i < 6; ++i)
    if ((i < 3 || reach128) && choices[i].cost < best->cost) best = &choices[i];
  return *best;
}
}  // namespace

double gemm_bf16_cost_us(const GemmDesc& d) { return choose_tile(d).cost; }

int gemm_bf16_launch(const GemmDesc& d, hipStream_t stream) {
  if (!gemm_bf16_supported(d)) return fail(MTF_ERR_UNSUPPORTED, "GEMM shape/alignment");
  GemmArgs a;
  for (int s = 0; s < kMaxSlots; ++s) {
    a.A[s] = s < d.nseg ? d.A[s] : d.A[0];
    a.B[s] = s < d.nseg ? d.B[s] : d.B[0];
    a.K[s] = s < d.nseg ? (int)d.K[s] : 0;
  }
  for (int s = 0; s < kMaxGroup; ++s) {
    a.M[s] = (int)d.M;
    a.N[s] = (int)d.N;
    a.lda[s] = d.lda;
    a.ldb[s] = d.ldb;
    a.ldc[s] = d.ldc;
    a.C[s] = d.C;
    a.tiles_m[s] = a.tiles_n[s] = 0;
  }
  a.nseg = d.nseg;
  a.ngroup = 1 + d.nextra;
  for (int p = 0; p < d.nextra; ++p) {
    const GemmDesc::Extra& e = d.extra[p];
    for (int s = 0; s < d.nseg; ++s) {
      const int slot = (p + 1) * d.nseg + s;
      a.A[slot] = e.A[s]; a.B[slot] = e.B[s]; a.K[slot] = (int)e.K[s];
    }
    a.C[p + 1] = e.C;
    a.M[p + 1] = (int)e.M; a.N[p + 1] = (int)e.N;
    a.lda[p + 1] = e.lda; a.ldb[p + 1] = e.ldb; a.ldc[p + 1] = e.ldc;
  }
  a.aux = d.aux;
  a.bias = d.bias;
  a.row_scale = d.row_scale;
  a.alpha = d.alpha;
  a.accumulate = d.accumulate || d.residual ? 1 : 0;
  a.old = d.residual ? static_cast<const void*>(d.residual) : d.C;
  a.batch1 = (int)d.batch1;
  a.sA0 = d.sA0; a.sA1 = d.sA1; a.sB0 = d.sB0; a.sB1 = d.sB1; a.sC0 = d.sC0; a.sC1 = d.sC1;
  const int batch = (int)(d.batch0 * d.batch1);
  return choose_tile(d).launch(d, a, batch, stream);
}

}  // namespace mtf
