// Which kernel takes an fp32 contraction of the form C[z][m][n] = sum_k A(z, m, k) B(z, k, n) (n innermost in
// C).  Host arithmetic on sizes only.
#pragma once
#include <algorithm>
#include <cstdint>

namespace mtf {

enum Fp32Kernel { kFp32Generic = 0, kFp32Tile16 = 1, kFp32Tile64 = 2 };

// Estimates in microseconds, fitted to 530 launches of all three (batches 1 .. 60000, M and N 1 .. 500000, K
// 2 .. 800, all operand orders; the chosen kernel is within 1 % of the fastest one on average):
//   generic: a thread per output walks k one load round trip at a time (0.144 us per k); beyond the waves
//     that hide behind that trip, what a wave's loads cost: more, the more cache lines its 64 outputs
//     touch per k (operands strided across the lanes), once k outgrows a line;
//   16 x 16 tiles: a round trip and two barriers per 128 k, and a workgroup per tile, full or not;
//   64 x 64 tiles: 0.1 us per k for a lone workgroup, else the tiles' FMAs and staging, full or not.
// So outputs of few rows or columns (batches of them above all) stay generic until k is long: generic / 16 /
// 64, batch 60000 of 4x1x32 20 / 143 / 389 us; 16384 of 8x8x4 10 / 34 / 53, of 8x4x256 227 / 158 / 650;
// 500000x2x2 8.5 / 60 / 27; 1x500000x64 43 / 103 / 95, with B strided 258 / 114 / 98.
inline Fp32Kernel fp32_kernel(int64_t M, int64_t N, int64_t K, int64_t batch, bool a_kcontig, bool b_kcontig) {
  const int64_t most = INT32_MAX / 2;  // the tiled kernel's ints; batch is its grid's y
  if (M > most || N > most || K > most || batch > 65535) return kFp32Generic;
  auto ceil_div = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t tiles16 = ceil_div(M, 16) * ceil_div(N, 16), tiles64 = ceil_div(M, 64) * ceil_div(N, 64);
  const double k = (double)K, waves = (double)batch * (double)M * (double)N / 64;
  // cache lines 64 neighbouring outputs touch per k in B (columns) and A (rows)
  const int64_t cols = std::min<int64_t>(N, 64), rows = std::min(M, std::max<int64_t>(1, 64 / cols));
  const int64_t slices = std::min(batch, std::max<int64_t>(1, 64 / (cols * rows)));
  const double lines = (double)slices * (double)((b_kcontig ? cols : ceil_div(cols, 32)) + (a_kcontig ? rows : 1));
  const double generic =
      4.4 + k * (0.144 + std::max(0.0, waves - 976) * (60 + 2.5 * lines * std::min(1.0, k / 32)) * 1e-6);
  const double t16 = 2.9 + 2.0 * (double)ceil_div(K, 128) + 0.0096 * k + (double)(tiles16 * batch) * (1.7 + 0.027 * k) * 1e-3;
  const double t64 = 4.8 + std::max(0.1 * k, (double)(tiles64 * batch) * (1.8 + 0.16 * k) * 1e-3);
  // 256 threads per tile: a grid of fewer than 2^32 threads
  const int64_t limit = (INT64_C(1) << 32) / 256;
  if (t64 <= std::min(generic, t16) && tiles64 < limit) return kFp32Tile64;
  if (t16 <= generic && tiles16 < limit) return kFp32Tile16;
  return t64 <= generic && tiles64 < limit ? kFp32Tile64 : kFp32Generic;
}

}  // namespace mtf
