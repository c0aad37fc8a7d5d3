// Which fp32 contractions of the form C[z][m][n] = sum_k A(z, m, k) B(z, k, n) go to the tiled kernel of
// einsum_local.hip.  Host arithmetic on sizes only.
#pragma once
#include <cstdint>

namespace mtf {

// Whether a launch of one workgroup of 256 threads per 64 x 64 tile is possible: sizes and tile numbers fit
// the kernel's ints, the batch fits the grid's y, and the grid's x has fewer than 2^32 threads.
inline bool folded_fits(int64_t M, int64_t N, int64_t K, int64_t batch) {
  const int64_t most = INT32_MAX / 2;
  if (M > most || N > most || K > most || batch > 65535) return false;
  return ((M + 63) / 64) * ((N + 63) / 64) < (INT64_C(1) << 32) / 256;
}

}  // namespace mtf
