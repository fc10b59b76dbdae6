// Host side of the small-batch GEMM (gemm_skinny.hip): where qx_gemm takes it. Plain C++, so
// that tests can include it on its own.
#pragma once

#include "qx_internal.h"

namespace qx {

// Formats with a form for a third activation tile (33 to 48 rows).
constexpr bool third_tile(int bits, int kind, int group) {
  return kind != QX_Q4X && !(kind == QX_CODEBOOK && group == 32) && !(kind == QX_CODEBOOK && bits == 4 && group == 64);
}

// Whether qx_gemm runs m rows on this kernel. Beyond 16 rows (a second activation tile,
// every code decoded again for it) only up to 32 of at most 32 chunks with one round of
// blocks (us at m = 24 / 32 against the matrix-core GEMM of gemm.hip, weights rotated over
// four copies: 11008x4096 uniform-3 g64 16.8 / 17.5 vs 21.6 / 21.5; 12288x4096 codebook-3
// 15.0 / 15.8 vs 19.9 / 19.9; 4096x4096 codebook-3 8.9 / 9.1 vs 14.8 / 14.9; 22016 rows, two
// rounds: 28.5 / 30.2 vs 24.5 / 24.9; against gemm_tile.hip 15.1 vs 17.1 at 12288x4096
// codebook-3, m = 28, and 8.1 vs 9.6 at 4096x4096 uniform-4, m = 19, but 29.9 vs 18.4 at
// 11008x4096 uniform-3 g64, m = 64). A third tile only on matrices of up to 4096 rows and 29 to
// 32 chunks (4096x4096 at m = 33 / 40 / 48 against gemm_tile.hip: codebook-4 g128 10.2 / 10.3 /
// 10.9 vs 12.0 / 11.9 / 11.7, uniform-3 g64 9.2 / 9.5 / 10.1 vs 10.4 / 10.2 / 10.2, uniform-4
// g128 9.5 / 9.8 / 10.3 vs 10.4 / 10.3 / 10.2, on 1376 rows 9.1 vs 8.9 at m = 40; codebook-3 g32
// 12.0 vs 10.9 at m = 33; 4096x3712 codebook-3 g128 9.9 vs 9.2 at m = 48, 3072x3712 uniform-4
// g128 9.0 vs 8.7 at m = 33). Up to 16 rows: measured against the
// small-batch GEMV-style kernel (m <= 4) and the matrix-core GEMM in all thirteen formats
// (us, 3-bit uniform g64 at m = 2 / 8 / 16: 11008x4096 8.4 / 9.0 / 9.9 against 9.2 / 15.7 /
// 15.8; 4096x4096 4.9 / 5.5 / 6.2 against 5.5 / 8.7 / 8.7). Rows of more than 32 chunks
// (two to four items per lane, the next item's codes requested as each item is staged),
// at m = 2 / 3 / 4 / 5 / 8 / 16: 4096x11008 uniform-3 g64 9.1 at m = 2 against 10.9 for the
// GEMV-style kernel, 5120x13824 18.3 against 16.2 (uniform codes at m = 2 on four items
// stay there); 4-bit codebooks of 128 codes faster at every m (4096x11008 12.4 / 12.8 /
// 12.9 / 13.2 / 13.8 / 15.8 against 13.7 / 18.0 / 18.4 / 17.1 / 17.3 / 19.4; 5120x13824
// 24.2 / .. / 34.1 against 24.5 / .. / 40.9), of 64 codes on two items up to m = 5 and on
// three up to m = 3 (4096x8192 12.3 / 13.9 / 15.1 / 16.6 / 22.2 against 15.2 / 16.8 / 17.1
// / 19.5 / 19.6); Q4X on two items up to m = 8 (4096x8192 9.8 / 10.0 / 10.1 / 11.8 / 15.2
// against 10.1 / 12.0 / 12.4 / 17.6 / 17.5) and on three at m = 3, 4 (14.1 / 15.8 against
// 16.2 / 16.5); 4-bit codebooks of 32 codes nowhere (their tables spill registers).
inline bool skinny_applies(const qx_desc* d, int m) {
  const int C = d->k / 128, J = (C + 31) / 32;  // items per lane (8 waves of 4 chunks)
#ifdef QX_SKINNY_FORCE
  return m >= 2 && m <= QX_SKINNY_MAX_M && J <= 4;
#endif
  if (m < 2 || m > QX_SKINNY_MAX_M || J > 4) return false;
  const bool cb = d->kind == QX_CODEBOOK, q4x = d->kind == QX_Q4X;
  if (m > 16) {  // 16-row activation tiles in turn, every code decoded again for each
    const int rf = d->n >= 8192 ? 3 : 1;
    if (J > 1 || (d->n + 16 * rf - 1) / (16 * rf) > 256 || q4x || (cb && d->bits == 4 && d->group <= 64)) return false;
    if (m <= 32) return true;
    if (!third_tile(d->bits, d->kind, d->group) || d->n > 4096 || C <= 28) return false;
    if (cb ? d->bits == 4 : d->bits == 3 || d->group == 32) return m <= (d->n >= 2048 && (cb || C > 30) ? 48 : 40);
    return C > 30 && m <= 40 && (d->n >= 2048 || (cb && d->group == 128));
  }
  if (cb && d->bits == 4) {
    if (d->group == 128) return true;
    if (d->group == 64) return J == 1 || (J == 2 && m <= 5) || (J == 3 && m <= 3);
    return false;
  }
  if (q4x) return J == 1 ? (m >= 3 || d->n <= 4096) : J == 2 ? m <= 8 : J == 3 && m >= 3 && m <= 4;
  if (J == 4 && m == 2) return cb;  // uniform codes at m = 2 on rows of 97-128 chunks: GEMV-style
  return true;
}

}  // namespace qx
