// Host side of the tiled GEMM (gemm_tile.hip): the layout of its block shapes and the choice
// between them and the older kernels. Plain C++, so that tests can include it on their own.
#pragma once

#include "qx_internal.h"

namespace qx {
namespace tile {

constexpr int kLdsBytes = 160 * 1024;
constexpr int kXRow = 128;  // LDS bytes of one activation row of a round: 64 fp16

template <int BITS, int KIND, int G, int MT, int NT, int WM, int SC, int KS>
struct TileShape {
  static constexpr int kThreads = KS > 1 ? 64 * KS : 256 * WM;
  static constexpr int WN = KS > 1 ? 1 : 4;  // waves on different weight rows
  static constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN, NG = 128 / G;
  static constexpr int kTable = 2 << BITS;  // bytes of a codebook group's table
  // LDS planes of BN rows x kMUnit bytes that hold a chunk's groups as the decoders take them
  // (prepared once a block when they are stored): uniform (s, s) and -(1024 + z), the lookup
  // tables of 8 entries, or the Q4X scales and selectors
  static constexpr int kMUnit = KIND == QX_CODEBOOK ? 16 : 8;
  static constexpr int kMPlanes = KIND == QX_UNIFORM ? NG : KIND == QX_Q4X ? 1 : NG * kTable / 16;  // per chunk
  static constexpr int kXBuf = BM * kXRow, kCBuf = BITS * BN * SC * 16, kMBuf = kMPlanes * SC * BN * kMUnit;
  static constexpr int kWaveLds = (KS > 1 ? 1 : 2) * kXBuf + 2 * (kCBuf + kMBuf);  // KS > 1: of one wave
  static constexpr int kLds = KS * kWaveLds + (KIND == QX_Q4X ? 128 : 0);
  // waves on a SIMD for which registers are allocated
  static constexpr int kWaves = KS > 1 ? KS / 4 * (2 * kLds <= kLdsBytes ? 2 : 1) : WM == 2 || 2 * kLds <= kLdsBytes ? 2 : 1;
};

// Where a lane's load reads, in bytes from its buffer's start: `lane`, which is held against
// the buffer's size (a load past it reads 0), and `scalar`, which the compiler defines as
// outside that check and the hardware as taken from the size. All that can leave the buffer is
// therefore in `lane` or in the buffer itself: rows past the matrix, and with SC = 2 the chunk,
// since a super-round can begin in the last one. `scalar` stays within a row.
struct ReadAt {
  int lane, scalar;
};

// The loads of thread t of NTH that stage half h of chunk c's activations, and piece i of the
// codes and group constants of the super-round that begins with chunk c.
template <int BITS, int KIND, int G, int MT, int NT, int WM, int SC, int KS, bool A8>
struct TileReads {
  using TS = TileShape<BITS, KIND, G, MT, NT, WM, SC, KS>;
  static constexpr int NTH = KS > 1 ? 64 : TS::kThreads, BN = TS::BN, NG = TS::NG;
  static constexpr int kXB = A8 ? 1 : 2;  // bytes of an activation
  static constexpr int kMRow = KIND == QX_UNIFORM ? 4 : KIND == QX_Q4X ? 2 : TS::kTable;  // of a group's word, scale or table
  static constexpr int XP = TS::BM * 8 / NTH;  // 16-byte activation pieces per thread and round
  static constexpr int CT = BITS * BN * SC, CP = (CT + NTH - 1) / NTH;
  static constexpr int MTOT = (KIND == QX_CODEBOOK ? TS::kMPlanes : 1) * BN * SC;  // table pieces, or rows x chunks
  static constexpr int MP = (MTOT + NTH - 1) / NTH;
  static constexpr int kXBytes = 8 * kXB, kCBytes = 16;  // of one load
  static constexpr int kMBytes = KIND == QX_UNIFORM ? 4 * NG : KIND == QX_Q4X ? 4 : 16;

  __host__ __device__ static ReadAt at(int lane, int scalar) {
    return SC == 1 ? ReadAt{lane, scalar} : ReadAt{lane + scalar, 0};
  }
  // Piece i of all threads has a buffer of its own, from its first row to the tile's last of
  // `rows` (a piece past them: the last row alone). With one buffer and the piece's row in
  // `lane` the additions cost 1.5 % (22016x4096 and 4096x11008 uniform-4 with 12288x4096 and
  // 4096x4096 codebook-3 at m = 2048: 903 against 887 us).
  __host__ __device__ static int x_row(int i, int rows) { return i * (NTH / 8) < rows ? i * (NTH / 8) : rows - 1; }
  __host__ __device__ static ReadAt x(int t, int c, int h, int k) {
    return {(t >> 3) * k * kXB + (t & 7) * 8 * kXB, (c * 128 + h * 64) * kXB};
  }
  // Code piece p of a super-round: SC neighbouring lanes take a row's SC pieces of a slice, in
  // an order that spreads 16 rows over the LDS banks.
  __host__ __device__ static ReadAt code(int t, int i, int c, int C) {
    const int p = t + i * NTH, q = p / SC, row = q % BN, cc = (p % SC) ^ (SC == 2 ? (row >> 3) & 1 : 0);
    if (BN * SC % NTH == 0)  // the slice is uniform
      return at((row * BITS * C + cc) * 16, (i * NTH / (BN * SC) * C + c) * 16);
    const int slice = q / BN < BITS ? q / BN : BITS - 1;
    return at(((row * BITS + slice) * C + cc) * 16, c * 16);
  }
  __host__ __device__ static int meta_piece(int t, int i) { return t + i * NTH < MTOT ? t + i * NTH : MTOT - 1; }
  __host__ __device__ static ReadAt meta(int t, int i, int c, int G_row) {
    const int p = meta_piece(t, i);
    if (KIND == QX_CODEBOOK)  // a row's tables of the super-round are one run
      return at(p / (TS::kMPlanes * SC) * G_row * kMRow + p % (TS::kMPlanes * SC) * 16, c * NG * kMRow);
    return at((p / SC * G_row + p % SC * NG) * kMRow, c * NG * kMRow);
  }
  // Q4X: the word with the selectors of the piece's chunk
  __host__ __device__ static ReadAt selectors(int t, int i, int c, int sel_words) {
    const int p = meta_piece(t, i);
    return {(p / SC * sel_words + (c + p % SC) / 8) * 4, 0};
  }
};

// Tile number -> (weight tile, activation tile) of nx x my. Workgroups are dealt to the 8 XCDs
// round-robin and every XCD takes an equal run of the tiles, which are numbered in `groups` of
// up to 8 activation tiles by consecutive weight tiles, so that the tiles in flight in its L2
// share both. (A run of whole weight tiles an XCD leaves units idle when they are few: 1024x5120
// uniform-4 g32 at m = 683, 22 x 11 tiles: 46 us against 31.) The groups are equal: a last one of a
// single activation tile would have one XCD read most of the codes (nine activation tiles,
// uniform-4 g128 14336x4096 at m = 1047: 217 us as 8 + 1, 148 as 5 + 4).
struct TileAt {
  int bn, bm;
};
__host__ __device__ inline TileAt tile_at(int tile, int nx, int my, int groups) {
  const int least = my / groups, more = my % groups;  // the first `more` groups have one more
  const int wide = more * (least + 1);
  const bool tail = tile >= wide * nx;
  const int rows = tail ? least : least + 1, at = tail ? tile - wide * nx : tile;
  const int g = at / (nx * rows), rem = at - g * nx * rows;
  return {rem / rows, (tail ? wide : 0) + g * rows + rem % rows};
}
inline int tile_groups(int my) { return (my + 7) / 8; }

// Block shapes, as activation x weight rows. Cost of a round of blocks with one, two or
// three of them on each of the 256 compute units, in us per 32 chunks of k (measured with
// uniform and codebook-3 g128 weights on 11008x4096, 4096x11008 and 4096x4096, m = 96 to
// 4096). A ranking more than a clock: over 1672 products of all formats that these shapes take
// (n = 1376 to 22016, k = 1024 to 11008, m = 24 to 4096) the sums over rounds are within 8 % of
// the measured time for 48 %, within 15 % for 80 % and within 25 % for 95 %; at worst 36 % too low
// (codebook-3 g64 int8 11008x1024, m = 2048: rows so short that the fixed part of a round counts) and 40 % too
// high (codebook-4 g64 4096x11008, m = 4096).
enum Shape { kA, kB, kC, kD, kE, kF, kG, kH, kShapes };
struct ShapeCost {
  int bm, bn, mt, nt, wm, sc;
  float us[3];
  int ks;
};
constexpr ShapeCost kShape[kShapes] = {
    {256, 256, 8, 4, 2, 2, {112.f, 0.f, 0.f}, 1},
    {128, 256, 8, 4, 1, 1, {80.f, 135.f, 0.f}, 1},
    {128, 192, 8, 3, 1, 1, {71.f, 121.f, 0.f}, 1},
    {128, 128, 8, 2, 1, 2, {60.f, 78.f, 0.f}, 1},
    {64, 128, 4, 2, 1, 2, {41.f, 54.f, 74.f}, 1},
    // k split over 8 waves: us[0] + us[1] a chunk for a round of 256 blocks (H: us[2] of it
    // for each round after the first, several blocks share a unit). Uniform-3 g64 at 32
    // chunks / 86 chunks, one round: F 18 / 35 us, G 13.5 / 28.5, H 9.9 / 20
    {64, 48, 4, 3, 1, 1, {8.f, 0.31f, 1.f}, 8},
    {64, 32, 4, 2, 1, 1, {4.6f, 0.278f, 1.f}, 8},
    {32, 32, 2, 2, 1, 1, {3.8f, 0.19f, 0.74f}, 8},
};

// Formats whose decoding leaves the registers of the 128 x 64 wave tile unspilled. With int8 rows
// codebook-3 spills 16 (g64: 38 products in B 14 % longer than in D, 18352x3072 at m = 1279 260 us and
// 188) or 6 (g128: 22 of them 2 % shorter than in D, 8192x5120 at m = 2048 192 us and 215).
template <int BITS, int KIND, int G, bool A8>
constexpr bool kLight = !A8 && (KIND == QX_UNIFORM || (KIND == QX_CODEBOOK && BITS == 3 && G >= 64));

// Shapes that are built: F, G and H not for the integer products of gemm_a8.hip, which split k
// themselves (11008x4096 uniform-3 g64 at m = 64: 24.1 us there, 22.9 with F; 4096x11008 24.5
// and 24.6 with H), nor F where its tables overflow LDS; the 128 x 64 wave tiles (A, B) for the light formats, and B for
// int8 rows of codebook-3 g128 and for codebook-4 g32, whose tables let one block of any shape on a compute unit.
template <int BITS, int KIND, int G, bool A8>
constexpr bool built(int s) {
  if (s == kA) return kLight<BITS, KIND, G, A8>;
  if (s == kB) return kLight<BITS, KIND, G, A8> || (KIND == QX_CODEBOOK && ((BITS == 4 && G == 32) || (BITS == 3 && G == 128)));
  // D is at no size the cheapest by the costs below with these codebooks, whose tables leave room
  // for one block of it on a compute unit, but for two of E
  if (s == kD) return !(KIND == QX_CODEBOOK && ((BITS == 3 && G == 32) || (BITS == 4 && G == 64)));
  if (s >= kF) return (KIND != QX_UNIFORM || !A8) && !(s == kF && KIND == QX_CODEBOOK && BITS == 4 && G == 32);
  return true;
}

template <int BITS, int KIND, int G, int S>
constexpr int per_unit() {  // blocks that fit a compute unit: LDS, and two or three by registers
  using TS = TileShape<BITS, KIND, G, kShape[S].mt, kShape[S].nt, kShape[S].wm, kShape[S].sc, 1>;
  constexpr int lds = kLdsBytes / TS::kLds, regs = S == kA ? 1 : S == kE ? 3 : 2;
  return lds < regs ? lds : regs;
}

// Cost of the heavier decoders over that of uniform codes on shapes C, D and E (the same
// sweep): 16-entry tables, tables of 32 or 64 codes.
template <int BITS, int KIND, int G, bool A8>
constexpr float decode_factor() {
  if (KIND == QX_Q4X) return 1.4f;
  if (KIND == QX_CODEBOOK)
    return (BITS == 4 ? (G == 32 ? 1.5f : G == 64 ? 1.35f : 1.2f) : G == 32 ? 1.2f : 1.f) * (A8 ? 1.08f : 1.f);
  return 1.f;
}

// A cost given for 32 chunks, at the matrix's chunks: 6 us of it fixed, with the scaled group
// sums of uniform codes 16 % of it (start and end of every round of blocks: shape D on 8192 rows
// at m = 1000, uniform-3 g128 at 8 / 32 / 86 chunks 36 / 94 / 228 us, C at m = 600 31 / 88).
template <int BITS, int KIND, int G, bool A8>
float at_chunks(float us, float chunks) {
  return A8 && KIND == QX_UNIFORM ? us * (0.16f + 0.02625f * chunks) : 6.f + (us - 6.f) * chunks / 32.f;
}

template <int BITS, int KIND, int G, bool A8, int S>
void consider(const qx_desc* d, int m, float& best, int& shape) {
  if constexpr (built<BITS, KIND, G, A8>(S)) {
    constexpr int per = per_unit<BITS, KIND, G, S>();
    const long blocks = (long)((d->n + kShape[S].bn - 1) / kShape[S].bn) * ((m + kShape[S].bm - 1) / kShape[S].bm);
    const long rest = blocks % (256 * per);
    const float us32 = decode_factor<BITS, KIND, G, A8>() *
                       ((float)(blocks / (256 * per)) * kShape[S].us[per - 1] + (rest ? kShape[S].us[(rest - 1) / 256] : 0.f));
    const float us = at_chunks<BITS, KIND, G, A8>(us32, (float)(d->k / 128));
    if (us < best) {
      best = us;
      shape = S;
    }
  }
}

// The same cost for the kernels that took these products before (gemm.hip, gemm_a8.hip),
// fitted to their times in the sweep:
//   fp16 activations, uniform: 128 x 256 blocks, from m = 384 where they take fewer rounds than
//     128 x 192, at 76 us a round (11008x4096 uniform-4 g128 at m = 1024 / 2048: 142 / 227 us); otherwise
//     128 x 64 tiles, 41 / 54 / 78 us for one, two or three of them on a unit (3-bit g32 57 and 85),
//     5 % less with 4-bit codes, up to 64 / 128 / 256 of them split over k (4096x4096 uniform-4 at m =
//     100 / 256 / 500: 20.6 / 25.8 / 37.6 us). All activation tiles of a weight tile run on one XCD,
//     so the weight tiles count as a multiple of 8 (10 and 13 of them: 1168x1280 uniform-3 g128, m =
//     2162, 35 us and 21.5 in E; 1636x11008, m = 2027, 153 and 133). Short rows take 2 us more unless
//     two tiles fill every unit (2432x640 uniform-3 g64, m = 1144: 17.8 and 14.0 in E; 16321x1024, m = 256:
//     20.9 and 22.9). Of 4000 products of two sweeps (n = 256 to 22016, k = 512 to 14336, m = 65 to 4096)
//     6 are more than 3 % slower than in gemm.hip (44 before the padded tiles and the 4-bit factor);
//   table formats: 64 x 64 tiles, 20 us + 0.07 us a tile (11008x4096 codebook-3 g128 at
//     m = 128 / 256 / 512 / 1024 / 2048: 43 / 68 / 116 / 209 / 437 us against 40 / 53 / 73 /
//     122 / 223 here), up to 256 tiles split over k (25 us); 257 to 512 are one round of two
//     blocks a unit, 44 us (512 tiles, us there and in shape E: codebook-4 g128 44 / 48,
//     codebook-3 g128 41 / 38, g32 44 / 46), of long rows (8-wave blocks) 0.05 us a tile;
//   int8 activations, uniform: 64 x 64 tiles, 1.5 ns times q a tile and chunk and 6 us, in the unit
//     of the shapes' costs, whose group sums take the same factor of 1.1 to 1.3 in all of them; q and
//     at_chunks fitted to 720 sizes (n = 1000 to 22016, k = 1024 to 11008, m = 200 to 2048), of which
//     11 then lose 3 % or more (14 % at most). 8192 rows, m = 1000, 2048 tiles, 8 / 32 / 86 chunks, us there
//     and here: 3-bit g128 31 / 36, 105 / 98, 246 / 228; g32 44 / 38, 144 / 107, 311 / 266.
// `share` of it, at the matrix's chunks.
template <int BITS, int KIND, int G, bool A8>
float other_cost(const qx_desc* d, int m, float share) {
  const float chunks = (float)(d->k / 128);
  const auto at = [&](float us) { return at_chunks<BITS, KIND, G, A8>(share * us, chunks); };
  const bool wide = d->k > 64 * 128;
  const long t64 = (long)((d->n + 63) / 64) * ((m + 63) / 64);
  if (KIND != QX_UNIFORM) {
    const bool one_round = t64 <= 512 && !wide && !(A8 && BITS == 3 && G == 32 && chunks < 16.f);
    const float us = t64 <= 128   ? 23.f
                     : t64 <= 256 ? (wide ? 24.f : 30.f)
                     : one_round  ? 44.f
                                  : 20.f + (wide && t64 <= 512 ? 0.05f : 0.07f) * (float)t64;
    const float tables = KIND == QX_CODEBOOK && BITS == 4 && G == 32 ? (t64 <= 256 ? 1.1f : 1.5f) : 1.f;
    return at(us * (A8 ? 1.12f : 1.f) * tables);
  }
  if (A8)
    return 6.f + 0.0015f * chunks * (float)t64 *
                     (G == 32 ? (wide ? 0.8f : 1.f) * (BITS == 3 ? 1.24f : 1.48f)
                              : (wide && BITS == 3 && G == 64 ? 0.9f : 1.f) *
                                    (BITS == 3 ? (G == 64 ? 1.f : 0.91f) : G == 64 ? 1.09f : 1.03f));
  // gemm.hip gives all activation tiles of a weight tile to one XCD: the fullest XCD counts
  const auto tiles = [&](int bn, int bm) { return (long)((d->n + bn - 1) / bn + 7) / 8 * 8 * ((m + bm - 1) / bm); };
  const long mb = (m + 127) / 128, big8 = ((d->n + 255) / 256 * mb + 255) / 256;
  if (kGemmBig8<BITS, G> && m >= 384 && big8 < ((d->n + 191) / 192 * mb + 255) / 256)
    return at(76.f * (float)((tiles(256, 128) + 255) / 256));
  constexpr float light = BITS == 4 ? 0.95f : 1.f;  // the 4-bit codes' shorter decoding
  const long t128 = (long)((d->n + 127) / 128) * ((m + 63) / 64);
  if (t128 <= 256) return at(light * (t128 <= 64 ? 20.7f : t128 <= 128 ? 25.5f : wide ? 33.f : 38.f) * (tiles(128, 64) > 256 ? 1.4f : 1.f));
  const long all = tiles(128, 64), rest = all % 768;
  constexpr float us[3] = {41.f, kGemmBig8<BITS, G> ? 54.f : 57.f, kGemmBig8<BITS, G> ? 78.f : 85.f};
  return at(light * (us[2] * (float)(all / 768) + (rest ? us[(rest - 1) / 256] : 0.f))) + (chunks <= 10.f && (all > t128 || all < 480) ? 2.f : 0.f);
}

// Split over k: every block's time is its fixed part and its chunks.
template <int BITS, int KIND, int G, bool A8, int S>
void consider_split(const qx_desc* d, int m, float& best, int& shape) {
  if constexpr (built<BITS, KIND, G, A8>(S)) {
    const long blocks = (long)((d->n + kShape[S].bn - 1) / kShape[S].bn) * ((m + kShape[S].bm - 1) / kShape[S].bm);
    const float rounds = (float)((blocks + 255) / 256);
    // H with 4-bit uniform codes falls behind on long rows (4656x13824 g128, m = 200: 85 us by the
    // rest of this, 98 measured, 84 in gemm.hip)
    const float late = S == kH && KIND == QX_UNIFORM && BITS == 4 && m > 64 && d->k > 64 * 128 ? 1.12f : 1.f;
    const float us = decode_factor<BITS, KIND, G, A8>() * (kShape[S].us[0] + kShape[S].us[1] * (float)(d->k / 128)) * (rounds > 1.f ? 1.08f : 1.f) * late *
                     (1.f - kShape[S].us[2] + kShape[S].us[2] * rounds);
    if (us < best) {
      best = us;
      shape = S;
    }
  }
}

// 17 to 64 rows: whether the 32 x 32 tiles of gemm.hip (4 waves, k over two of them) take less
// time than every shape here. They have a shorter start and end than a k split over 8 waves,
// which counts where rows are short, and hold three and more tiles on a compute unit, which
// streams the codes and tables faster where there are several rounds of tiles and decoding is
// heavy. Measured in all formats, n = 4096 to 28672, k = 1024 to 11008, m = 24 and 48 (us there
// and in the best shape here; up to 32 rows unless stated):
//   more than 512 weight tiles: 22016x5120 codebook-4 g32 54.6 / 71.7, 22016x8192 codebook-4 g64
//     61.5 / 76.2, 22016x2048 codebook-4 g128 16.5 / 18.6, uniform-4 g128 14.3 / 16.5, Q4X
//     18.0 / 20.4, 22016x8192 codebook-3 g32 57.8 / 65.5; the lighter decoders only where rows
//     are short: 22016 rows uniform-3 g64 at 8 / 16 / 32 chunks 10.0 / 11.8, 16.1 / 16.8, 27.3 / 25.3;
//   257 to 512: codebook-4 g32 always (11008x4096 26.4 / 31.2), codebook-4 g64 and Q4X up to 40
//     chunks (11008x2048 13.8 / 16.2, 11008x4096 Q4X 21.4 / 22.9; 11008x8192 41.5 / 37.6 and
//     38.6 / 38.7; codebook-4 g64 from 385 tiles on always, 14224x8192 47.0 / 50.0), others up to 16 or 12; uniform-4 up to 384 tiles, where the shapes here have
//     one round of 64 x 48 for half as many rows, up to 40 (12288x5120 g128 21.6 / 23.5; beyond,
//     14336x5120 g32 24.1 / 23.0);
//   33 to 64 rows: where 64 x 128 tiles leave half of the units idle (14336x1024 Q4X 12.7 / 16.7,
//     uniform-4 g128 10.5 / 13.0, uniform-3 g64 12.0 / 12.6; 18944x2048 codebook-4 g64 25.4 /
//     30.3), and codebook-4 g32, whose tables leave room for one of them (11008x4096 36.9 / 43.5);
//     rows of up to 8 chunks in 193 or 257 to 384 weight tiles (8103x768 uniform-4 6.6 / 7.2,
//     11008x1024 codebook-4 g128 9.7 / 10.4).
//   513 to 640 at 33 to 64 rows, where one round of 64 x 128 tiles leaves three units in eight idle:
//     uniform-4 up to 28 chunks (18016x3072 g128 27.4 / 31.5), codebook-4 g64 32 (20432x3072 36.0 /
//     44.0), g32 codes 24 (20432x3072 codebook-3 34.8 / 37.4).
// Rows of 4 chunks (4 of 8 waves idle in a k split) and, above 32 rows, uniform-4 of 6 and 8, up to
// 256 weight tiles: 3346x512 uniform-4 g64 5.1 / 5.7, 960x512 codebook-4 g128 5.2 / 5.8, 1536x1024 uniform-4
// g128 at m = 44 6.0 / 6.6; from 129 tiles on uniform-3 of 4 chunks too (4672x512 g128 at m = 41 5.9 /
// 6.5); int8 rows of codebook-4 g128 above 256: 18016x512 8.8 / 10.7.
// Codebook-4 g32 on rows of more than 64 chunks, up to 256 weight tiles: its 32 x 32 tiles with k
// split over 8 waves from about one tile a unit on (chunks x tiles: 3792x12288 38.9 / 43.5, 4208x10240
// 32.5 / 37.1, 7424x12288 44.5 / 51.9; 4368x9216 29.2 / 27.5, 3328x10240 31.0 / 30.5).
// Q4X and codebook-4 g32 rows of few chunks: Q4X 12288x640 at m = 21 7.5 / 8.1, 4096x1024 at m = 24 5.9 / 6.3;
// codebook-4 g32 639x640 at m = 27 5.8 / 6.1.
template <int BITS, int KIND, int G, bool A8>
bool small_tiles_win(const qx_desc* d, int m) {
  constexpr int kAll = 1 << 20;  // chunks
  constexpr bool kQ4x = KIND == QX_Q4X, kCb4g32 = KIND == QX_CODEBOOK && BITS == 4 && G == 32;
  const int chunks = d->k / 128, tiles = (d->n + 31) / 32;
  if (kQ4x && tiles <= (m <= 32 ? 256 : 512) && chunks <= (A8 ? 7 : 8)) return true;
  if (kCb4g32 && !A8 && tiles <= 256 && chunks <= 8) return true;
  if (BITS == 4 && !A8 && !kQ4x && tiles <= 256 &&
      (chunks <= 4 || (KIND == QX_UNIFORM && m > 32 && chunks <= 8 && chunks % 2 == 0)))
    return true;
  if (BITS == 3 && KIND == QX_UNIFORM && m > 32 && tiles > 128 && tiles <= 256 && chunks <= 4) return true;
  if (m <= 32) {
    if (tiles <= 256) return wide_small_tiles<BITS, KIND, G, A8> && chunks > 64 && tiles * chunks > 11000;
    const bool two = tiles <= 512;
    if (kQ4x) return chunks <= (A8 ? (two ? 16 : 40) : two ? 40 : kAll);
    if (KIND == QX_UNIFORM) return chunks <= (BITS == 3 ? (two ? 12 : 16) : !two ? kAll : tiles <= 384 ? 40 : 16);
    if (BITS == 3) return chunks <= (G == 32 ? (A8 ? (two ? 12 : 16) : two ? 16 : kAll) : A8 ? 0 : 12);
    if (G == 128) return chunks <= (A8 ? 4 : two ? 16 : kAll) || (!two && chunks > 64);
    return chunks <= (G == 32 || tiles > 384 ? kAll : A8 ? 16 : 40);
  }
  if (kCb4g32) return tiles > 256 && (tiles <= 384 ? chunks <= (A8 ? 64 : kAll) : tiles <= 512 ? chunks <= 8 : !A8 && tiles <= 600);
  if (BITS == 4 && !A8 && tiles > (KIND == QX_UNIFORM ? 192 : 256) && tiles <= 384 && chunks <= 8) return true;
  if (tiles > 512 && tiles <= 640 && chunks > 16)
    return KIND == QX_UNIFORM ? BITS == 4 && chunks <= 28
                              : chunks <= (G == 32 ? 24 : G == 64 && BITS == 4 && !kQ4x ? (A8 ? 24 : 32) : 0);
  if (tiles <= 384 || tiles > (A8 || BITS == 3 ? 512 : kQ4x ? 700 : 600)) return false;
  return chunks <= (BITS == 3 ? (A8 ? 0 : 8) : A8 && !kQ4x ? (G == 64 ? 12 : 8) : 16);
}

template <int BITS, int KIND, int G, bool A8>
int pick(const qx_desc* d, int m) {
  // 17 to 64 rows: one of these shapes unless small_tiles_win; qx_gemm keeps up to 32 rows of
  // up to 32 chunks with gemm_skinny.hip where that applies (4096x4096 uniform-4 at m = 19:
  // 8.1 us there, 9.6 here; 12288x4096 codebook-3 at m = 28: 15.1 and 17.1). Above, a shape must
  // promise 4 % less than gemm.hip; the fit for the integer products of gemm_a8.hip weighs both.
  float best = 1e30f;
  int shape = kShapes;
  if (m <= 64 && (!A8 || KIND != QX_UNIFORM) && small_tiles_win<BITS, KIND, G, A8>(d, m)) return shape;
  if (m > 64) {
    best = other_cost<BITS, KIND, G, A8>(d, m, 0.96f);
    consider<BITS, KIND, G, A8, kA>(d, m, best, shape);
    consider<BITS, KIND, G, A8, kB>(d, m, best, shape);
    consider<BITS, KIND, G, A8, kC>(d, m, best, shape);
    consider<BITS, KIND, G, A8, kD>(d, m, best, shape);
  }
  if (m > 32 && (m > 64 || !A8 || KIND != QX_UNIFORM)) consider<BITS, KIND, G, A8, kE>(d, m, best, shape);
  consider_split<BITS, KIND, G, A8, kF>(d, m, best, shape);
  consider_split<BITS, KIND, G, A8, kG>(d, m, best, shape);
  consider_split<BITS, KIND, G, A8, kH>(d, m, best, shape);
  return shape;
}

#define QX_TILE_FORMATS(F)                                                              \
  F(3, 0, 32) F(3, 0, 64) F(3, 0, 128) F(4, 0, 32) F(4, 0, 64) F(4, 0, 128) F(3, 1, 32) \
  F(3, 1, 64) F(3, 1, 128) F(4, 1, 32) F(4, 1, 64) F(4, 1, 128) F(4, 2, 64)

// The shape for m rows of X (int8 rows with a8), kShapes if another kernel takes them.
inline int pick_shape(const qx_desc* d, int m, bool a8) {
  if (m <= 16) return kShapes;  // one activation tile: gemm_skinny.hip, gemm.hip, gemm_a8.hip
#define QX_TILE_PICK(B, K, G)                        \
  if (d->bits == B && d->kind == K && d->group == G) \
    return a8 ? pick<B, K, G, true>(d, m) : pick<B, K, G, false>(d, m);
  QX_TILE_FORMATS(QX_TILE_PICK)
#undef QX_TILE_PICK
  return kShapes;
}

}  // namespace tile
}  // namespace qx
