// Quantized GEMM for many activation rows: Y[m][n] = sum_k X[m][k] W'[n][k] on the fp16
// matrix cores with wave tiles of 16*MT activation rows x 16*NT weight rows.
//
// What bounds it. A 16x16x32 product takes 16 cycles of a SIMD and the LDS of a compute
// unit delivers 128 bytes a cycle to its four SIMDs, so a wave tile of 128 x 32 already
// reads activation fragments as fast as LDS can deliver them; at 128 x 64 these reads take
// half of that. Weights never pass through LDS as fp16: every wave decodes its own weight
// rows from packed codes in registers, and each decoded fragment feeds MT products. Timed
// with parts left out (22016x4096 uniform-4 g128, m = 2048, 483 us with 16-byte code runs):
// the products, their activation reads and the barriers alone take 260 us, decoding adds 30,
// LDS writes 40, the loads of activations 70 and those of codes 90; hence code runs of SC
// chunks (below), which took that product to 401 us.
//
// Block. WM x 4 waves: 4 take different weight rows, WM different activation rows. A round
// is half a chunk (64 k): its activations sit in one of two LDS buffers in decoder pair
// order, the codes of SC chunks (a super-round) in one of two code buffers as
// [slice][row][chunk] pieces of 16 bytes. The next round's activations and the next
// super-round's codes travel from memory into registers meanwhile and are written to LDS
// after their round: one barrier a round. Blocks of 4 waves and 128 x 256 or less use at
// most half of the LDS and of the registers in most formats, so two or three of them share
// a compute unit and one decodes while another multiplies; a block of 256 x 256 has two
// waves on every SIMD itself.
//
// Few tiles (KS > 1): a block of KS waves owns one tile of 16*MT x 16*NT and wave ks takes
// the chunks ks, ks + KS, .. of k. With few blocks the time is one wave's chain of loads,
// decoding and products over all of k, so the chain is cut in KS; every wave stages its own
// activations and codes in its own part of the LDS and meets the others only when the
// partial tiles are added in the order of the waves (deterministic).
// 11008x4096 uniform-3 g64 at m = 64: 29.9 us before (gemm_skinny.hip), 18.4 now;
// 4096x11008 29.9 -> 21.0 us; 1376x4096 uniform-4 g32 at m = 77: 20.7 us (gemm.hip) -> 9.6;
// 4001x1408 codebook-4 g64 13.8 -> 9.3 us.
//
// LDS banks. Activation rows of 128 bytes with 16-byte pieces swizzled by row (padding by
// 16 bytes left 37 % of the LDS cycles to conflicts, because the lanes that the LDS serves
// together come from two pieces), codes swizzled so that 16 rows of one chunk hit all banks.
//
// k order. k-step T of a chunk (32 of 128 k) takes 8 consecutive codes 8f .. 8f + 7 in lane
// group g (f = 4T + g), so that a k-step lies in one quantization group:
//   b = 4: code dword f;
//   b = 3: T = 0: bits 0-2 of dwords 2g, 2g+1; T = 1: bits 0-2 of dwords 8+2g, 9+2g (g < 2)
//          or bits 3-5 of dwords 2(g-2), 2(g-2)+1; T = 2: bits 3-5 of dwords 4+2g, 5+2g;
//          T = 3: the spare codes of dwords 2g, 2g+1.
//
// A8: X holds int8 codes (qx_quantize_a8), which enter the products as exact binary16
// integers; Y is scaled by the row's sx. Uniform and Q4X weights then enter as the exact
// integers q - z or the sub-codebook's entries, and the sum of a group (of half a group of
// 128) is scaled by its s in fp32. The products are exact; so are the sums of uniform codes (at
// most 64 * 15 * 127), those of Q4X round as fp32 sums do.
#include <type_traits>

#include "gemm_tile_plan.h"
#include "qx_device.h"

namespace qx {
using namespace tile;
namespace {

typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}

// Four neighbouring columns of Y, whose rows may start at any multiple of 2 bytes: the target
// stores 8 bytes at any alignment. Stored one by one where n % 4 != 0 they cost short rows up to a
// third of their time (uniform-4 g128, 15545x640 at m = 565: 42.6 us, 33.0 with these).
typedef uint32_t u32x2_at2 __attribute__((ext_vector_type(2), aligned(2)));

// What decodes a fragment: the lane's code dwords (b = 4: L.x; b = 3: L, and H for the
// spare codes) and its group's constants or table.
template <int BITS, int KIND>
struct RawFrag {
  u32x2 L, H;
  uint32_t sp, z0;  // uniform: (s, s) and -(1024 + z) pairs; Q4X: sp
  LutGroup<BITS> lut;
};

template <int BITS, int KIND, bool SCALE>
__device__ __forceinline__ uint32_t level(uint32_t mq, uint32_t zc, uint32_t sp) {
  const uint32_t v = hadd2(mq, zc);
  return SCALE ? hmul2(v, sp) : v;
}

// B fragment of k-step T.
template <int BITS, int KIND, int T, bool SCALE>
__device__ __forceinline__ h8_t tile_frag(const RawFrag<BITS, KIND>& gd, const DecodeConsts& k, uint32_t t1,
                                          uint32_t up, uint32_t dn, uint32_t ssh) {
  // -(M + z) for M = 128 (b = 3) or 64 (b = 4), and 16: z in steps of 8 or 16, and 64
  const uint32_t z1 = BITS == 3 ? (gd.z0 << 3) + (0xD800D800u - (0xE400E400u << 3))
                                : (gd.z0 << 4) + (0xD400D400u - (0xE400E400u << 4));
  const uint32_t z2 = (gd.z0 << 6) + (0xCC00CC00u - (0xE400E400u << 6));
  if constexpr (BITS == 4) {
    const uint32_t D = gd.L.x;
    if constexpr (KIND == QX_UNIFORM) {
      const uint32_t Ds = D >> 8;
      return frag(level<4, KIND, SCALE>((D & k.m000f) | k.mag1024, gd.z0, gd.sp),    // (0, 4)
                  level<4, KIND, SCALE>((D & k.m00f0) | k.mag64, z1, gd.sp),      // (1, 5)
                  level<4, KIND, SCALE>((Ds & k.m000f) | k.mag1024, gd.z0, gd.sp),   // (2, 6)
                  level<4, KIND, SCALE>((Ds & k.m00f0) | k.mag64, z1, gd.sp));    // (3, 7)
    } else {
      uint32_t elo, ehi, olo, ohi;
      lut4_bytes(gd.lut, D & 0x0F0F0F0Fu, elo, ehi);         // codes 0 2 4 6
      lut4_bytes(gd.lut, (D >> 4) & 0x0F0F0F0Fu, olo, ohi);  // codes 1 3 5 7
      const uint32_t p0 = perm(ehi, elo, 0x06020400u), p1 = perm(ohi, olo, 0x06020400u);
      const uint32_t p2 = perm(ehi, elo, 0x07030501u), p3 = perm(ohi, olo, 0x07030501u);
      if constexpr (KIND == QX_Q4X && SCALE)  // fp16(s * CB[t][q]): one rounding, as qx_dequant
        return frag(hmul2(p0, gd.sp), hmul2(p1, gd.sp), hmul2(p2, gd.sp), hmul2(p3, gd.sp));
      return frag(p0, p1, p2, p3);
    }
  } else {
    const uint32_t d[2] = {gd.L.x, gd.L.y}, h[2] = {gd.H.x, gd.H.y};
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t D = T == 1 ? d[i] >> t1 : d[i];  // T = 1: both field kinds to bits 0-2
      if constexpr (KIND == QX_UNIFORM) {
        const uint32_t Ds = D >> 8;
        if constexpr (T < 2) {
          w[2 * i] = level<3, KIND, SCALE>((D & k.m0007) | k.mag1024, gd.z0, gd.sp);
          w[2 * i + 1] = level<3, KIND, SCALE>((Ds & k.m0007) | k.mag1024, gd.z0, gd.sp);
        } else if constexpr (T == 2) {
          w[2 * i] = level<3, KIND, SCALE>((D & k.m0038) | k.mag128, z1, gd.sp);
          w[2 * i + 1] = level<3, KIND, SCALE>((Ds & k.m0038) | k.mag128, z1, gd.sp);
        } else {
          const uint32_t u0 = ((h[i] << up) & k.m0100) | k.mag16, u1 = ((h[i] >> dn) & k.m0100) | k.mag16;
          w[2 * i] = level<3, KIND, SCALE>((D & k.m00c0) | u0, z2, gd.sp);
          w[2 * i + 1] = level<3, KIND, SCALE>((Ds & k.m00c0) | u1, z2, gd.sp);
        }
      } else {
        const uint32_t S = T < 2    ? D & 0x07070707u
                           : T == 2 ? (D >> 3) & 0x07070707u
                                    : ((D >> 6) & 0x03030303u) | ((h[i] >> ssh) & 0x04040404u);
        lut3_pairs(gd.lut, S, w[2 * i], w[2 * i + 1]);
      }
    }
    return frag(w[0], w[1], w[2], w[3]);
  }
}

template <int BITS, int KIND, int G, int MT, int NT, int WM, int SC, int KS, bool A8,
          int THREADS = TileShape<BITS, KIND, G, MT, NT, WM, SC, KS>::kThreads,
          int WAVES = TileShape<BITS, KIND, G, MT, NT, WM, SC, KS>::kWaves>
__global__ __launch_bounds__(THREADS, WAVES) void gemm_tile_kernel(
    const char* __restrict__ packed, const void* __restrict__ Xv, const float* __restrict__ sx,
    uint16_t* __restrict__ Y, int n, int k, int m, int nx, int my, int groups) {
  using TS = TileShape<BITS, KIND, G, MT, NT, WM, SC, KS>;
  using TR = TileReads<BITS, KIND, G, MT, NT, WM, SC, KS, A8>;
  constexpr int NTH = TR::NTH, BM = TS::BM, BN = TS::BN, NG = TS::NG, kXB = TR::kXB, kMRow = TR::kMRow;
  constexpr bool kSums = A8 && KIND != QX_CODEBOOK;  // group sums scaled in fp32
  constexpr int XP = TR::XP, CT = TR::CT, CP = TR::CP, MTOT = TR::MTOT, MP = TR::MP;
  constexpr int MD = KIND == QX_UNIFORM ? NG : KIND == QX_Q4X ? 2 : 4;  // dwords of a table piece
  static_assert(BM * 8 % NTH == 0, "activation pieces divide evenly");
  __shared__ __align__(16) char lds[TS::kLds];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const xs = lds + (KS > 1 ? wave * TS::kWaveLds : 0);
  char* const cts = xs + (KS > 1 ? 1 : 2) * TS::kXBuf;
  char* const mts = cts + 2 * TS::kCBuf;
  uint32_t* const q4lut = reinterpret_cast<uint32_t*>(lds + KS * TS::kWaveLds);

  const int total = nx * my, share = (total + 7) >> 3, at = blockIdx.x >> 3;
  const int tile = (int)(blockIdx.x & 7) * share + at;
  if (tile >= total) return;  // whole block, before any barrier
  const TileAt block = tile_at(tile, nx, my, groups);
  const int n0 = block.bn * BN, m0 = block.bm * BM;
  const int C = k >> 7, G_row = k / G;
  const size_t meta_off = (size_t)n * k * BITS / 8;
  const int t = KS > 1 ? threadIdx.x & 63 : threadIdx.x, lane = t & 63, g = lane >> 4, li = lane & 15;
  const int wn = KS > 1 ? 0 : wave & 3, wm = KS > 1 ? 0 : wave >> 2, ks = KS > 1 ? wave : 0;
  const int CW = (C - ks + KS - 1) / KS;  // this wave's chunks: ks, ks + KS, ..
  const DecodeConsts kc = decode_consts();
  const uint32_t t1 = g < 2 ? 0u : 3u, up = g < 2 ? 2u : 1u, dn = g < 2 ? 6u : 7u, ssh = g < 2 ? 4u : 5u;

  // Loads of the next round or chunk into registers (rows and chunks clamped in bounds;
  // the clamped copies are never stored to Y or never multiplied) and their LDS writes.
  u32x4 xr[XP], cr[CP];
  uint32_t mr[MP][MD];
  // Buffer loads: 32-bit offsets, rows past the matrix outside the bounds (they read 0). The
  // 64-bit addresses that the compiler keeps for plain loads would not leave room for the
  // accumulators.
  const int xrows = min(BM, m - m0), wrows = min(BN, n - n0);
  BufferRsrc xres[XP];
#pragma unroll
  for (int i = 0; i < XP; ++i) {
    const int row = TR::x_row(i, xrows);
    xres[i] = buffer(static_cast<const char*>(Xv) + (size_t)(m0 + row) * k * kXB, (xrows - row) * k * kXB);
  }
  const BufferRsrc cres = buffer(packed + (size_t)n0 * BITS * C * 16, wrows * BITS * C * 16);
  const BufferRsrc mres = buffer(packed + meta_off + (size_t)n0 * G_row * kMRow, wrows * G_row * kMRow);
  const int sel_words = (G_row + 15) / 16;
  const BufferRsrc sres = buffer(packed + meta_off + meta_off / 16 + (size_t)n0 * sel_words * 4,
                                 KIND == QX_Q4X ? wrows * sel_words * 4 : 0);
  auto load_x = [&](int c, int h) {
    const int cx = min(c * KS + ks, C - 1);
    const ReadAt r = TR::x(t, cx, h, k);
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      if constexpr (A8) {
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(xres[i], r.lane, r.scalar, 0));
        xr[i].x = v.x; xr[i].y = v.y;
      } else {
        xr[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xres[i], r.lane, r.scalar, 0));
      }
    }
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      const int p = t + i * NTH;
      u32x2 lo = {xr[i].x, xr[i].y}, hh = {xr[i].z, xr[i].w};
      if constexpr (A8) {
        hh = i8x4_to_h4(xr[i].y);
        lo = i8x4_to_h4(xr[i].x);
      }
      *reinterpret_cast<u32x4*>(xs + (KS > 1 ? 0 : buf) * TS::kXBuf + (p >> 3) * kXRow + ((p ^ (p >> 4)) & 7) * 16) = x_piece<BITS>(lo, hh);
    }
  };
  // Codes and tables of super-round j. Past the last chunk of a row the loads run on into
  // what follows (or out of bounds, 0); it is never multiplied.
  static_assert(KS == 1 || SC == 1, "waves on their own chunks take them one by one");
  const int last_j = KS > 1 ? CW - 1 : (C - 1) / SC;
  auto load_codes = [&](int j) {
    const int c = KS > 1 ? min(j * KS + ks, C - 1) : min(j, last_j) * SC;
#pragma unroll
    for (int i = 0; i < CP; ++i) {
      const ReadAt r = TR::code(t, i, c, C);
      cr[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(cres, r.lane, r.scalar, 0));
    }
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const ReadAt r = TR::meta(t, i, c, G_row);
      if constexpr (KIND == QX_Q4X) {  // the scales of a chunk's groups and their selectors (4 bits)
        const ReadAt w = TR::selectors(t, i, c, sel_words);
        mr[i][0] = __builtin_amdgcn_raw_buffer_load_b32(mres, r.lane, r.scalar, 0);
        mr[i][1] = __builtin_amdgcn_raw_buffer_load_b32(sres, w.lane, w.scalar, 0) >>
                   (4 * ((c + TR::meta_piece(t, i) % SC) % 8));
      } else if constexpr (TR::kMBytes == 4) {
        mr[i][0] = __builtin_amdgcn_raw_buffer_load_b32(mres, r.lane, r.scalar, 0);
      } else if constexpr (TR::kMBytes == 8) {
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(mres, r.lane, r.scalar, 0));
        mr[i][0] = v.x; mr[i][1] = v.y;
      } else {
        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(mres, r.lane, r.scalar, 0));
        mr[i][0] = v.x; mr[i][1] = v.y; mr[i][2] = v.z; mr[i][3] = v.w;
      }
    }
  };
  auto store_codes = [&](int buf) {
#pragma unroll
    for (int i = 0; i < CP; ++i) {
      const int p = t + i * NTH;
      if (CT % NTH == 0 || p < CT) *reinterpret_cast<u32x4*>(cts + buf * TS::kCBuf + p * 16) = cr[i];
    }
    char* const mb = mts + buf * TS::kMBuf;
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const int p = t + i * NTH;
      if (MTOT % NTH == 0 || p < MTOT) {
        if constexpr (KIND == QX_CODEBOOK) {
          *reinterpret_cast<u32x4*>(mb + (p % (TS::kMPlanes * SC) * BN + p / (TS::kMPlanes * SC)) * 16) =
              u32x4{perm(mr[i][1], mr[i][0], 0x06040200u), perm(mr[i][3], mr[i][2], 0x06040200u),
                    perm(mr[i][1], mr[i][0], 0x07050301u), perm(mr[i][3], mr[i][2], 0x07050301u)};
        } else if constexpr (KIND == QX_Q4X) {
          *reinterpret_cast<u32x2*>(mb + (p % SC * BN + p / SC) * 8) = u32x2{mr[i][0], mr[i][1]};
        } else {
#pragma unroll
          for (int j = 0; j < NG; ++j) {
            const uint32_t w = mr[i][j];
            // z is an integer-valued fp16: the bits of -(1024 + z) are those of -1024 plus z
            const uint32_t z = (uint32_t)(unsigned short)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
            *reinterpret_cast<u32x2*>(mb + ((p % SC * NG + j) * BN + p / SC) * 8) =
                u32x2{perm(w, w, 0x01000100u), (0xE400u + z) * 0x00010001u};
          }
        }
      }
    }
  };

  f4_t acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f4_t{0.f, 0.f, 0.f, 0.f};

  // Codes and group constants of the fragment of weight rows 16 nt .. of this wave at k-step
  // T of chunk cc of the super-round in code buffer cb.
  auto read_raw = [&](auto tc, int cb, int cc, int nt) {
    constexpr int T = decltype(tc)::value;
    RawFrag<BITS, KIND> r;
    const int row = wn * 16 * NT + 16 * nt + li;
    constexpr int SL = BN * SC * 16;  // bytes of a slice
    const char* const cr0 = cts + cb * TS::kCBuf + row * SC * 16 + (SC == 2 ? (cc ^ (li >> 3)) * 16 : 0);
    const char* const mb = mts + cb * TS::kMBuf + cc * TS::kMPlanes * BN * TS::kMUnit;
    constexpr int grp = 32 * T / G;
    r.H = u32x2{0u, 0u};
    if constexpr (BITS == 4) {
      r.L = u32x2{*reinterpret_cast<const uint32_t*>(cr0 + T * SL + 4 * g), 0u};
    } else {
      const int sl = T == 0 || T == 3 ? g >> 1 : T == 1 ? (g < 2 ? 2 : 0) : g < 2 ? 1 : 2;
      r.L = *reinterpret_cast<const u32x2*>(cr0 + sl * SL + 8 * (g & 1));
      if constexpr (T == 3) r.H = *reinterpret_cast<const u32x2*>(cr0 + 2 * SL + 8 * (g & 1));
    }
    if constexpr (KIND == QX_UNIFORM) {
      const u32x2 v = *reinterpret_cast<const u32x2*>(mb + (grp * BN + row) * 8);
      r.sp = v.x; r.z0 = v.y;
    } else if constexpr (KIND == QX_Q4X) {
      const u32x2 v = *reinterpret_cast<const u32x2*>(mb + row * 8);
      r.sp = perm(v.x, v.x, grp == 0 ? 0x01000100u : 0x03020302u);
      r.z0 = 0u;
      const uint32_t* tp = q4lut + 8 * ((v.y >> (2 * grp)) & 3u);
      const u32x4 tl = *reinterpret_cast<const u32x4*>(tp), th = *reinterpret_cast<const u32x4*>(tp + 4);
      r.lut = LutGroup<BITS>{{tl.x, tl.y, tl.z, tl.w}, {th.x, th.y, th.z, th.w}};
    } else {
      r.sp = r.z0 = 0u;
#pragma unroll
      for (int u = 0; u < TS::kTable / 16; ++u) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(mb + ((grp * (TS::kTable / 16) + u) * BN + row) * 16);
        r.lut.lo[2 * u] = v.x; r.lut.lo[2 * u + 1] = v.y; r.lut.hi[2 * u] = v.z; r.lut.hi[2 * u + 1] = v.w;
      }
    }
    return r;
  };
  // piece j of activation row r sits at position j ^ (r / 2) % 8 of the row: the 16 lanes that
  // the LDS serves together (of 16 rows, or of 8 rows and two pieces) hit all 64 banks
  const char* const xl[2] = {xs + (wm * 16 * MT + li) * kXRow + ((g ^ (li >> 1)) & 7) * 16,
                             xs + (wm * 16 * MT + li) * kXRow + (((4 + g) ^ (li >> 1)) & 7) * 16};
  h8_t b[2][NT];

  // k-step T of a chunk: the weight fragments are decoded, then the activation fragments
  // are read one tile ahead of the products. The fences keep that order (left alone, the
  // scheduler reads a fragment right before its use and hoists more code reads than the
  // registers hold).
  auto kstep = [&](auto tc, int cb, int cc) {
    constexpr int T = decltype(tc)::value;
    const char* const xb = xl[T % 2] + (KS > 1 ? 0 : T / 2) * TS::kXBuf;
    h8_t pa = *reinterpret_cast<const h8_t*>(xb);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      b[0][nt] = tile_frag<BITS, KIND, T, true>(read_raw(tc, cb, cc, nt), kc, t1, up, dn, ssh);
      if constexpr (MT * NT == 32 && (BITS == 3 || KIND != QX_UNIFORM))
        if (nt % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const h8_t a = pa;
      if (mt + 1 < MT) pa = *reinterpret_cast<const h8_t*>(xb + 16 * (mt + 1) * kXRow);
#pragma unroll
      for (int j = 0; j < NT; ++j)  // weights as rows: a lane ends with four neighbouring columns of Y
        acc[mt][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b[0][j], a, acc[mt][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // With group sums: half h of the chunk in code buffer cb, both k-steps of 16 activation
  // rows together (a group of 64 spans them; half a group of 128 is summed alone).
  auto round = [&](auto hc, int cb, int cc) {
    constexpr int H = decltype(hc)::value;
    constexpr int GR = G == 32 ? 2 : 1;  // groups of the half chunk
    float sg[GR][NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const RawFrag<BITS, KIND> r0 = read_raw(std::integral_constant<int, 2 * H>{}, cb, cc, nt);
      const RawFrag<BITS, KIND> r1 = read_raw(std::integral_constant<int, 2 * H + 1>{}, cb, cc, nt);
      sg[0][nt] = half_bits_to_float(r0.sp & 0xFFFFu);
      if constexpr (GR == 2) sg[1][nt] = half_bits_to_float(r1.sp & 0xFFFFu);
      b[0][nt] = tile_frag<BITS, KIND, 2 * H, false>(r0, kc, t1, up, dn, ssh);
      b[1][nt] = tile_frag<BITS, KIND, 2 * H + 1, false>(r1, kc, t1, up, dn, ssh);
      // the reads of later rows, hoisted here, would not fit the registers
      if constexpr (MT * NT == 32)
        if (nt % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    const char *const xb = xl[0] + (KS > 1 ? 0 : H) * TS::kXBuf, *const xc = xl[1] + (KS > 1 ? 0 : H) * TS::kXBuf;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const h8_t a0 = *reinterpret_cast<const h8_t*>(xb + 16 * mt * kXRow);
      const h8_t a1 = *reinterpret_cast<const h8_t*>(xc + 16 * mt * kXRow);
      const f4_t zero = {0.f, 0.f, 0.f, 0.f};
      f4_t s0[NT], s1[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) s0[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, b[0][nt], zero, 0, 0, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        s1[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, b[1][nt], GR == 2 ? zero : s0[nt], 0, 0, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        if constexpr (GR == 2) acc[mt][nt] += sg[0][nt] * s0[nt];
        acc[mt][nt] += sg[GR - 1][nt] * s1[nt];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  if constexpr (KIND == QX_Q4X) stage_q4x_tables(packed + q4x_offsets(n, k).codebook, q4lut);
  load_codes(0);
  load_x(0, 0);
  store_codes(0);
  load_codes(1);
  store_x(0);
  __syncthreads();
  // Super-round j + 1's codes go to the buffer last read in super-round j - 1; at least one
  // barrier follows before their first read. Each activation buffer is written one barrier
  // after its last read.
  auto k0 = std::integral_constant<int, 0>{};
  auto k1 = std::integral_constant<int, 1>{};
  auto k2 = std::integral_constant<int, 2>{};
  auto k3 = std::integral_constant<int, 3>{};
  // KS > 1: every wave works in its own part of the LDS and only its own order counts
  auto round_end = [&]() {
    if constexpr (KS > 1) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  };
  for (int j = 0; j <= last_j; ++j) {
#pragma unroll
    for (int cc = 0; cc < SC; ++cc) {
      const int c = j * SC + cc;
      if (c < CW) {
        load_x(c, 1);
        if (cc == 0) {
          store_codes((j + 1) & 1);
          load_codes(j + 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kSums) {
          round(k0, j & 1, cc);
        } else {
          kstep(k0, j & 1, cc);
          kstep(k1, j & 1, cc);
        }
        if (KS > 1) round_end();
        store_x(1);
        round_end();
        load_x(c + 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kSums) {
          round(k1, j & 1, cc);
        } else {
          kstep(k2, j & 1, cc);
          kstep(k3, j & 1, cc);
        }
        if (KS > 1) round_end();
        store_x(0);
        round_end();
      }
    }
  }

  // The waves' partial tiles, added in the order of the waves: tile i by wave i % KS.
  if constexpr (KS > 1) {
    static_assert(MT * NT * 1024 <= TS::kWaveLds, "a wave's partial tiles fit its LDS");
#pragma unroll
    for (int i = 0; i < MT * NT; ++i) *reinterpret_cast<f4_t*>(xs + i * 1024 + lane * 16) = acc[i / NT][i % NT];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MT * NT; ++i) {
      if (i % KS != wave) continue;
      f4_t sum = *reinterpret_cast<const f4_t*>(lds + i * 1024 + lane * 16);
#pragma unroll
      for (int w = 1; w < KS; ++w) sum += *reinterpret_cast<const f4_t*>(lds + w * TS::kWaveLds + i * 1024 + lane * 16);
      acc[i / NT][i % NT] = sum;
    }
  }

#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if constexpr (!kSums) {  // lane: activation row li, weight rows 4g + r
      const int row = m0 + (wm * MT + mt) * 16 + li;
      if (row < m) {
        const float sr = A8 ? sx[row] : 1.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (KS > 1 && (mt * NT + nt) % KS != wave) continue;
          const int col = n0 + (wn * NT + nt) * 16 + 4 * g;
          uint32_t v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = float_to_half_bits(A8 ? acc[mt][nt][r] * sr : acc[mt][nt][r]);
          uint16_t* const dst = Y + (size_t)row * n + col;
          if (col + 4 <= n) {
            *reinterpret_cast<u32x2_at2*>(dst) = u32x2{v[0] | (v[1] << 16), v[2] | (v[3] << 16)};
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (col + r < n) dst[r] = (uint16_t)v[r];
          }
        }
      }
    } else {  // lane: weight row li, activation rows 4g + r
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + (wm * MT + mt) * 16 + 4 * g + r;
        if (row < m) {
          const float sr = sx[row];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            if (KS > 1 && (mt * NT + nt) % KS != wave) continue;
            const int col = n0 + (wn * NT + nt) * 16 + li;
            if (col < n) Y[(size_t)row * n + col] = (uint16_t)float_to_half_bits(sr * acc[mt][nt][r]);
          }
        }
      }
    }
  }
}

template <int BITS, int KIND, int G, bool A8, int MT, int NT, int WM, int SC, int KS = 1>
int launch_cfg(const qx_desc* d, const void* packed, int m, const void* X, const float* sx, uint16_t* Y,
               hipStream_t s) {
  using TS = TileShape<BITS, KIND, G, MT, NT, WM, SC, KS>;
  static_assert(TS::kLds <= kLdsBytes, "LDS");
  const int nx = (d->n + TS::BN - 1) / TS::BN, my = (m + TS::BM - 1) / TS::BM;
  const unsigned blocks = ((unsigned)nx * (unsigned)my + 7u) / 8u * 8u;
  hipLaunchKernelGGL((gemm_tile_kernel<BITS, KIND, G, MT, NT, WM, SC, KS, A8>), dim3(blocks), dim3(TS::kThreads), 0,
                     s, static_cast<const char*>(packed), X, sx, Y, d->n, d->k, m, nx, my, tile_groups(my));
  return hipGetLastError() == hipSuccess ? QX_OK : QX_E_HIP;
}

template <int BITS, int KIND, int G, bool A8, int S>
int launch_shape(const qx_desc* d, const void* packed, int m, const void* X, const float* sx, uint16_t* Y,
                 hipStream_t s) {
  if constexpr (built<BITS, KIND, G, A8>(S))
    return launch_cfg<BITS, KIND, G, A8, kShape[S].mt, kShape[S].nt, kShape[S].wm, kShape[S].sc, kShape[S].ks>(d, packed, m, X, sx, Y, s);
  else
    return QX_E_UNSUPPORTED;
}

template <int BITS, int KIND, int G, bool A8>
int run(const qx_desc* d, const void* packed, int m, const void* X, const float* sx, uint16_t* Y, int shape,
        hipStream_t s) {
  switch (shape) {
    case kA: return launch_shape<BITS, KIND, G, A8, kA>(d, packed, m, X, sx, Y, s);
    case kB: return launch_shape<BITS, KIND, G, A8, kB>(d, packed, m, X, sx, Y, s);
    case kC: return launch_shape<BITS, KIND, G, A8, kC>(d, packed, m, X, sx, Y, s);
    case kD: return launch_shape<BITS, KIND, G, A8, kD>(d, packed, m, X, sx, Y, s);
    case kE: return launch_shape<BITS, KIND, G, A8, kE>(d, packed, m, X, sx, Y, s);
    case kF: return launch_shape<BITS, KIND, G, A8, kF>(d, packed, m, X, sx, Y, s);
    case kG: return launch_shape<BITS, KIND, G, A8, kG>(d, packed, m, X, sx, Y, s);
    case kH: return launch_shape<BITS, KIND, G, A8, kH>(d, packed, m, X, sx, Y, s);
    default: return QX_E_UNSUPPORTED;
  }
}

}  // namespace

bool gemm_tile_applies(const qx_desc* d, int m, bool a8) { return pick_shape(d, m, a8) != kShapes; }

int launch_gemm_tile(const qx_desc* d, const void* packed, int m, const void* X, const float* sx, uint16_t* Y,
                     hipStream_t s) {
  const int shape = pick_shape(d, m, sx != nullptr);
#define QX_TILE_RUN(B, K, G)                                                             \
  if (d->bits == B && d->kind == K && d->group == G)                                     \
    return sx != nullptr ? run<B, K, G, true>(d, packed, m, X, sx, Y, shape, s)          \
                         : run<B, K, G, false>(d, packed, m, X, sx, Y, shape, s);
  QX_TILE_FORMATS(QX_TILE_RUN)
#undef QX_TILE_RUN
  return QX_E_UNSUPPORTED;
}

}  // namespace qx
