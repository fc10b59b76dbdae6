// The host side of the tiled GEMM for the CPU tests. Arguments:
//   reads  checks where the loads of every built kernel read: every thread, piece and chunk, for
//          1 .. BM activation rows and 1 .. BN weight rows in a block; prints one line per kernel
//          with the number of loads that leave their buffer by either rule of the range check
//   order  reads "nx my" and prints 1 when every tile has one number, and the most weight tiles in
//          the run of one of the 8 XCDs
//   route  reads "bits kind group a8 n k m" from standard input (more than 4 rows) and prints the
//          kernel that qx_gemm or qx_gemm_a8 launches: the letter of a tiled shape, or its file
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "../../paper_2505_07531_amd/csrc/gemm_skinny_plan.h"
#include "../../paper_2505_07531_amd/csrc/gemm_tile_plan.h"

// Stand-ins for the launchers that qx_api.cpp calls.
static char g_route[16];
static int took(const char* name) {
  std::snprintf(g_route, sizeof g_route, "%s", name);
  return QX_OK;
}
namespace qx {
int launch_dequant(const qx_desc*, const void*, int, void*, hipStream_t) { return QX_E_HIP; }
int launch_gemv(const qx_desc*, const void*, const uint16_t*, uint16_t*, hipStream_t) { return QX_E_HIP; }
int launch_gemv_a8(const qx_desc*, const void*, const uint16_t*, uint16_t*, hipStream_t) { return QX_E_HIP; }
int launch_quantize_a8(int, int, const uint16_t*, int8_t*, float*, hipStream_t) { return QX_E_HIP; }
int launch_gemv_a8_multi(const qx_desc*, const void*, int, const int8_t*, const float*, uint16_t*, hipStream_t) {
  return QX_E_HIP;
}
int launch_gemv_lut_a8(const qx_desc*, const void*, const uint16_t*, uint16_t*, hipStream_t) { return QX_E_HIP; }
int launch_gemv_a8q(const qx_desc*, const void*, const int8_t*, const float*, uint16_t*, hipStream_t) {
  return QX_E_HIP;
}
bool gemv_multi_applies(const qx_desc*, int) { return false; }
int launch_gemv_multi(const qx_desc*, const void*, int, const uint16_t*, uint16_t*, hipStream_t) { return QX_E_HIP; }
int launch_gemm(const qx_desc*, const void*, int, const uint16_t*, uint16_t*, hipStream_t) { return took("gemm"); }
int launch_gemm_a8(const qx_desc*, const void*, int, const int8_t*, const float*, uint16_t*, hipStream_t) {
  return took("gemm_a8");
}
int launch_gemm_lut_a8(const qx_desc*, const void*, int, const int8_t*, const float*, uint16_t*, hipStream_t) {
  return took("gemm");
}
bool gemm_skinny_applies(const qx_desc* d, int m) { return skinny_applies(d, m); }
int launch_gemm_skinny(const qx_desc*, const void*, int, const uint16_t*, uint16_t*, hipStream_t) {
  return took("skinny");
}
bool gemm_tile_applies(const qx_desc* d, int m, bool a8) { return tile::pick_shape(d, m, a8) != tile::kShapes; }
int launch_gemm_tile(const qx_desc* d, const void*, int m, const void*, const float* sx, uint16_t*, hipStream_t) {
  const char name[2] = {(char)('A' + tile::pick_shape(d, m, sx != nullptr)), 0};
  return took(name);
}
}  // namespace qx

using namespace qx;
using namespace qx::tile;

namespace {

// The load passes the range check by one of two rules (the scalar offset left out of it, or taken
// from the size) and its bytes are not all in the buffer.
bool leaves(ReadAt r, int size, int bytes) {
  const bool out = (unsigned)r.lane >= (unsigned)size;
  const bool out_sub = (unsigned)r.lane >= (unsigned)size - (unsigned)r.scalar;
  return !(out && out_sub) && (long)r.lane + r.scalar + bytes > size;
}

template <int BITS, int KIND, int G, bool A8, int S>
void check_reads() {
  if constexpr (built<BITS, KIND, G, A8>(S)) {
    constexpr ShapeCost sh = kShape[S];
    using TR = TileReads<BITS, KIND, G, sh.mt, sh.nt, sh.wm, sh.sc, sh.ks, A8>;
    long bad_x = 0, bad_code = 0, bad_meta = 0;
    for (const int C : {1, 2, 3, 16}) {
      const int k = 128 * C, G_row = k / G, words = (G_row + 15) / 16;
      for (int t = 0; t < TR::NTH; ++t) {
        for (int rows = 1; rows <= sh.bm; ++rows)
          for (int i = 0; i < TR::XP; ++i) {
            const int row = TR::x_row(i, rows), first = i * (TR::NTH / 8);
            bad_x += row < 0 || row >= rows || (first < rows && row != first);
            for (const int h : {0, 1})
              for (int c = 0; c < C; c += C > 1 ? C - 1 : 1)
                bad_x += leaves(TR::x(t, c, h, k), (rows - row) * k * TR::kXB, TR::kXBytes);
          }
        for (int rows = 1; rows <= sh.bn; ++rows)
          for (int c = 0; c < C; c += sh.sc) {
            for (int i = 0; i < TR::CP; ++i) bad_code += leaves(TR::code(t, i, c, C), rows * BITS * C * 16, TR::kCBytes);
            for (int i = 0; i < TR::MP; ++i) {
              bad_meta += leaves(TR::meta(t, i, c, G_row), rows * G_row * TR::kMRow, TR::kMBytes);
              if (KIND == QX_Q4X) bad_meta += leaves(TR::selectors(t, i, c, words), rows * words * 4, 4);
            }
          }
      }
    }
    std::printf("%d %d %d %d %c %ld %ld %ld\n", BITS, KIND, G, (int)A8, 'A' + S, bad_x, bad_code, bad_meta);
  }
}

template <int BITS, int KIND, int G, bool A8, int S = 0>
void check_format() {
  if constexpr (S < kShapes) {
    check_reads<BITS, KIND, G, A8, S>();
    check_format<BITS, KIND, G, A8, S + 1>();
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 2 && std::strcmp(argv[1], "reads") == 0) {
#define CHECK(B, K, G) check_format<B, K, G, false>(), check_format<B, K, G, true>();
    QX_TILE_FORMATS(CHECK)
    return 0;
  }
  if (argc == 2 && std::strcmp(argv[1], "order") == 0) {
    int nx, my;
    while (std::scanf("%d %d", &nx, &my) == 2) {
      std::vector<int> seen(nx * my);
      bool once = true;
      size_t most = 0;
      const int share = (nx * my + 7) / 8;
      for (int x = 0; x < 8; ++x) {
        std::set<int> weights;
        for (int t = x * share; t < std::min((x + 1) * share, nx * my); ++t) {
          const TileAt at = tile_at(t, nx, my, tile_groups(my));
          once &= at.bn >= 0 && at.bn < nx && at.bm >= 0 && at.bm < my && seen[at.bn * my + at.bm]++ == 0;
          weights.insert(at.bn);
        }
        most = std::max(most, weights.size());
      }
      std::printf("%d %zu\n", (int)once, most);
    }
    return 0;
  }
  if (argc == 2 && std::strcmp(argv[1], "route") == 0) {
    alignas(16) static char buf[16];  // pointers that pass the checks; nothing is read or written
    uint16_t* const h = reinterpret_cast<uint16_t*>(buf);
    int b, kd, g, a8, n, k, m;
    while (std::scanf("%d %d %d %d %d %d %d", &b, &kd, &g, &a8, &n, &k, &m) == 7) {
      const qx_desc d = {n, k, b, g, kd, 0};
      const int st = a8 ? qx_gemm_a8(&d, buf, m, reinterpret_cast<int8_t*>(buf), reinterpret_cast<float*>(buf), h, nullptr)
                        : qx_gemm(&d, buf, m, h, h, nullptr);
      std::printf("%s\n", st == QX_OK ? g_route : "error");
    }
    return 0;
  }
  return 2;
}
