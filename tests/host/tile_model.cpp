// The host side of the tiled GEMM for the CPU tests. Arguments:
//   reads  checks where the loads of every built kernel read: every thread, piece and chunk, for
//          1 .. BM activation rows and 1 .. BN weight rows in a block; prints one line per kernel
//          with the number of loads that leave their buffer by either rule of the range check
//   pick   reads "bits kind group a8 n k m" from standard input, prints the shape's letter, or -
#include <cstdio>
#include <cstring>

#include "../../paper_2505_07531_amd/csrc/gemm_tile_plan.h"

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
  if (argc == 2 && std::strcmp(argv[1], "pick") == 0) {
    int b, kd, g, a8, n, k, m;
    while (std::scanf("%d %d %d %d %d %d %d", &b, &kd, &g, &a8, &n, &k, &m) == 7) {
      const qx_desc d = {n, k, b, g, kd, 0};
      const int shape = pick_shape(&d, m, a8 != 0);
      std::printf("%c\n", shape == kShapes ? '-' : 'A' + shape);
    }
    return 0;
  }
  return 2;
}
