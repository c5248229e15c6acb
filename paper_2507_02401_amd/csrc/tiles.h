// Tile shapes and coarse-kernel sizes: compile-time tables shared by the kernels (which are
// instantiated for them) and the host planner (which tiles level blocks with them).
#pragma once

#include "composite.h"
#include "internal.h"

namespace es {

constexpr int kThreads = 256;  // threads of every level-kernel work-group
constexpr int kA1Rows = 4;     // outputs a thread of the axis-1 pass (K_LP_DOWN_A1) forms

struct Shape3 {
  int a, b, c;
};
constexpr Shape3 shape_of(int K, int D, int V, int L) {
  // V: 0 wide, 1 narrow, 2 medium
  if (K == K_LP_UP2) return V == 0 ? Shape3{1, 64, 128} : (V == 1 ? Shape3{1, 32, 64} : Shape3{1, 32, 128});
  if (K == K_LP_DOWN_P) return V == 0 ? Shape3{1, 16, 64} : (V == 1 ? Shape3{1, 16, 16} : Shape3{1, 16, 32});  // plane, axis 0, axis 2
  if (K == K_LP_DOWN_A1) return Shape3{kThreads, kA1Rows, 1};  // lines (16-byte groups), axis 1
  if (K == K_LP_DOWN_S && D == 3) return V == 0 ? Shape3{16, 8, 32} : (V == 1 ? Shape3{8, 8, 16} : Shape3{8, 8, 32});
  if (K == K_LP_DOWN_S) return V == 0 ? Shape3{1, 64, 64} : (V == 1 ? Shape3{1, 16, 64} : Shape3{1, 32, 64});
  if (K == K_LP_UP_S) return V == 0 ? Shape3{16, 16, 32} : (V == 1 ? Shape3{8, 8, 32} : Shape3{8, 16, 32});
  if (K == K_FB_DOWN_S) return V == 0 ? Shape3{16, 8, 32} : (V == 1 ? Shape3{8, 8, 16} : Shape3{8, 8, 32});
  if (K == K_FB_UP_S) return V == 0 ? Shape3{16, 16, 32} : (V == 1 ? Shape3{8, 8, 32} : Shape3{8, 16, 32});
  if (D == 1) {
    const bool an = (K == K_LP_DOWN || K == K_FB_DOWN);
    return an ? (V == 0 ? Shape3{1, 1, 256} : (V == 1 ? Shape3{1, 1, 64} : Shape3{1, 1, 128}))
              : (V == 0 ? Shape3{1, 1, 512} : (V == 1 ? Shape3{1, 1, 128} : Shape3{1, 1, 256}));
  }
  if (D == 2) {
    switch (K) {
      case K_LP_DOWN: return V == 0 ? Shape3{1, 32, 64} : (V == 1 ? Shape3{1, 8, 16} : Shape3{1, 16, 64});
      case K_LP_UP: return V == 0 ? Shape3{1, 64, 128} : (V == 1 ? Shape3{1, 16, 32} : Shape3{1, 32, 128});
      case K_FB_DOWN: return V == 0 ? Shape3{1, 16, 32} : (V == 1 ? Shape3{1, 8, 16} : Shape3{1, 16, 64});
      default: return V == 0 ? Shape3{1, 32, 64} : (V == 1 ? Shape3{1, 16, 32} : Shape3{1, 32, 128});
    }
  }
  switch (K) {
    case K_LP_DOWN:
      return V == 0 ? (L <= 8 ? Shape3{4, 8, 16} : Shape3{2, 4, 16})
                    : (V == 1 ? Shape3{2, 4, 8} : (L <= 8 ? Shape3{2, 8, 16} : Shape3{2, 4, 8}));
    case K_LP_UP: return V == 0 ? Shape3{4, 16, 32} : (V == 1 ? Shape3{4, 8, 16} : Shape3{4, 8, 32});
    case K_FB_DOWN:
      return V == 0 ? (L <= 8 ? Shape3{2, 8, 16} : Shape3{2, 4, 8}) : (V == 1 ? Shape3{2, 4, 8} : Shape3{2, 4, 16});
    default:
      return V == 0 ? (L <= 8 ? Shape3{4, 16, 16} : Shape3{4, 8, 16})
                    : (V == 1 ? Shape3{4, 8, 16} : (L <= 8 ? Shape3{4, 8, 32} : Shape3{4, 8, 16}));
  }
}
// Output rows per chunk of the streamed 2-D low-pass analysis kernel (measured on 64 x 1024^2 and
// 64 x 512^2 db8 levels against 4 and 16, with strips of 64, 128 and 256 columns).
constexpr int kStreamRows = 8;
// Threads of the low-pass coarse kernel for blocks of at most cmax floats.  A pass of a block of 4096 has 512
// items of four outputs or fewer, and the kernel takes up to 128 registers: 512 threads leave room for two
// work-groups per CU, 1024 for one (batches of more than 256 such blocks then take up to twice as long: 8178 of
// 12 x 20, 8 taps, 110 -> 62 us; 4230 of 16 x 32, 8 taps, 61 -> 34 us; single blocks are as fast with either).
constexpr int coarse_threads(int cmax) { return cmax <= kCoarseMaxBlock ? 512 : 1024; }
// The full-bank coarse kernels' two sizes likewise (41287 blocks of 16 x 8, 16 taps, 1063 -> 550 us; blocks above
// 4096 floats are up to 8 % slower with 512 threads).  Their 3-D analysis of 14 and 16 taps needs 66 registers
// unless it is held to the 64 of two work-groups of 1024.
constexpr int fb_coarse_small(int D) { return D == 1 ? 2048 : 4096; }
constexpr int fb_coarse_threads(int D, int bmax) { return bmax <= fb_coarse_small(D) ? 512 : 1024; }
constexpr int fb_coarse_waves(int D, int L, bool syn, int bmax) {
  return D == 3 && L >= 14 && !syn && bmax > fb_coarse_small(D) ? 8 : 4;
}

// LDS of a block of at most CMAX floats: the pyramid (< 2B in 1-D, < 4B/3 in 2-D, < 8B/7 in 3-D)
// plus the temporaries (1-D: none; 2-D: B/2; 3-D: B/2 + B/2, the second synthesis pass writes a
// half block) stay below 9B/4.  2-D blocks whose coarsest levels run as matrix products (sides of at most
// kDenseSide) hold two of their arrays over (or past) the temporaries, two more and tables behind.
constexpr int kDenseRow = kDenseSide + 4;
constexpr int kDenseBuf = kDenseSide * kDenseRow;
constexpr int kDenseTables = 2 * kDenseSide + kDenseLevels + 2;
constexpr int dense_extra_floats(int tmp) { return (tmp > 2 * kDenseBuf ? tmp : 2 * kDenseBuf) + 2 * kDenseBuf + kDenseTables; }
constexpr int coarse_lds_floats(int D, int cmax) {
  const int passes = cmax / 4 * 9, dense = (cmax / 3 * 4 + 8 + dense_extra_floats(cmax / 2) + 3) & ~3;
  return D != 2 || passes > dense ? passes : dense;
}

inline TileShape tile_shape(int kind, int ndim, int variant, int taps) {
  const Shape3 sh = shape_of(kind, ndim, variant, taps);
  TileShape t;
  t.t[0] = sh.a;
  t.t[1] = sh.b;
  t.t[2] = sh.c;
  return t;
}
inline int tile_threads(int, int, int) { return kThreads; }

// LDS that a coarse kernel needs for a block; it selects one of the kernel's two sizes at launch.
inline size_t tail_lds_bytes(int kind, int D, const int b[3], int) {
  const int block = b[0] * b[1] * b[2];
  return sizeof(float) * (size_t)(kind == 3 ? coarse_lds_floats(D, block) : 2 * block);
}

}  // namespace es
