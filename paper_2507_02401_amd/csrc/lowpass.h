// Low-pass (projection-form) tile and coarse-level bodies: the work of one work-group, used by
// the level kernels (one launch per level) and by the persistent plan kernel alike, so that
// both give identical results.
#pragma once

#include "kcommon.h"
#include "tiles.h"

namespace es {

// ---------------------------------------------------------------------------------------
// LP_DOWN: a_out = A a_in on a (T0,T1,T2) tile of the half-resolution output.

// LDS of one LP_DOWN tile.
template <int D, int L, int T0, int T1, int T2>
struct LpDownSmem {
  using G = DownGeom<D, L, T0, T1, T2>;
  alignas(16) float s_in[G::NROW * G::I2P];
  float s_b[D >= 3 ? T0 * G::I1 * T2 : 1];
  int s_row[G::NROW];
  int s_col[G::NV];
};

// One LP_DOWN tile: work-group index `wg` of task `t` (decoded with the task's tile counts).
// PLANE (D = 2): axes 0 and 2 of a 3-D block on the plane c0 of axis 1; output rows b1 * b2/2 apart.
template <int D, int L, int T0, int T1, int T2, int NT, bool VEC, bool PLANE = false>
DEVI void lp_down_tile(const Task& t, int wg, const Filter& f, LpDownSmem<D, L, T0, T1, T2>& sm) {
  using G = DownGeom<D, L, T0, T1, T2>;
  constexpr int P2 = 4, P1 = 4, P0 = 2;
  float* s_in = sm.s_in;
  float* s_b = sm.s_b;
  int* s_row = sm.s_row;
  int* s_col = sm.s_col;
  const Tile tl = decode_tile(t, wg);
  static_assert(!PLANE || D == 2, "planes are 2-D tiles");
  const int plane = PLANE ? tl.c0 : 0;
  const float* __restrict__ src = t.in0 + tl.inst * t.bs_in0 + plane * t.st_in0[1];
  float* __restrict__ dst = t.out0 + tl.inst * t.bs_out0 + plane * t.st_out0[1];
  const int b0 = t.b[0], b1 = PLANE ? t.b[0] : t.b[1], b2 = t.b[2];
  const int o0 = 2 * T0 * tl.c0, o1 = 2 * T1 * tl.c1, o2 = 2 * T2 * tl.c2;
  const int st1 = PLANE ? t.st_in0[0] : t.st_in0[1];

  for (int i = threadIdx.x; i < G::NROW; i += NT) {
    const int i1 = i % G::I1, i0 = i / G::I1;
    s_row[i] = (D >= 3 ? pmod(o0 + i0, b0) * t.st_in0[0] : 0) + (D >= 2 ? pmod(o1 + i1, b1) * st1 : 0);
  }
  for (int i = threadIdx.x; i < G::NV; i += NT) s_col[i] = VEC ? pmod(o2 + 4 * i, b2) : o2 + 4 * i;
  __syncthreads();
  stage_rows<NT, G::NROW, G::NV, VEC>(src, s_row, s_col, s_in, G::I2P, b2);
  __syncthreads();

  // contiguous dim: (NROW, I2) -> (NROW, T2); results go through registers so that s_a can
  // reuse the staging buffer (smaller LDS footprint, more resident work-groups)
  float* s_a = s_in;
  row_pass_inplace<L, P2, G::NROW, T2, G::I2P, NT, false>(s_in, f);

  const int n1o = b1 >> 1, n2o = b2 >> 1, n0o = b0 >> 1;
  if constexpr (D == 1) {
    // already the output: (1, T2)
    for (int k = threadIdx.x; k < T2; k += NT) {
      const int g2 = T2 * tl.c2 + k;
      if (g2 < n2o) gst(dst + g2, s_a[k]);
    }
  } else if constexpr (D == 2) {
    analysis_pass<L, P1, false, true, NT>(
        T2, T1 / P1, f,
        [&](int c, int j0, float* w) {
#pragma unroll
          for (int j = 0; j < 2 * P1 + L - 2; ++j) w[j] = s_a[(j0 + j) * T2 + c];
        },
        [&](int c, int k, float lo, float) {
          const int g1 = T1 * tl.c1 + k, g2 = T2 * tl.c2 + c;
          if (g1 < n1o && g2 < n2o) gst(dst + g1 * (PLANE ? t.st_out0[0] : n2o) + g2, lo);
        });
  } else {
    // dim 0: (I0, I1, T2) -> (T0, I1, T2), lines are (i1, c)
    analysis_pass<L, P0, false, true, NT>(
        G::I1 * T2, T0 / P0, f,
        [&](int l, int j0, float* w) {
#pragma unroll
          for (int j = 0; j < 2 * P0 + L - 2; ++j) w[j] = s_a[(j0 + j) * G::I1 * T2 + l];
        },
        [&](int l, int k, float lo, float) { s_b[k * G::I1 * T2 + l] = lo; });
    __syncthreads();
    // dim 1: (T0, I1, T2) -> (T0, T1, T2), lines are (k0, c)
    analysis_pass<L, P1, false, true, NT>(
        T0 * T2, T1 / P1, f,
        [&](int l, int j0, float* w) {
          const int c = l % T2, k0 = l / T2;
#pragma unroll
          for (int j = 0; j < 2 * P1 + L - 2; ++j) w[j] = s_b[(k0 * G::I1 + j0 + j) * T2 + c];
        },
        [&](int l, int k, float lo, float) {
          const int c = l % T2, k0 = l / T2;
          const int g0 = T0 * tl.c0 + k0, g1 = T1 * tl.c1 + k, g2 = T2 * tl.c2 + c;
          if (g0 < n0o && g1 < n1o && g2 < n2o) gst(dst + (g0 * n1o + g1) * n2o + g2, lo);
        });
  }
}

// ---------------------------------------------------------------------------------------
// LP_DOWN streamed along axis 1 (2-D): a_out = A a_in for a strip of T2 output columns and a
// run of R output rows per work-group.  The run's input rows are visited in chunks of CR = 2 RB
// rows; each row is filtered along axis 2 exactly once, into a ring holding the last W = CR + L - 2
// filtered rows (the rows that RB output rows read), and RB output rows are formed per chunk from
// the ring along axis 1.  Every ring row but the last is also written W rows further on (a
// mirror), so a window of up to W consecutive ring rows never wraps and is read at fixed offsets.
// The next chunk's 16-byte loads are in flight while the current chunk is filtered.  The
// arithmetic per output is that of lp_down_tile (axis 2, then axis 1, taps in order), so both
// give identical results.
template <int L, int R, int T2, int RB>
struct LpDownStreamGeom {
  static constexpr int CR = 2 * RB;                          // input rows per chunk
  static constexpr int W = CR + L - 2;                       // ring rows the outputs of a chunk read
  static constexpr int NRING = 2 * W - 1;                    // with the mirror
  static constexpr int NC = (2 * R + L - 2 + CR - 1) / CR;   // chunks of a run
  static constexpr int I2 = 2 * T2 + L - 2;
  static constexpr int I2P = (I2 + 3) & ~3;
  static constexpr int NV = I2P / 4;
};

template <int L, int R, int T2, int RB>
struct LpDownStreamSmem {
  using G = LpDownStreamGeom<L, R, T2, RB>;
  alignas(16) float s_in[G::CR * G::I2P];
  alignas(16) float s_ring[G::NRING * T2];
  int s_row[G::NC * G::CR];
  int s_col[G::NV];
};

template <int L, int R, int T2, int RB, int NT, bool VEC>
DEVI void lp_down_stream(const Task& t, int wg, const Filter& f, LpDownStreamSmem<L, R, T2, RB>& sm) {
  using G = LpDownStreamGeom<L, R, T2, RB>;
  constexpr int CR = G::CR, W = G::W, NC = G::NC, I2P = G::I2P, NV = G::NV;
  constexpr int P = 4, NCH = T2 / P;              // axis-2 pass: P outputs per task
  constexpr int CPT = NT / T2 > 0 ? NT / T2 : 1;  // axis-1 pass: tasks per column
  constexpr int RPT = RB / CPT;                   // output rows per axis-1 task
  constexpr int WC = 2 * RPT + L - 2;             // ring rows one axis-1 task reads
  static_assert(T2 % P == 0 && RB % CPT == 0 && RPT >= 1 && WC <= W, "tile shape");
  float* s_in = sm.s_in;
  float* s_ring = sm.s_ring;
  int* s_row = sm.s_row;
  int* s_col = sm.s_col;
  const Tile tl = decode_tile(t, wg);
  const float* __restrict__ src = t.in0 + tl.inst * t.bs_in0;
  float* __restrict__ dst = t.out0 + tl.inst * t.bs_out0;
  const int b1 = t.b[1], b2 = t.b[2];
  const int h1 = b1 >> 1, h2 = b2 >> 1;
  const int k0 = R * tl.c1, o2 = 2 * T2 * tl.c2;
  for (int i = threadIdx.x; i < NC * CR; i += NT) s_row[i] = pmod(2 * k0 + i, b1) * t.st_in0[1];
  for (int i = threadIdx.x; i < NV; i += NT) s_col[i] = VEC ? pmod(o2 + 4 * i, b2) : o2 + 4 * i;
  __syncthreads();

  constexpr int NLD = CR * NV, ITL = (NLD + NT - 1) / NT;
  float4 pf[VEC ? ITL : 1];
  auto load_chunk = [&](int c) {
#pragma unroll
    for (int it = 0; it < ITL; ++it) {
      const int q = min(int(threadIdx.x) + it * NT, NLD - 1);
      pf[it] = gld4(src + s_row[c * CR + q / NV] + s_col[q % NV]);
    }
  };
  if constexpr (VEC) load_chunk(0);

  for (int c = 0; c < NC; ++c) {
    if constexpr (VEC) {
      float4* d4 = reinterpret_cast<float4*>(s_in);  // row length I2P = 4 NV: LDS slot = load index
#pragma unroll
      for (int it = 0; it < ITL; ++it) d4[min(int(threadIdx.x) + it * NT, NLD - 1)] = pf[it];
      __syncthreads();
      if (c + 1 < NC) load_chunk(c + 1);
    } else {
      stage_rows<NT, CR, NV, false>(src, s_row + c * CR, s_col, s_in, I2P, b2);
      __syncthreads();
    }
    // axis 2: the chunk's rows into their ring slots (and mirrors)
    const int sb = (c * CR) % W;
    for (int task = threadIdx.x; task < CR * NCH; task += NT) {
      const int ch = task % NCH, r = task / NCH;
      constexpr int WN = 2 * P + L - 2, W4 = (WN + 3) / 4;
      const float4* p4 = reinterpret_cast<const float4*>(s_in + r * I2P + 2 * P * ch);
      float win[4 * W4];
#pragma unroll
      for (int v = 0; v < W4; ++v) {
        const float4 x = p4[v];
        win[4 * v] = x.x; win[4 * v + 1] = x.y; win[4 * v + 2] = x.z; win[4 * v + 3] = x.w;
      }
      float a[P];
#pragma unroll
      for (int q = 0; q < P; ++q) {
        a[q] = 0.f;
#pragma unroll
        for (int tt = 0; tt < L; ++tt) a[q] = fmaf(f.h[tt], win[2 * q + tt], a[q]);
      }
      const float4 o = make_float4(a[0], a[1], a[2], a[3]);
      const int slot = sb + r >= W ? sb + r - W : sb + r;
      *reinterpret_cast<float4*>(s_ring + slot * T2 + P * ch) = o;
      if (slot < W - 1) *reinterpret_cast<float4*>(s_ring + (slot + W) * T2 + P * ch) = o;
    }
    __syncthreads();
    // axis 1: output rows kb .. kb + RB - 1 of the run (input rows 2 kb .. 2 kb + W - 1)
    const int kb = RB * c - (L / 2 - 1);
    if (kb + RB > 0) {
      for (int task = threadIdx.x; task < T2 * CPT; task += NT) {
        const int col = task % T2, part = task / T2;
        const int kp = kb + RPT * part;
        const float* rp = s_ring + pmod(2 * kp, W) * T2 + col;
        float win[WC];
#pragma unroll
        for (int j = 0; j < WC; ++j) win[j] = rp[j * T2];
        const int g2 = T2 * tl.c2 + col;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          float a = 0.f;
#pragma unroll
          for (int tt = 0; tt < L; ++tt) a = fmaf(f.h[tt], win[2 * r + tt], a);
          const int k = kp + r;
          if (k >= 0 && k < R && k0 + k < h1 && g2 < h2) gst(dst + (k0 + k) * h2 + g2, a);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// LP_UP: out = alpha*same + beta*(A^T z) on a (U0,U1,U2) full-resolution tile.

// LDS of one LP_UP tile.
template <int D, int L, int U0, int U1, int U2>
struct LpUpSmem {
  using G = UpGeom<D, L, U0, U1, U2>;
  alignas(16) float s_in[G::NROW * G::J2P];
  alignas(16) float s_a[G::NROW * U2];
  float s_b[D >= 3 ? U0 * G::J1 * U2 : 1];
  int s_row[G::NROW];
  int s_col[G::NV];
};

// One LP_UP tile: work-group index `wg` of task `t`.
// CGE (2-D vector path only; the conjugate-gradient solver's operator step): the output is
// out = (alpha + gamma * m) * same + beta * (A^T z) with m = in2 (a per-element mask), and the
// work-group's compensated sum of same * out goes to out1[wg - tile_begin] (one float).
template <int D, int L, int U0, int U1, int U2, int NT, bool VEC, bool CGE = false>
DEVI void lp_up_tile(const Task& t, int wg, const Filter& f, LpUpSmem<D, L, U0, U1, U2>& sm) {
  using G = UpGeom<D, L, U0, U1, U2>;
  constexpr int H = G::H;
  constexpr int P2 = 4, P1 = 4, P0 = 2;
  float* s_in = sm.s_in;
  float* s_a = sm.s_a;
  float* s_b = sm.s_b;
  int* s_row = sm.s_row;
  int* s_col = sm.s_col;
  const Tile tl = decode_tile(t, wg);
  const float* __restrict__ z = t.in0 + tl.inst * t.bs_in0;
  const float* same = t.in1 + tl.inst * t.bs_in1;  // may alias out (in-place z over a)
  float* out = t.out0 + tl.inst * t.bs_out0;
  const int b0 = t.b[0], b1 = t.b[1], b2 = t.b[2];
  const int h0 = b0 >> 1, h1 = b1 >> 1, h2 = b2 >> 1;  // z dims
  const int r0 = tl.c0 * (U0 / 2) - (H - 1), r1 = tl.c1 * (U1 / 2) - (H - 1);
  const int r2 = tl.c2 * (U2 / 2) - (H - 1) - G::OFF;

  // 2-D vector path: the last pass gives each lane 4 adjacent columns and PQ row pairs; the
  // lane's `same` values are loaded first, so that their latency overlaps the staging and
  // filtering of z (same has no halo: each work-group reads and writes only its own tile)
  constexpr int C4 = U2 / 4, PQ = 2;
  constexpr bool FAST2 = D == 2 && VEC && (U1 / 2) % PQ == 0;
  constexpr int NT2 = C4 * (U1 / 2 / PQ), IT2 = (NT2 + NT - 1) / NT;
  static_assert(!CGE || FAST2, "the solver epilogue exists on the 2-D vector path only");
  float4 xs[FAST2 ? IT2 : 1][FAST2 ? 2 * PQ : 1];
  float4 ms[CGE ? IT2 : 1][CGE ? 2 * PQ : 1];
  const float* mask = CGE && t.in2 ? t.in2 + tl.inst * t.bs_in2 : nullptr;  // the same for the whole launch
  if constexpr (FAST2) {
#pragma unroll
    for (int it = 0; it < IT2; ++it) {
      const int task = threadIdx.x + it * NT;
      const int c4 = task % C4, ch = task / C4;
      const int g2 = tl.c2 * U2 + 4 * c4;
#pragma unroll
      for (int r = 0; r < 2 * PQ; ++r) {
        const int g1 = tl.c1 * U1 + 2 * PQ * ch + r;
        const bool in = task < NT2 && g1 < b1 && g2 < b2;
        xs[it][r] = in ? gld4(same + g1 * b2 + g2) : make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (CGE) ms[it][r] = in && mask ? gld4(mask + g1 * b2 + g2) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
  KSum cg_acc;
  const bool stream = (t.flags & kStream) != 0;

  for (int i = threadIdx.x; i < G::NROW; i += NT) {
    const int i1 = i % G::J1, i0 = i / G::J1;
    s_row[i] = (D >= 3 ? pmod(r0 + i0, h0) * (h1 * h2) : 0) + (D >= 2 ? pmod(r1 + i1, h1) * h2 : 0);
  }
  for (int i = threadIdx.x; i < G::NV; i += NT) s_col[i] = VEC ? pmod(r2 + 4 * i, h2) : r2 + 4 * i;
  __syncthreads();
  stage_rows<NT, G::NROW, G::NV, VEC>(z, s_row, s_col, s_in, G::J2P, h2);
  __syncthreads();

  // contiguous dim: (NROW, J2) -> (NROW, U2)
  synthesis_pass<L, P2, false, false, NT>(
      G::NROW, U2 / 2 / P2, f,
      [&](int l, int j0, float* lo, float*) {
        const float* p = s_in + l * G::J2P + G::OFF + j0;
#pragma unroll
        for (int j = 0; j < P2 + H - 1; ++j) lo[j] = p[j];
      },
      [&](int l, int p, float e0, float e1) {
        s_a[l * U2 + p] = e0;
        s_a[l * U2 + p + 1] = e1;
      });
  __syncthreads();

  const float alpha = t.alpha, beta = t.beta;
  if constexpr (D == 1) {
    for (int p = threadIdx.x; p < U2; p += NT) {
      const int g2 = tl.c2 * U2 + p;
      if (g2 < b2) gst(out + g2, fmaf(alpha, gld(same + g2), beta * s_a[p]));
    }
  } else if constexpr (FAST2) {
    // axis 1 with 4 columns per lane: float4 LDS reads, float4 global stores; per output the
    // arithmetic of synthesis_pass (oldest window sample first)
#pragma unroll
    for (int it = 0; it < IT2; ++it) {
      const int task = threadIdx.x + it * NT;
      if (task < NT2) {
        const int c4 = task % C4, ch = task / C4;
        const int g2 = tl.c2 * U2 + 4 * c4;
        float4 lo[PQ + H - 1];
#pragma unroll
        for (int j = 0; j < PQ + H - 1; ++j) lo[j] = *reinterpret_cast<const float4*>(s_a + (PQ * ch + j) * U2 + 4 * c4);
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
          float4 e0 = make_float4(0.f, 0.f, 0.f, 0.f), e1 = e0;
#pragma unroll
          for (int j = H - 1; j >= 0; --j) {
            const float4 v = lo[q + H - 1 - j];
            e0.x = fmaf(f.h[2 * j], v.x, e0.x); e1.x = fmaf(f.h[2 * j + 1], v.x, e1.x);
            e0.y = fmaf(f.h[2 * j], v.y, e0.y); e1.y = fmaf(f.h[2 * j + 1], v.y, e1.y);
            e0.z = fmaf(f.h[2 * j], v.z, e0.z); e1.z = fmaf(f.h[2 * j + 1], v.z, e1.z);
            e0.w = fmaf(f.h[2 * j], v.w, e0.w); e1.w = fmaf(f.h[2 * j + 1], v.w, e1.w);
          }
          const int g1 = tl.c1 * U1 + 2 * (PQ * ch + q);
          if (g1 < b1 && g2 < b2) {
            const float4 s0 = xs[it][2 * q], s1 = xs[it][2 * q + 1];
            if constexpr (CGE) {
              const float gm = t.gamma;
              const float4 m0 = ms[it][2 * q], m1 = ms[it][2 * q + 1];
              const float4 y0 = make_float4(
                  fmaf(fmaf(gm, m0.x, alpha), s0.x, beta * e0.x), fmaf(fmaf(gm, m0.y, alpha), s0.y, beta * e0.y),
                  fmaf(fmaf(gm, m0.z, alpha), s0.z, beta * e0.z), fmaf(fmaf(gm, m0.w, alpha), s0.w, beta * e0.w));
              const float4 y1 = make_float4(
                  fmaf(fmaf(gm, m1.x, alpha), s1.x, beta * e1.x), fmaf(fmaf(gm, m1.y, alpha), s1.y, beta * e1.y),
                  fmaf(fmaf(gm, m1.z, alpha), s1.z, beta * e1.z), fmaf(fmaf(gm, m1.w, alpha), s1.w, beta * e1.w));
              gst4(out + g1 * b2 + g2, y0);
              gst4(out + (g1 + 1) * b2 + g2, y1);
              cg_acc.add(s0.x * y0.x); cg_acc.add(s0.y * y0.y); cg_acc.add(s0.z * y0.z); cg_acc.add(s0.w * y0.w);
              cg_acc.add(s1.x * y1.x); cg_acc.add(s1.y * y1.y); cg_acc.add(s1.z * y1.z); cg_acc.add(s1.w * y1.w);
            } else {
              const float4 y0 = make_float4(fmaf(alpha, s0.x, beta * e0.x), fmaf(alpha, s0.y, beta * e0.y),
                                            fmaf(alpha, s0.z, beta * e0.z), fmaf(alpha, s0.w, beta * e0.w));
              const float4 y1 = make_float4(fmaf(alpha, s1.x, beta * e1.x), fmaf(alpha, s1.y, beta * e1.y),
                                            fmaf(alpha, s1.z, beta * e1.z), fmaf(alpha, s1.w, beta * e1.w));
              gst4_if(stream, out + g1 * b2 + g2, y0);
              gst4_if(stream, out + (g1 + 1) * b2 + g2, y1);
            }
          }
        }
      }
    }
  } else if constexpr (D == 2) {
    synthesis_pass<L, P1, false, true, NT>(
        U2, U1 / 2 / P1, f,
        [&](int c, int j0, float* lo, float*) {
#pragma unroll
          for (int j = 0; j < P1 + H - 1; ++j) lo[j] = s_a[(j0 + j) * U2 + c];
        },
        [&](int c, int p, float e0, float e1) {
          const int g1 = tl.c1 * U1 + p, g2 = tl.c2 * U2 + c;
          if (g1 < b1 && g2 < b2) {
            const int o = g1 * b2 + g2;
            const float s0 = gld(same + o), s1 = gld(same + o + b2);
            gst(out + o, fmaf(alpha, s0, beta * e0));
            gst(out + o + b2, fmaf(alpha, s1, beta * e1));
          }
        });
  } else {
    // dim 0: (J0, J1, U2) -> (U0, J1, U2)
    synthesis_pass<L, P0, false, true, NT>(
        G::J1 * U2, U0 / 2 / P0, f,
        [&](int l, int j0, float* lo, float*) {
#pragma unroll
          for (int j = 0; j < P0 + H - 1; ++j) lo[j] = s_a[(j0 + j) * G::J1 * U2 + l];
        },
        [&](int l, int p, float e0, float e1) {
          s_b[p * G::J1 * U2 + l] = e0;
          s_b[(p + 1) * G::J1 * U2 + l] = e1;
        });
    __syncthreads();
    synthesis_pass<L, P1, false, true, NT>(
        U0 * U2, U1 / 2 / P1, f,
        [&](int l, int j0, float* lo, float*) {
          const int c = l % U2, p0 = l / U2;
#pragma unroll
          for (int j = 0; j < P1 + H - 1; ++j) lo[j] = s_b[(p0 * G::J1 + j0 + j) * U2 + c];
        },
        [&](int l, int p, float e0, float e1) {
          const int c = l % U2, p0 = l / U2;
          const int g0 = tl.c0 * U0 + p0, g1 = tl.c1 * U1 + p, g2 = tl.c2 * U2 + c;
          if (g0 < b0 && g1 < b1 && g2 < b2) {
            const int o = (g0 * b1 + g1) * b2 + g2;
            const float s0 = gld(same + o), s1 = gld(same + o + b2);
            gst(out + o, fmaf(alpha, s0, beta * e0));
            gst(out + o + b2, fmaf(alpha, s1, beta * e1));
          }
        });
  }
  if constexpr (CGE) {
    __shared__ float2 cg_sum;
    store_wg_sum<NT>(cg_acc, &cg_sum);  // every thread; thread 0 holds the pair
    if (threadIdx.x == 0) gst(t.out1 + (wg - t.tile_begin), cg_sum.x + cg_sum.y);
  }
}

// ---------------------------------------------------------------------------------------
// LP_COARSE: the coarse levels of the projection form for one instance in one work-group.
// Input a_T (a contiguous block of at most CMAX floats), output z_T in place (or y when
// T = 0).  Everything between the load and the store stays in a static LDS array addressed by
// integer offsets: A_0 = a_T, A_1 = a_{T+1}, ..., A_K, then two half-size temporaries.
//   down:  A_{j+1} = A A_j                       (separable, contiguous axis first)
//   top:   A_K *= c_{T+K}
//   up:    A_j = coef_j A_j + A^T A_{j+1}        (j = K-1 .. 0; coef_0 is the output weight)
// Axes at least L long wrap with one compare; shorter ones use the modulo (periodic folding).


// Block of B <= CMAX contiguous floats into LDS and back, in 16-byte accesses where the address and
// the length allow, every load of a thread in flight before its first LDS store; `meanwhile` runs while
// they are.
template <int NT, int CMAX, class F>
DEVI void block_to_lds(const float* in, float* sm, int B, F meanwhile) {
  if ((((uintptr_t)in & 15) | (B & 3)) == 0) {
    constexpr int U = (CMAX / 4 + NT - 1) / NT;
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = threadIdx.x + u * NT;
      v[u] = e < B / 4 ? gld4(in + 4 * e) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    meanwhile();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = threadIdx.x + u * NT;
      if (e < B / 4) reinterpret_cast<float4*>(sm)[e] = v[u];
    }
  } else {
    meanwhile();
    gather_to_lds<NT, CMAX / NT>(
        B, [&](int e) { return gld(in + e); }, [&](int e, float v) { sm[e] = v; });
  }
}
template <int NT>
DEVI void block_from_lds(const float* sm, float* out, int B) {
  if ((((uintptr_t)out & 15) | (B & 3)) == 0)
    for (int e = threadIdx.x; e < B / 4; e += NT) gst4(out + 4 * e, reinterpret_cast<const float4*>(sm)[e]);
  else
    for (int e = threadIdx.x; e < B; e += NT) gst(out + e, sm[e]);
}

template <int L, bool SHORT, int NT>
DEVI void coarse_analysis_w(float* sm, int src, int dst, int n0, int n1, int n2, int ax, const Filter& f) {
  // sm[src] holds an (n0, n1, n2) block; writes the low half along ax, (.., n_ax/2, ..), to sm[dst]
  const int n = ax == 0 ? n0 : (ax == 1 ? n1 : n2);
  const int o0 = ax == 0 ? n0 >> 1 : n0, o1 = ax == 1 ? n1 >> 1 : n1, o2 = ax == 2 ? n2 >> 1 : n2;
  const int total = o0 * o1 * o2;
  const int l1 = ilog2_or_neg(o1), l2 = ilog2_or_neg(o2);
  const int step = ax == 0 ? n1 * n2 : (ax == 1 ? n2 : 1);
  for (int e = threadIdx.x; e < total; e += NT) {
    int c0, c1, c2;
    split3(e, o1, o2, l1, l2, c0, c1, c2);
    const int k = ax == 0 ? c0 : (ax == 1 ? c1 : c2);
    const int base = src + (ax == 0 ? 0 : c0 * n1 * n2) + (ax == 1 ? 0 : c1 * n2) + (ax == 2 ? 0 : c2);
    float acc = 0.f;
    if (!SHORT) {  // n >= L: an index wraps at most once
#pragma unroll
      for (int t = 0; t < L; ++t) {
        const int i = 2 * k + t;
        acc = fmaf(f.h[t], sm[base + (i >= n ? i - n : i) * step], acc);
      }
    } else {
#pragma unroll
      for (int t = 0; t < L; ++t) acc = fmaf(f.h[t], sm[base + ((2 * k + t) % n) * step], acc);
    }
    sm[dst + e] = acc;
  }
}

template <int L, bool SHORT, int NT>
DEVI void coarse_synthesis_w(float* sm, int src, int dst, int n0, int n1, int n2, int ax, const Filter& f, bool combine,
                             float alpha) {
  // sm[src] holds the low half along ax of an (n0, n1, n2) block; writes the full block to
  // sm[dst] (dst = alpha*dst + value when combine)
  const int n = ax == 0 ? n0 : (ax == 1 ? n1 : n2), half = n >> 1;
  const int h0 = ax == 0 ? half : n0, h1 = ax == 1 ? half : n1, h2 = ax == 2 ? half : n2;
  const int total = n0 * n1 * n2;
  const int step = ax == 0 ? h1 * h2 : (ax == 1 ? h2 : 1);
  const int l1 = ilog2_or_neg(n1), l2 = ilog2_or_neg(n2);
  (void)h0;
  for (int e = threadIdx.x; e < total; e += NT) {
    int c0, c1, c2;
    split3(e, n1, n2, l1, l2, c0, c1, c2);
    const int p = ax == 0 ? c0 : (ax == 1 ? c1 : c2);
    const int base = src + (ax == 0 ? 0 : c0 * h1 * h2) + (ax == 1 ? 0 : c1 * h2) + (ax == 2 ? 0 : c2);
    const int par = p & 1, q = p >> 1;
    float acc = 0.f;
    if (!SHORT) {  // half >= L/2: an index wraps at most once
#pragma unroll
      for (int j = 0; j < L / 2; ++j) {
        const int k = q - j;
        acc = fmaf(par ? f.h[2 * j + 1] : f.h[2 * j], sm[base + (k < 0 ? k + half : k) * step], acc);
      }
    } else {
#pragma unroll
      for (int j = 0; j < L / 2; ++j)
        acc = fmaf(par ? f.h[2 * j + 1] : f.h[2 * j], sm[base + pmod(q - j, half) * step], acc);
    }
    sm[dst + e] = combine ? fmaf(alpha, sm[dst + e], acc) : acc;
  }
}

// The passes of a coarse level are bound by issued instructions: a pass of a small level takes as long
// as one wave's chain of them, a pass of a large level as the ~200 instructions that a task took while its
// indices were split by shifts or divisions, multiplied by strides and wrapped element by element
// (1100-4000 cycles a pass, a quarter of them sums).  So items are laid out on powers of two (idle
// lanes where a count is none), a thread keeps its place along the contiguous direction and steps along
// the other one, and window offsets are formed once per thread; windows are 16-byte vectors along the
// contiguous axis and four columns per lane along the strided ones, and the last pass stores to global
// memory.  Per output the taps are summed in the order of the _w versions.  Together with the matrix
// products below, between the first and the last instruction of one work-group: 128^2, 8 taps, 5 levels
// 34800 -> 23200 cycles; 64^2, 16 taps, 4 levels 22600 -> 13900.  As a launch: one 128^2 db4 image 16.2 -> 11.7
// us, the 64 blocks of 128^2 of a 64 x 1024^2 db8 batch 19.5 -> 17.9, one 128^2 db6 block 15.4 -> 12.5.

DEVI int ceil_log2(int v) { return v <= 1 ? 0 : 32 - __builtin_clz(v - 1); }

// Row passes: a thread takes chunk ch (four half-resolution positions) of every 2^lg-th line.  Lines of a 1-D block may
// have more chunks than the work-group threads (each(): one after the other); those of 2-D and 3-D blocks, whose
// lines of CMAX / 2 samples at most leave no more, run their pass once.
template <int D, int NT, class F>
DEVI void coarse_chunks(int half, int lines, F each) {
  const int nch = half / 4;
  if constexpr (D == 1) {
    const int lg = min(ceil_log2(nch), ceil_log2(NT));
    for (int ch = threadIdx.x & ((1 << lg) - 1); ch < nch; ch += 1 << lg) each(ch, lg);
  } else {
    const int lg = ceil_log2(nch), ch = threadIdx.x & ((1 << lg) - 1);
    if (ch < nch && (int)(threadIdx.x >> lg) < lines) each(ch, lg);
  }
}

// (lines, n) -> (lines, n / 2); n / 2 and the offsets multiples of 4
template <int L, int NT>
DEVI void coarse_rows_down(float* sm, int src, int dst, int lines, int n, int ch, int lg, const Filter& f) {
  constexpr int PO = 4, W4 = (2 * PO + L - 2 + 3) / 4;
  const int o = n >> 1, l0 = threadIdx.x >> lg;
  int off[W4];
#pragma unroll
  for (int v = 0; v < W4; ++v) {
    const int i = 2 * PO * ch + 4 * v;
    off[v] = i >= n ? i - n : i;
  }
  const float* in = sm + src + l0 * n;
  float* out = sm + dst + l0 * o + PO * ch;
  const int ls = NT >> lg;
  for (int l = l0; l < lines; l += ls, in += ls * n, out += ls * o) {
    float win[4 * W4];
#pragma unroll
    for (int v = 0; v < W4; ++v) {
      const float4 x = *reinterpret_cast<const float4*>(in + off[v]);
      win[4 * v] = x.x; win[4 * v + 1] = x.y; win[4 * v + 2] = x.z; win[4 * v + 3] = x.w;
    }
    float r[PO];
#pragma unroll
    for (int q = 0; q < PO; ++q) {
      r[q] = 0.f;
#pragma unroll
      for (int t = 0; t < L; ++t) r[q] = fmaf(f.h[t], win[2 * q + t], r[q]);
    }
    *reinterpret_cast<float4*>(out) = make_float4(r[0], r[1], r[2], r[3]);
  }
}

// Items of a strided pass: (position along the axis, four columns), the columns padded to a power of two;
// a thread keeps its columns and steps over positions, then over the outer index.
struct ColItems {
  int c, p, ps;  // first column, first position (outer * count + k) and its step
};
template <int NT>
DEVI ColItems col_items(int inner) {
  const int lc = ceil_log2(inner >> 2);
  const int c = 4 * (threadIdx.x & ((1 << lc) - 1));
  return ColItems{c < inner ? c : -1, (int)(threadIdx.x >> lc), NT >> lc};
}
DEVI float4 axpy4(float a, const float4& x, const float4& y) {
  return make_float4(fmaf(a, x.x, y.x), fmaf(a, x.y, y.y), fmaf(a, x.z, y.z), fmaf(a, x.w, y.w));
}

// (outer, n, inner) -> (outer, n / 2, inner); inner and the offsets multiples of 4
template <int L, int NT>
DEVI void coarse_cols_down(float* sm, int src, int dst, int outer, int n, int inner, const Filter& f) {
  const int o = n >> 1;
  const ColItems it = col_items<NT>(inner);
  if (it.c < 0) return;
  for (int p = it.p; p < outer * o; p += it.ps) {
    const int q = outer == 1 ? 0 : p / o, k = p - q * o, wrap = n - 2 * k;
    const float* in = sm + src + (q * n + 2 * k) * inner + it.c;
    float4 win[L];
#pragma unroll
    for (int j = 0; j < L; ++j) win[j] = *reinterpret_cast<const float4*>(in + (j >= wrap ? j - n : j) * inner);
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < L; ++j) r = axpy4(f.h[j], win[j], r);
    *reinterpret_cast<float4*>(sm + dst + p * inner + it.c) = r;
  }
}

// (lines, n / 2) -> (lines, n): four half-resolution positions per item; n / 2 and the offsets multiples of
// 4; combine: dst = alpha dst + value
template <int L, int NT>
DEVI void coarse_rows_up(float* sm, int src, int dst, int lines, int n, int ch, int lg, const Filter& f, bool combine,
                         float alpha) {
  constexpr int H = L / 2, PO = 4, A = (H - 1 + 3) & ~3, NW = (A + PO) / 4;
  const int half = n >> 1, l0 = threadIdx.x >> lg;
  int off[NW];
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    const int k = PO * ch - A + 4 * v;
    off[v] = k < 0 ? k + half : k;
  }
  const float* in = sm + src + l0 * half;
  float* out = sm + dst + l0 * n + 2 * PO * ch;
  const int ls = NT >> lg;
  for (int l = l0; l < lines; l += ls, in += ls * half, out += ls * n) {
    float win[A + PO];
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      const float4 x = *reinterpret_cast<const float4*>(in + off[v]);
      win[4 * v] = x.x; win[4 * v + 1] = x.y; win[4 * v + 2] = x.z; win[4 * v + 3] = x.w;
    }
    float v[2 * PO];
#pragma unroll
    for (int r = 0; r < 2 * PO; ++r) {
      v[r] = 0.f;
#pragma unroll
      for (int j = 0; j < H; ++j) v[r] = fmaf(f.h[2 * j + (r & 1)], win[A + (r >> 1) - j], v[r]);
    }
#pragma unroll
    for (int r = 0; r < 2 * PO; r += 4) {
      float4 s = make_float4(v[r], v[r + 1], v[r + 2], v[r + 3]);
      float4* o = reinterpret_cast<float4*>(out + r);
      if (combine) s = axpy4(alpha, *o, s);
      *o = s;
    }
  }
}

// (outer, n / 2, inner) -> (outer, n, inner), both outputs of a half-resolution position per item; inner and
// the offsets multiples of 4; combine as above.  gout (16-byte aligned): the result goes there instead of
// to dst.
template <int L, int NT>
DEVI void coarse_cols_up(float* sm, int src, int dst, int outer, int n, int inner, const Filter& f, bool combine,
                         float alpha, float* gout) {
  constexpr int H = L / 2;
  const int half = n >> 1;
  const ColItems it = col_items<NT>(inner);
  if (it.c < 0) return;
  for (int p = it.p; p < outer * half; p += it.ps) {
    const int q = outer == 1 ? 0 : p / half, k = p - q * half;
    const float* in = sm + src + p * inner + it.c;
    float4 win[H];
#pragma unroll
    for (int j = 0; j < H; ++j) win[j] = *reinterpret_cast<const float4*>(in - (j > k ? j - half : j) * inner);
    float4 e0 = make_float4(0.f, 0.f, 0.f, 0.f), e1 = e0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
      e0 = axpy4(f.h[2 * j], win[j], e0);
      e1 = axpy4(f.h[2 * j + 1], win[j], e1);
    }
    const int o = 2 * p * inner + it.c;
    if (combine) {
      e0 = axpy4(alpha, *reinterpret_cast<const float4*>(sm + dst + o), e0);
      e1 = axpy4(alpha, *reinterpret_cast<const float4*>(sm + dst + o + inner), e1);
    }
    if (gout) {
      gst4(gout + o, e0);
      gst4(gout + o + inner, e1);
    } else {
      *reinterpret_cast<float4*>(sm + dst + o) = e0;
      *reinterpret_cast<float4*>(sm + dst + o + inner) = e1;
    }
  }
}

// Analysis of strided axes whose inner count is no multiple of 4 (rows halved to 18, say; the synthesis has whole
// rows): a thread forms four outputs of one column from one window.  In the kernels of small blocks only: the larger
// ones' code stays short, since much of a launch of few work-groups is the wait for it.
template <int L, int NT>
DEVI void coarse_cols_down_1(float* sm, int src, int dst, int outer, int n, int inner, const Filter& f) {
  constexpr int PO = 4, WN = 2 * PO + L - 2;
  const int o = n >> 1, per = o / PO * inner;
  for (int e = threadIdx.x; e < outer * per; e += NT) {
    const int q = outer == 1 ? 0 : e / per, r = e - q * per, k0 = PO * (r / inner), c = r % inner, wrap = n - 2 * k0;
    const float* in = sm + src + (q * n + 2 * k0) * inner + c;
    float win[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) win[j] = in[(j >= wrap ? j - n : j) * inner];
    float* out = sm + dst + (q * o + k0) * inner + c;
#pragma unroll
    for (int p = 0; p < PO; ++p) {
      float v = 0.f;
#pragma unroll
      for (int t = 0; t < L; ++t) v = fmaf(f.h[t], win[2 * p + t], v);
      out[p * inner] = v;
    }
  }
}

// Uniform dispatch over an (n0, n1, n2) block.  Axes shorter than the filter (halves shorter than L / 2
// for the synthesis) fold periodically: the _w versions, as where a count or an offset does not divide.
// One instantiation serves every level: variants of its own for the largest and the smallest levels were
// up to 20 % faster per pass in a loop of the same launch, but between other launches each variant's
// first pass waits for its code (~100 cycles per 64 bytes), which cost more than it gave.
template <int D, int L, int NT>
DEVI void coarse_analysis(float* sm, int src, int dst, int n0, int n1, int n2, int ax, const Filter& f) {
  const int n = ax == 0 ? n0 : (ax == 1 ? n1 : n2), o = n >> 1;
  const int inner = ax == 0 ? n1 * n2 : (ax == 1 ? n2 : 1), outer = ax == 0 ? 1 : (ax == 1 ? n0 : n0 * n1);
  const bool v4 = ((src | dst) & 3) == 0;
  if (n < L) return coarse_analysis_w<L, true, NT>(sm, src, dst, n0, n1, n2, ax, f);
  if (ax == 2) {
    if (v4 && o % 4 == 0)
      return coarse_chunks<D, NT>(o, outer, [&](int ch, int lg) { coarse_rows_down<L, NT>(sm, src, dst, outer, n, ch, lg, f); });
  } else if (v4 && inner % 4 == 0 && ceil_log2(inner / 4) <= ceil_log2(NT)) {
    return coarse_cols_down<L, NT>(sm, src, dst, outer, n, inner, f);
  } else if (NT <= 512 && o % 4 == 0) {
    return coarse_cols_down_1<L, NT>(sm, src, dst, outer, n, inner, f);
  }
  coarse_analysis_w<L, false, NT>(sm, src, dst, n0, n1, n2, ax, f);
}
// gout: the block's final place in global memory, taken only where *direct says so
template <int D, int L, int NT>
DEVI void coarse_synthesis(float* sm, int src, int dst, int n0, int n1, int n2, int ax, const Filter& f, bool combine,
                           float alpha, float* gout = nullptr, bool* direct = nullptr) {
  const int n = ax == 0 ? n0 : (ax == 1 ? n1 : n2), half = n >> 1;
  const int inner = ax == 0 ? n1 * n2 : (ax == 1 ? n2 : 1), outer = ax == 0 ? 1 : (ax == 1 ? n0 : n0 * n1);
  const bool v4 = ((src | dst) & 3) == 0;
  if (half < L / 2) return coarse_synthesis_w<L, true, NT>(sm, src, dst, n0, n1, n2, ax, f, combine, alpha);
  if (ax == 2) {
    if (v4 && half % 4 == 0)
      return coarse_chunks<D, NT>(half, outer, [&](int ch, int lg) {
        coarse_rows_up<L, NT>(sm, src, dst, outer, n, ch, lg, f, combine, alpha);
      });
  } else if (v4 && inner % 4 == 0 && ceil_log2(inner / 4) <= ceil_log2(NT)) {
    if (direct) *direct = true;
    return coarse_cols_up<L, NT>(sm, src, dst, outer, n, inner, f, combine, alpha, gout);
  }
  coarse_synthesis_w<L, false, NT>(sm, src, dst, n0, n1, n2, ax, f, combine, alpha);
}

// ---------------------------------------------------------------------------------------
// The coarsest levels as matrix products.  A pass of a level of at most 32 x 32 samples is latency
// (~900 cycles for a handful of sums), and such a block has up to ten of them; but its whole remaining
// operator is a sum of separable projections,
//   z = c_0 a + sum_i c_i (U_i U_i^T) a (V_i V_i^T),
// with U_i^T, V_i^T the i-level low-pass analysis of the two axes (rows: the i-fold composite filter,
// folded to the axis length, shifted by 2^i).  With the rows of every level stacked into T1 (s1 x n1)
// and T2 (s2 x n2), s = sum_i n / 2^i < n <= 32, that is four products of at most 32 x 32 x 32 on the matrix
// cores, one 16 x 16 tile per wave:
//   P = T1 a,  M = (P T2^T) on the blocks of equal level, times c_i,  Q = M T2,  z = c_0 a + T1^T Q.
// FP32 products and sums throughout.  Where an infinity or a NaN met the zeros of the tables, it would reach
// every output of the block.  So a block that holds one, or a value so large that a product or sum
// could overflow (dense_scale), goes through the passes instead, which keep it to the outputs that depend on
// it.
// Scratch of the dense levels: P (then Q) and M over the passes' temporaries, then T1, T2 and tables.  Rows
// of kDenseRow floats: the 16 rows x 4 columns that a wave reads of a left factor hit distinct banks.
struct DenseLds {
  int P, M, T1, T2, lev1, lev2, coef, bad;
};
DEVI DenseLds dense_lds(int tmp, int tmp_floats, int n1, int n2) {
  DenseLds d;
  d.P = tmp;
  d.M = tmp + kDenseBuf;
  d.T1 = tmp + max(tmp_floats, 2 * kDenseBuf);
  d.T2 = n1 == n2 ? d.T1 : d.T1 + kDenseBuf;
  d.lev1 = d.T1 + 2 * kDenseBuf;
  d.lev2 = n1 == n2 ? d.lev1 : d.lev1 + kDenseSide;
  d.coef = d.lev1 + 2 * kDenseSide;
  d.bad = d.coef + kDenseLevels + 1;
  return d;
}

// T1, T2 (one array for a square block; zero outside s x n), the rows' levels (0: no row) and the
// coefficients c_0 .. c_K of the K <= kDenseLevels levels below the (n1, n2) block; no barrier.  Row r of an axis of
// length n is row n / 2^(i-1) - (n - r) of its level i.
template <int L, int NT>
DEVI void dense_tables(float* sm, const DenseLds& d, const TailTask* tp, int j0, int n1, int n2, int K) {
  constexpr int N = kDenseSide * kDenseSide;
  const int axes = n1 == n2 ? 1 : 2;
  for (int e = threadIdx.x; e < axes * N; e += NT) {
    const int ax = e / N, r = e / kDenseSide % kDenseSide, j = e % kDenseSide;
    const int n = ax ? n2 : n1, u = n - r;
    const int lev = dense_level(n, r);
    const bool row = u > 0 && lev <= K;
    const int i = j - (((n >> (lev - 1)) - u) << lev);
    const int at = row && j < n ? (n / 2 * kDenseLevels + lev - 1) * kDenseSide + (i < 0 ? i + n : i) : 0;
    const float v = gld(&kComposite<L>.c[0][0][0] + at);
    sm[(ax ? d.T2 : d.T1) + r * kDenseRow + j] = row && j < n ? v : 0.f;
    if (j == 0) reinterpret_cast<int*>(sm)[(ax ? d.lev2 : d.lev1) + r] = row ? lev : 0;
  }
  if (threadIdx.x <= (unsigned)K) sm[d.coef + threadIdx.x] = tp->coef[j0 + threadIdx.x];
  if (threadIdx.x == 0) reinterpret_cast<int*>(sm)[d.bad] = 0;
}

// Operands and product of a wave's 16 x 16 tile: lane l supplies A(l % 16, 4 s + l / 16) and B(4 s + l / 16,
// l % 16) of step s, and gets rows 4 (l / 16) + 0 .. 3 of column l % 16.  The inner index runs to `len`
// rounded up to 16; two chains of products, since one waits for its own sums.
typedef float mfma_f4 __attribute__((ext_vector_type(4)));
constexpr int kDenseSteps = kDenseSide / 4;
struct DenseOp {
  float x[kDenseSteps];
};
DEVI DenseOp dense_get(const float* p, int step) {  // p: the lane's element of step 0
  DenseOp r;
#pragma unroll
  for (int s = 0; s < kDenseSteps; ++s) r.x[s] = p[s * step];
  return r;
}
DEVI mfma_f4 dense_mul(const DenseOp& a, const DenseOp& b, int len) {
  mfma_f4 u = {0.f, 0.f, 0.f, 0.f}, v = u;
#pragma unroll
  for (int s = 0; s < kDenseSteps / 2; s += 2) {
    u = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s], b.x[s], u, 0, 0, 0);
    v = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s + 1], b.x[s + 1], v, 0, 0, 0);
  }
  if (len > 16) {
#pragma unroll
    for (int s = kDenseSteps / 2; s < kDenseSteps; s += 2) {
      u = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s], b.x[s], u, 0, 0, 0);
      v = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s + 1], b.x[s + 1], v, 0, 0, 0);
    }
  }
  return u + v;
}

// z over a in place for the (n1, n2) block at sm[ao], K levels below it.  Returns false, with a unchanged,
// where a holds a value that is not finite or overflows times `scale`.  Ends with a barrier.  T1 and T2 are zero past s x n, a is
// masked, and P, M and Q are written as whole tiles up to the inner lengths.  What a product takes from
// the tables and from a is read before the barrier that its other factor waits for.
template <int NT>
DEVI bool coarse_dense(float* sm, const DenseLds& d, int ao, int n1, int n2, int K, float scale) {
  constexpr int S = kDenseRow;
  const int s1 = n1 - (n1 >> K), s2 = n2 - (n2 >> K);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int lo = lane & 15, hi = lane >> 4;
  const int r0 = 16 * (wave >> 1), c0 = 16 * (wave & 1);  // tile of waves 0 .. 3
  int* words = reinterpret_cast<int*>(sm);
  static_assert(NT >= 256, "a tile per wave");
  const bool mine = wave < 4;
  const bool tP = mine && r0 < s1 && c0 < n2, tM = mine && r0 < s1 && c0 < s2, tZ = mine && r0 < n1 && c0 < n2;
  const int col = c0 + lo, row = r0 + 4 * hi;  // this lane's column, its four rows of a product
  float* const tile = sm + row * S + col;      // and its place in an array of kDenseRow floats a row
  DenseOp t;                                   // the next product's table factor
  int lr[4], lc = 0;
  float w = 0.f, x[4];
  // P = T1 a (reads past the block stay inside the LDS array, which holds more than 32 rows behind it)
  if (tP) {
    DenseOp av = dense_get(sm + ao + hi * n2 + col, 4 * n2);
    const int rows = (col < n2 ? n1 : 0) - hi;
    float zero = 0.f;  // NaN once a value is not finite or too large
#pragma unroll
    for (int s = 0; s < kDenseSteps; ++s) {
      av.x[s] = 4 * s < rows ? av.x[s] : 0.f;
      zero = fmaf(av.x[s] * scale, 0.f, zero);
    }
    const mfma_f4 v = dense_mul(dense_get(sm + d.T1 + (r0 + lo) * S + hi, 4), av, n1);
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[d.P + q * S] = v[q];
    if (__any(zero != 0.f) && lane == 0) words[d.bad] = 1;
  }
  if (tM) {
    t = dense_get(sm + d.T2 + col * S + hi, 4);
    lc = words[d.lev2 + col];
    w = sm[d.coef + lc];
#pragma unroll
    for (int q = 0; q < 4; ++q) lr[q] = words[d.lev1 + row + q];
  }
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(words[d.bad])) return false;
  // M = P T2^T on the blocks of equal level, weighted
  if (tM) {
    const mfma_f4 v = dense_mul(dense_get(sm + d.P + (r0 + lo) * S + hi, 4), t, n2);
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[d.M + q * S] = lr[q] == lc && lc > 0 ? w * v[q] : 0.f;
  }
  if (tP) t = dense_get(sm + d.T2 + hi * S + col, 4 * S);
  __syncthreads();
  // Q = M T2 (over P)
  if (tP) {
    const mfma_f4 v = dense_mul(dense_get(sm + d.M + (r0 + lo) * S + hi, 4), t, s2);
#pragma unroll
    for (int q = 0; q < 4; ++q) tile[d.P + q * S] = v[q];
  }
  float* const z = sm + ao + row * n2 + col;
  if (tZ) {
    t = dense_get(sm + d.T1 + hi * S + r0 + lo, 4 * S);
    w = sm[d.coef];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = z[q * n2];
  }
  __syncthreads();
  // z = c_0 a + T1^T Q
  if (tZ) {
    const mfma_f4 v = dense_mul(t, dense_get(sm + d.P + hi * S + col, 4 * S), s1);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (row + q < n1 && col < n2) z[q * n2] = fmaf(w, x[q], v[q]);
  }
  __syncthreads();
  return true;
}

// Every coarse level of instance `inst` of tail task `tp` in one work-group of NT threads; `sm`
// holds coarse_lds_floats(D, CMAX) floats of LDS (16-byte aligned).
template <int D, int L, int CMAX, int NT>
DEVI void lp_coarse_block(const TailTask* tp, int inst, const Filter& f, float* sm) {
  const float* in = tp->in + inst * tp->bs_in;
  float* out = tp->out + inst * tp->bs_out;
  const int K = tp->nlev;
  const int m0 = tp->b[0], m1 = tp->b[1], m2 = tp->b[2];
  const int B = m0 * m1 * m2;
  // offsets of A_0 .. A_K, then the temporaries
  int tmpA = 0;
  for (int j = 0; j <= K; ++j) tmpA += B >> (D * j);
  const int tmpB = tmpA + (B >> 1);
  // levels from Kd on (2-D, at most 32 x 32 samples) as matrix products
  int Kd = D == 2 && tp->dense >= 0 ? tp->dense : K;
  const DenseLds dl = dense_lds(tmpA, B >> 1, m1 >> Kd, m2 >> Kd);
  block_to_lds<NT, CMAX>(in, sm, B, [&] {
    if (D == 2 && Kd < K) dense_tables<L, NT>(sm, dl, tp, Kd, m1 >> Kd, m2 >> Kd, K - Kd);
  });
  __syncthreads();
  int off = 0;
  for (int j = 0;; ++j) {
    if (D == 2 && j == Kd && Kd < K) {
      if (coarse_dense<NT>(sm, dl, off, m1 >> j, m2 >> j, K - j, tp->dense_scale)) break;
      Kd = K;
    }
    if (j == K) break;
    const int a0 = D >= 3 ? m0 >> j : 1, a1 = D >= 2 ? m1 >> j : 1, a2 = m2 >> j;
    const int nxt = off + a0 * a1 * a2;
    if (D == 1) {
      coarse_analysis<D, L, NT>(sm, off, nxt, a0, a1, a2, 2, f);
    } else if (D == 2) {
      coarse_analysis<D, L, NT>(sm, off, tmpA, a0, a1, a2, 2, f);
      __syncthreads();
      coarse_analysis<D, L, NT>(sm, tmpA, nxt, a0, a1, a2 >> 1, 1, f);
    } else {
      coarse_analysis<D, L, NT>(sm, off, tmpA, a0, a1, a2, 2, f);
      __syncthreads();
      coarse_analysis<D, L, NT>(sm, tmpA, tmpB, a0, a1, a2 >> 1, 1, f);
      __syncthreads();
      coarse_analysis<D, L, NT>(sm, tmpB, nxt, a0, a1 >> 1, a2 >> 1, 0, f);
    }
    __syncthreads();
    off = nxt;
  }
  if (Kd == K) {
    const int sz = B >> (D * K);
    const float ck = tp->coef[K];
    for (int e = threadIdx.x; e < sz; e += NT) sm[off + e] *= ck;
    __syncthreads();
  }
  // the last synthesis pass (j = 0) writes the result to global memory itself where it can
  bool stored = false;
  float* const gout = (((uintptr_t)out) & 15) == 0 ? out : nullptr;
  for (int j = Kd - 1; j >= 0; --j) {
    float* const g = j == 0 ? gout : nullptr;
    bool* const d = g ? &stored : nullptr;
    const int a0 = D >= 3 ? m0 >> j : 1, a1 = D >= 2 ? m1 >> j : 1, a2 = m2 >> j;  // output block
    const int cur = off - a0 * a1 * a2;  // A_j precedes A_{j+1}
    const float alpha = tp->coef[j];
    if (D == 1) {
      coarse_synthesis<D, L, NT>(sm, off, cur, a0, a1, a2, 2, f, true, alpha);
    } else if (D == 2) {
      // contiguous axis first: (a1/2, a2/2) -> (a1/2, a2) in tmpA, then rows -> A_j
      coarse_synthesis<D, L, NT>(sm, off, tmpA, a0, a1 >> 1, a2, 2, f, false, 0.f);
      __syncthreads();
      coarse_synthesis<D, L, NT>(sm, tmpA, cur, a0, a1, a2, 1, f, true, alpha, g, d);
    } else {
      coarse_synthesis<D, L, NT>(sm, off, tmpA, a0 >> 1, a1 >> 1, a2, 2, f, false, 0.f);
      __syncthreads();
      coarse_synthesis<D, L, NT>(sm, tmpA, tmpB, a0 >> 1, a1, a2, 1, f, false, 0.f);
      __syncthreads();
      coarse_synthesis<D, L, NT>(sm, tmpB, cur, a0, a1, a2, 0, f, true, alpha, g, d);
    }
    __syncthreads();
    off = cur;
  }
  if (!stored) block_from_lds<NT>(sm, out, B);
}

}  // namespace es
