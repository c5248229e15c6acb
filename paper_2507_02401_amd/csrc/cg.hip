// Matrix-free Tikhonov / MAP solver around the wavelet prior: preconditioned conjugate gradients
// on the normal equations of J(x) = 1/2 ||M x - p||^2 + alpha/2 ||x||^2_{H^s} (Sec. 3: the
// Tikhonov functional and the linear equation of its minimiser; Sec. 4: the wavelet form of the
// Sobolev operators and the remark that iterative solvers such as conjugate gradients apply to
// it), i.e.
//     (M + alpha Gamma^2) x = M p,   Gamma^2 = W^T D_{-2s} W,   M = diag(mask),
// preconditioned with W^T D_{2s} W (the covariance: the inverse of the penalty term up to the
// factor 1/alpha, which CG's iterates do not depend on).
//
// Every step runs on the device: the two operator applications per iteration are the library's
// matern_cov_apply (smoothness -s and +s), the vector updates are fused element-wise kernels
// that also produce per-work-group partial inner products; the next launch's work-groups each sum
// those partials in one fixed order and form the instance's CG scalars.  All sums are
// FP32 with compensation (Neumaier) per thread and pairwise trees across threads; results are
// deterministic.  The host looks at the residuals only every `check_every` iterations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "../../include/eswave.h"
#include "internal.h"
#include "kcommon.h"

namespace es {
namespace {

constexpr int kCgThreads = 256;
// Elements of one instance per work-group of the element-wise kernels.  Instances of up to 2^19
// elements take one 16-byte access per thread: a single 512^2 image then fills the 256 CUs (64
// work-groups of 4096 left three quarters idle).  Larger ones fill the chip with either and keep
// fewer partial sums.  The rule looks at the instance only, so an instance's sums do not depend on
// the batch.
constexpr int kCgChunkSmall = 1024, kCgChunkLarge = 4096;
inline __host__ __device__ int cg_chunk(int64_t n) { return n <= (int64_t)1 << 19 ? kCgChunkSmall : kCgChunkLarge; }

// Per-instance CG scalars (device).  Two copies: an iteration reads one and writes the next
// iteration's, so that every work-group of a launch may read them.
struct CgScal {
  float bn;      // ||b||
  float rz;      // r . z
  float a;       // step length of this iteration (0 once converged)
  float rel;     // ||r|| / ||b||
  float active;  // 1 while rel > rtol at the start of the iteration
  float pad_[3];
};

// Partials of a sum over an instance, `n` of them from p[inst * n] on.
struct Partials {
  const float* p;
  int32_t n;
};

// Partials are summed by the kernel that needs the sum where an instance has at most this many
// (every work-group of the instance repeats the short sum, four loads a thread; a launch of its own
// costs ~4 us), by k_cg_reduce first otherwise.
constexpr int kCgMaxParts = 1024;

// Sum of one value per thread over the work-group, pairwise (fixed order); thread 0 gets it.
DEVI float wg_sum(float v) {
  __shared__ float part[kCgThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) part[w] = v;
  __syncthreads();
  float t = 0.f;
  if (threadIdx.x == 0) t = (part[0] + part[1]) + (part[2] + part[3]);
  __syncthreads();
  return t;
}

// Sums of two values per thread over the work-group, pairwise (fixed order); thread 0 gets them.
DEVI float2 wg_sum2(float v, float u) {
  __shared__ float2 part2[kCgThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v += __shfl_down(v, o, 64);
    u += __shfl_down(u, o, 64);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) part2[w] = make_float2(v, u);
  __syncthreads();
  float2 t = make_float2(0.f, 0.f);
  if (threadIdx.x == 0)
    t = make_float2((part2[0].x + part2[1].x) + (part2[2].x + part2[3].x),
                    (part2[0].y + part2[1].y) + (part2[2].y + part2[3].y));
  __syncthreads();
  return t;
}

// Work-group -> (instance, chunk) of the element-wise kernels.
struct Span {
  int64_t inst, lo, hi;  // elements [lo, hi) of instance inst
};
DEVI Span span_of(int64_t n, int per) {
  Span sp;
  sp.inst = blockIdx.x / per;
  sp.lo = (int64_t)(blockIdx.x % per) * cg_chunk(n);
  sp.hi = min(n, sp.lo + cg_chunk(n));
  return sp;
}

// Element-wise loop over one chunk; vectors of four where the instance size allows.
template <class F>
DEVI void for_chunk(const Span& sp, int64_t n, F f) {
  const int64_t base = sp.inst * n;
  if ((n & 3) == 0) {
    for (int64_t i = sp.lo + 4 * threadIdx.x; i < sp.hi; i += 4 * kCgThreads) f(base + i, 4);
  } else {
    for (int64_t i = sp.lo + threadIdx.x; i < sp.hi; i += kCgThreads) f(base + i, 1);
  }
}

// r = mask * p, x = 0; partial r . r
__global__ void __launch_bounds__(kCgThreads) k_cg_init(int64_t n, int per, const float* __restrict__ p,
                                                        const float* __restrict__ mask, float* __restrict__ x,
                                                        float* __restrict__ r, float* __restrict__ part) {
  const Span sp = span_of(n, per);
  KSum acc;
  for_chunk(sp, n, [&](int64_t i, int w) {
    for (int k = 0; k < w; ++k) {
      const float v = gld(mask + i + k) * gld(p + i + k);
      gst(r + i + k, v);
      gst(x + i + k, 0.f);
      acc.add(v * v);
    }
  });
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

// partial a . b (and, when dst is given, dst = b: the first direction d = z)
__global__ void __launch_bounds__(kCgThreads) k_cg_dot(int64_t n, int per, const float* __restrict__ a,
                                                       const float* __restrict__ b, float* __restrict__ dst,
                                                       float* __restrict__ part) {
  const Span sp = span_of(n, per);
  KSum acc;
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {
      const float4 u = gld4(a + i), v = gld4(b + i);
      if (dst) gst4(dst + i, v);
      acc.add(u.x * v.x);
      acc.add(u.y * v.y);
      acc.add(u.z * v.z);
      acc.add(u.w * v.w);
    } else {
      const float v = gld(b + i);
      if (dst) gst(dst + i, v);
      acc.add(gld(a + i) * v);
    }
  });
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

// ad = alpha * ad + mask * d (ad holds W^T D_{-2s} W d on entry); partial d . ad
__global__ void __launch_bounds__(kCgThreads) k_cg_apply(int64_t n, int per, float alpha, const float* __restrict__ mask,
                                                         const float* __restrict__ d, float* __restrict__ ad,
                                                         float* __restrict__ part) {
  const Span sp = span_of(n, per);
  KSum acc;
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {
      const float4 m = gld4(mask + i), dv = gld4(d + i), g = gld4(ad + i);
      const float4 o = make_float4(fmaf(m.x, dv.x, alpha * g.x), fmaf(m.y, dv.y, alpha * g.y),
                                   fmaf(m.z, dv.z, alpha * g.z), fmaf(m.w, dv.w, alpha * g.w));
      gst4(ad + i, o);
      acc.add(dv.x * o.x);
      acc.add(dv.y * o.y);
      acc.add(dv.z * o.z);
      acc.add(dv.w * o.w);
    } else {
      const float dv = gld(d + i);
      const float o = fmaf(gld(mask + i), dv, alpha * gld(ad + i));
      gst(ad + i, o);
      acc.add(dv * o);
    }
  });
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

DEVI KSum thread_sum(const Partials& q, int64_t inst) {
  KSum acc;
  for (int k = threadIdx.x; k < q.n; k += kCgThreads) acc.add(q.p[inst * q.n + k]);
  return acc;
}

// dst[inst] = sum of the instance's partials, in a fixed order
__global__ void __launch_bounds__(kCgThreads) k_cg_reduce(Partials q, float* __restrict__ dst) {
  const float sum = wg_sum(thread_sum(q, blockIdx.x).value());
  if (threadIdx.x == 0) dst[blockIdx.x] = sum;
}

// First scalars of every instance: rr = ||b||^2, rz = r . z
__global__ void __launch_bounds__(kCgThreads) k_cg_start(Partials rr, Partials rz, CgScal* __restrict__ sc, float rtol) {
  const int64_t inst = blockIdx.x;
  const float2 sum = wg_sum2(thread_sum(rr, inst).value(), thread_sum(rz, inst).value());
  if (threadIdx.x != 0) return;
  CgScal c{};
  c.bn = sqrtf(sum.x);
  c.rz = sum.y;
  c.rel = c.bn > 0.f ? 1.f : 0.f;
  c.active = c.rel > rtol ? 1.f : 0.f;
  sc[inst] = c;
}

// a = r.z / d.ad (dad: the partials of d . ad; kept in sc for the direction pass); r -= a ad; partial
// r . r  (x += a d waits for the direction pass, which reads d anyway)
__global__ void __launch_bounds__(kCgThreads) k_cg_step(int64_t n, int per, Partials dad, CgScal* __restrict__ sc,
                                                        float* __restrict__ r, const float* __restrict__ ad,
                                                        float* __restrict__ part) {
  __shared__ float step;
  const Span sp = span_of(n, per);
  const float sum = wg_sum(thread_sum(dad, sp.inst).value());
  if (threadIdx.x == 0) {
    const float rz = sc[sp.inst].rz, act = sc[sp.inst].active;
    step = (act != 0.f && sum > 0.f) ? rz / sum : 0.f;
    if (sp.lo == 0) sc[sp.inst].a = step;
  }
  __syncthreads();
  const float a = step;
  KSum acc;
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {
      const float4 rv = gld4(r + i), g = gld4(ad + i);
      const float4 rn = make_float4(fmaf(-a, g.x, rv.x), fmaf(-a, g.y, rv.y), fmaf(-a, g.z, rv.z), fmaf(-a, g.w, rv.w));
      gst4(r + i, rn);
      acc.add(rn.x * rn.x);
      acc.add(rn.y * rn.y);
      acc.add(rn.z * rn.z);
      acc.add(rn.w * rn.w);
    } else {
      const float rn = fmaf(-a, gld(ad + i), gld(r + i));
      gst(r + i, rn);
      acc.add(rn * rn);
    }
  });
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

// beta = r.z / (r.z of the iteration's start); x += a d (this iteration's step), then d = beta d + z;
// and the next iteration's scalars (rr, rz: the partials of r . r and r . z of the new residual)
__global__ void __launch_bounds__(kCgThreads) k_cg_dir(int64_t n, int per, Partials rr, Partials rz,
                                                       const CgScal* __restrict__ sc, CgScal* __restrict__ next, float rtol,
                                                       float* __restrict__ x, float* __restrict__ d,
                                                       const float* __restrict__ z) {
  __shared__ float2 ab;
  const Span sp = span_of(n, per);
  const float2 sum = wg_sum2(thread_sum(rr, sp.inst).value(), thread_sum(rz, sp.inst).value());
  if (threadIdx.x == 0) {
    CgScal c = sc[sp.inst];
    ab = make_float2(c.a, (c.active != 0.f && c.rz > 0.f) ? sum.y / c.rz : 0.f);
    if (sp.lo == 0) {
      c.rel = c.bn > 0.f ? sqrtf(sum.x) / c.bn : 0.f;
      c.rz = sum.y;
      c.active = c.rel > rtol ? c.active : 0.f;  // converged instances stay frozen
      next[sp.inst] = c;
    }
  }
  __syncthreads();
  const float a = ab.x, beta = ab.y;
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {
      const float4 xv = gld4(x + i), dv = gld4(d + i), zv = gld4(z + i);
      gst4(x + i, make_float4(fmaf(a, dv.x, xv.x), fmaf(a, dv.y, xv.y), fmaf(a, dv.z, xv.z), fmaf(a, dv.w, xv.w)));
      gst4(d + i, make_float4(fmaf(beta, dv.x, zv.x), fmaf(beta, dv.y, zv.y), fmaf(beta, dv.z, zv.z),
                              fmaf(beta, dv.w, zv.w)));
    } else {
      const float dv = gld(d + i);
      gst(x + i, fmaf(a, dv, gld(x + i)));
      gst(d + i, fmaf(beta, dv, gld(z + i)));
    }
  });
}

// ---- GMRES on (E_s^* K^* K + alpha I) x = E_s^* K^* p (K = diag(mask)) ----------------------
constexpr int kGmMaxBasis = 64;  // largest restart length
// Vectors of the basis are batch * n floats, `vs` floats apart.  Per-instance coefficients
// (inner products, norms, least-squares solutions) are device arrays indexed inst * ld + j.

// out = (sq ? m * m : m) * v
__global__ void __launch_bounds__(kCgThreads) k_gm_mask(int64_t n, int per, int sq, const float* __restrict__ mask,
                                                        const float* __restrict__ v, float* __restrict__ out) {
  const Span sp = span_of(n, per);
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {
      float4 m = gld4(mask + i);
      const float4 x = gld4(v + i);
      if (sq) m = make_float4(m.x * m.x, m.y * m.y, m.z * m.z, m.w * m.w);
      gst4(out + i, make_float4(m.x * x.x, m.y * x.y, m.z * x.z, m.w * x.w));
    } else {
      const float m = gld(mask + i);
      gst(out + i, (sq ? m * m : m) * gld(v + i));
    }
  });
}

// out = a x + b y + c z (a null vector contributes nothing); partial ||out||^2 when part is given.
// out may be one of x, y, z (each element is read, then written, by the same thread).
__global__ void __launch_bounds__(kCgThreads) k_gm_lin3(int64_t n, int per, float a, const float* x, float b,
                                                        const float* y, float c, const float* z, float* out,
                                                        float* __restrict__ part) {
  const Span sp = span_of(n, per);
  KSum acc;
  auto l4 = [](const float* q, int64_t i) { return q ? gld4(q + i) : make_float4(0.f, 0.f, 0.f, 0.f); };
  for_chunk(sp, n, [&](int64_t i, int w) {
    if (w == 4) {  // every vector's three loads issued before the arithmetic
      const float4 xv = l4(x, i), yv = l4(y, i), zv = l4(z, i);
      const float4 o = make_float4(fmaf(c, zv.x, fmaf(b, yv.x, a * xv.x)), fmaf(c, zv.y, fmaf(b, yv.y, a * xv.y)),
                                   fmaf(c, zv.z, fmaf(b, yv.z, a * xv.z)), fmaf(c, zv.w, fmaf(b, yv.w, a * xv.w)));
      gst4(out + i, o);
      acc.add(o.x * o.x);
      acc.add(o.y * o.y);
      acc.add(o.z * o.z);
      acc.add(o.w * o.w);
    } else {
      const float o = fmaf(c, z ? gld(z + i) : 0.f, fmaf(b, y ? gld(y + i) : 0.f, x ? a * gld(x + i) : 0.f));
      gst(out + i, o);
      acc.add(o * o);
    }
  });
  if (part) {
    const float t = wg_sum(acc.value());
    if (threadIdx.x == 0) gst(part + blockIdx.x, t);
  } else {
    (void)acc;
  }
}

// w += alpha v_{nv-1} (the operator's shift: w holds E_s^*(mask^2 v) on entry), then over this
// work-group's chunk, for j < nv: part[j * nblk + blk] = <v_j, w> and part[(nv + j) * nblk + blk] =
// <v_j, u> (u = v_{nv-1}, the newest basis vector: the new column of the basis's Gram matrix).  The
// chunks of w and u are read once, into registers (PER elements per thread, 16-byte loads when the
// instance size is a multiple of 4), and the next basis vector is in flight while one is summed; each
// product is summed within the wave per basis vector and across the four waves, in a fixed order,
// once at the end.  Memory-bound on large instances (the shift in a kernel of its own read and wrote
// w once more and read v), latency-bound on small ones.
template <int PER>
__global__ void __launch_bounds__(kCgThreads) k_gm_dots(int64_t n, int per, int nv, const float* __restrict__ V,
                                                        int64_t vs, float alpha, float* __restrict__ w,
                                                        float* __restrict__ part) {
  __shared__ float2 wp[kCgThreads / 64][kGmMaxBasis + 1];
  const Span sp = span_of(n, per);
  const int64_t base = sp.inst * n;
  const float* u = V + (int64_t)(nv - 1) * vs + base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto wave_store = [&](int j, KSum& aw, KSum& au) {
    float x = aw.value(), y = au.value();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      x += __shfl_down(x, o, 64);
      y += __shfl_down(y, o, 64);
    }
    if (lane == 0) wp[wave][j] = make_float2(x, y);
  };
  if ((n & 3) == 0) {
    constexpr int G = PER / 4;  // float4 groups per thread
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const int64_t i0 = sp.lo + 4 * threadIdx.x;
    auto load = [&](const float* v, float4* x) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int64_t i = i0 + (int64_t)g * 4 * kCgThreads;
        x[g] = i < sp.hi ? gld4(v + i) : zero;
      }
    };
    float4 wv[G], uv[G], xv[G], nx[G];
    load(w + base, wv);
    load(u, uv);
    load(V + base, nx);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      wv[g] = make_float4(fmaf(alpha, uv[g].x, wv[g].x), fmaf(alpha, uv[g].y, wv[g].y), fmaf(alpha, uv[g].z, wv[g].z),
                          fmaf(alpha, uv[g].w, wv[g].w));
      const int64_t i = i0 + (int64_t)g * 4 * kCgThreads;
      if (i < sp.hi) gst4(w + base + i, wv[g]);
    }
    for (int j = 0; j < nv; ++j) {
#pragma unroll
      for (int g = 0; g < G; ++g) xv[g] = nx[g];
      if (j + 1 < nv) load(V + (int64_t)(j + 1) * vs + base, nx);
      KSum aw, au;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        aw.add(xv[g].x * wv[g].x);
        aw.add(xv[g].y * wv[g].y);
        aw.add(xv[g].z * wv[g].z);
        aw.add(xv[g].w * wv[g].w);
        au.add(xv[g].x * uv[g].x);
        au.add(xv[g].y * uv[g].y);
        au.add(xv[g].z * uv[g].z);
        au.add(xv[g].w * uv[g].w);
      }
      wave_store(j, aw, au);
    }
  } else {
    float wv[PER], uv[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int64_t i = sp.lo + threadIdx.x + (int64_t)k * kCgThreads;
      uv[k] = i < sp.hi ? gld(u + i) : 0.f;
      wv[k] = i < sp.hi ? fmaf(alpha, uv[k], gld(w + base + i)) : 0.f;
      if (i < sp.hi) gst(w + base + i, wv[k]);
    }
    for (int j = 0; j < nv; ++j) {
      const float* v = V + j * vs + base;
      KSum aw, au;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int64_t i = sp.lo + threadIdx.x + (int64_t)k * kCgThreads;
        if (i < sp.hi) {
          const float x = gld(v + i);
          aw.add(x * wv[k]);
          au.add(x * uv[k]);
        }
      }
      wave_store(j, aw, au);
    }
  }
  __syncthreads();
  const int nblk = gridDim.x;
  for (int q = threadIdx.x; q < 2 * nv; q += kCgThreads) {
    const int j = q >> 1;
    const bool second = q & 1;
    auto pick = [&](int wv_) { return second ? wp[wv_][j].y : wp[wv_][j].x; };
    const float t = (pick(0) + pick(1)) + (pick(2) + pick(3));
    gst(part + (int64_t)(second ? nv + j : j) * nblk + blockIdx.x, t);
  }
}

// Partials are reduced by the kernel that needs the sums where an instance has at most this many
// (every work-group of the instance repeats the short sum; a launch of its own costs ~4 us), by
// k_gm_final otherwise.
constexpr int kGmMaxParts = 256;

// dst[j * batch + inst] = sum of instance inst's `per` partials of vector j, in a fixed order;
// grid (batch, vectors)
__global__ void __launch_bounds__(kCgThreads) k_gm_final(int per, int nblk, const float* __restrict__ part,
                                                         float* __restrict__ dst) {
  const int inst = blockIdx.x, j = blockIdx.y;
  KSum acc;
  for (int k = threadIdx.x; k < per; k += kCgThreads) acc.add(part[(int64_t)j * nblk + (int64_t)inst * per + k]);
  const float sum = wg_sum(acc.value());
  if (threadIdx.x == 0) dst[(int64_t)j * gridDim.x + inst] = sum;
}

// Coefficients of step k (one work-group per instance): the sums of the 2 (k + 1) inner products (one
// wave per vector), the new Gram column G[j][k] = G[k][j] = <v_j, v_k> into the instance's
// (m+1) x (m+1) Gram matrix, and c = 2 h - G h (j, i <= k) with h = V^T w: the two classical
// Gram-Schmidt passes of CGS2, the second written through the Gram matrix (exact when the first
// subtraction is).  A wave per inner product of a step of eight vectors; fewer waves, which take the same sums
// in turn, where a launch of so many instances would hold 2^32 threads.
constexpr int kGmCoefThreads = 1024, kGmCoefThreadsMany = 128;
__global__ void __launch_bounds__(kGmCoefThreads) k_gm_coef(int k, int per, int nblk, const float* __restrict__ part,
                                                            float* __restrict__ G, int ldG, float* __restrict__ c, int ldc) {
  __shared__ float h[2 * (kGmMaxBasis + 1)];  // h[0..k], then the Gram column [k+1 .. 2k+1]
  const int inst = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int v = wave; v < 2 * (k + 1); v += (int)blockDim.x / 64) {
    const float* p = part + (int64_t)v * nblk + (int64_t)inst * per;
    KSum acc;
    for (int i = lane; i < per; i += 64) acc.add(p[i]);
    float x = acc.value();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    if (lane == 0) h[v] = x;
  }
  __syncthreads();
  float* Gi = G + (int64_t)inst * ldG * ldG;
  const int j = threadIdx.x;
  if (j <= k) {
    const float gj = h[k + 1 + j];
    Gi[j * ldG + k] = gj;
    Gi[k * ldG + j] = gj;
    float acc = 0.f;
    for (int i = 0; i < k; ++i) acc = fmaf(j == k ? h[k + 1 + i] : Gi[j * ldG + i], h[i], acc);
    acc = fmaf(gj, h[k], acc);
    c[(int64_t)inst * ldc + j] = 2.f * h[j] - acc;
  }
}

// w -= sum_j h[inst * ld + j] v_j (j < nv); partial ||w||^2
__global__ void __launch_bounds__(kCgThreads) k_gm_sub(int64_t n, int per, int nv, const float* __restrict__ V,
                                                       int64_t vs, const float* __restrict__ h, int ld,
                                                       float* __restrict__ w, float* __restrict__ part) {
  const Span sp = span_of(n, per);
  const int64_t base = sp.inst * n;
  __shared__ float hs[kGmMaxBasis + 1];
  for (int j = threadIdx.x; j < nv; j += kCgThreads) hs[j] = h[sp.inst * ld + j];
  __syncthreads();
  KSum acc;
  if ((n & 3) == 0) {
    for (int64_t i = sp.lo + 4 * threadIdx.x; i < sp.hi; i += 4 * kCgThreads) {
      float4 o = gld4(w + base + i);
      const float* v = V + base + i;
      int j = 0;
      constexpr int U = 4;  // basis vectors in flight
      for (; j + U <= nv; j += U) {
        float4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = gld4(v + (j + u) * vs);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float hj = -hs[j + u];
          o = make_float4(fmaf(hj, x[u].x, o.x), fmaf(hj, x[u].y, o.y), fmaf(hj, x[u].z, o.z), fmaf(hj, x[u].w, o.w));
        }
      }
      for (; j < nv; ++j) {
        const float4 x = gld4(v + j * vs);
        const float hj = -hs[j];
        o = make_float4(fmaf(hj, x.x, o.x), fmaf(hj, x.y, o.y), fmaf(hj, x.z, o.z), fmaf(hj, x.w, o.w));
      }
      gst4(w + base + i, o);
      acc.add(o.x * o.x);
      acc.add(o.y * o.y);
      acc.add(o.z * o.z);
      acc.add(o.w * o.w);
    }
  } else {
    for (int64_t i = sp.lo + threadIdx.x; i < sp.hi; i += kCgThreads) {
      float o = gld(w + base + i);
      for (int j = 0; j < nv; ++j) o = fmaf(-hs[j], gld(V + j * vs + base + i), o);
      gst(w + base + i, o);
      acc.add(o * o);
    }
  }
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

// x = 0; partial ||b||^2
__global__ void __launch_bounds__(kCgThreads) k_gm_begin(int64_t n, int per, const float* __restrict__ b,
                                                         float* __restrict__ x, float* __restrict__ part) {
  const Span sp = span_of(n, per);
  KSum acc;
  for_chunk(sp, n, [&](int64_t i, int wdt) {
    if (wdt == 4) {
      const float4 v = gld4(b + i);
      gst4(x + i, make_float4(0.f, 0.f, 0.f, 0.f));
      acc.add(v.x * v.x);
      acc.add(v.y * v.y);
      acc.add(v.z * v.z);
      acc.add(v.w * v.w);
    } else {
      const float v = gld(b + i);
      gst(x + i, 0.f);
      acc.add(v * v);
    }
  });
  const float t = wg_sum(acc.value());
  if (threadIdx.x == 0) gst(part + blockIdx.x, t);
}

// v = w / ||w||, or 0 when the norm is 0 (an exhausted or zero instance), ||w||^2 the sum of the
// instance's `nparts` partials, kept in nrm[inst * ld]; and t = mask^2 v (the next operator
// application's input)
__global__ void __launch_bounds__(kCgThreads) k_gm_scale(int64_t n, int per, int nparts, const float* __restrict__ part,
                                                         float* __restrict__ nrm, int ld, const float* __restrict__ w,
                                                         float* __restrict__ v, const float* __restrict__ mask,
                                                         float* __restrict__ t) {
  __shared__ float total;
  const Span sp = span_of(n, per);
  KSum acc;
  for (int k = threadIdx.x; k < nparts; k += kCgThreads) acc.add(part[sp.inst * nparts + k]);
  const float sum = wg_sum(acc.value());
  if (threadIdx.x == 0) {
    total = sum;
    if (sp.lo == 0) nrm[sp.inst * ld] = sum;
  }
  __syncthreads();
  const float q = total;
  const float sc = q > 0.f ? 1.f / sqrtf(q) : 0.f;
  for_chunk(sp, n, [&](int64_t i, int wdt) {
    if (wdt == 4) {
      const float4 x = gld4(w + i), m = gld4(mask + i);
      const float4 o = make_float4(sc * x.x, sc * x.y, sc * x.z, sc * x.w);
      gst4(v + i, o);
      gst4(t + i, make_float4(m.x * m.x * o.x, m.y * m.y * o.y, m.z * m.z * o.z, m.w * m.w * o.w));
    } else {
      const float o = sc * gld(w + i), m = gld(mask + i);
      gst(v + i, o);
      gst(t + i, m * m * o);
    }
  });
}

// x += sum_j y[inst * ld + j] v_j (j < nv)
__global__ void __launch_bounds__(kCgThreads) k_gm_combine(int64_t n, int per, int nv, const float* __restrict__ V,
                                                           int64_t vs, const float* __restrict__ y, int ld,
                                                           float* __restrict__ x) {
  const Span sp = span_of(n, per);
  const int64_t base = sp.inst * n;
  __shared__ float ys[kGmMaxBasis + 1];
  for (int j = threadIdx.x; j < nv; j += kCgThreads) ys[j] = y[sp.inst * ld + j];
  __syncthreads();
  if ((n & 3) == 0) {
    for (int64_t i = sp.lo + 4 * threadIdx.x; i < sp.hi; i += 4 * kCgThreads) {
      float4 o = gld4(x + base + i);
      for (int j = 0; j < nv; ++j) {
        const float4 v = gld4(V + j * vs + base + i);
        o = make_float4(fmaf(ys[j], v.x, o.x), fmaf(ys[j], v.y, o.y), fmaf(ys[j], v.z, o.z), fmaf(ys[j], v.w, o.w));
      }
      gst4(x + base + i, o);
    }
  } else {
    for (int64_t i = sp.lo + threadIdx.x; i < sp.hi; i += kCgThreads) {
      float o = gld(x + base + i);
      for (int j = 0; j < nv; ++j) o = fmaf(ys[j], gld(V + j * vs + base + i), o);
      gst(x + base + i, o);
    }
  }
}

int64_t cg_parts(int64_t n) { return (n + cg_chunk(n) - 1) / cg_chunk(n); }
size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

struct GmLayout {
  size_t V, b, w, t, part, hg, c, G, y, cov, total;
  int64_t vs;  // floats between basis vectors
};

GmLayout gm_layout(int64_t n, int64_t batch, int m, size_t cov_bytes, int64_t per) {
  GmLayout L;
  const size_t vec = a256((size_t)(n * batch) * sizeof(float));
  L.vs = (int64_t)(vec / sizeof(float));
  L.V = 0;
  L.b = L.V + vec * (size_t)(m + 1);
  L.w = L.b + vec;
  L.t = L.w + vec;
  L.part = L.t + vec;
  L.hg = L.part + a256((size_t)(2 * (m + 1) * per * batch) * sizeof(float));
  L.c = L.hg + a256((size_t)(batch * 2 * (m + 1)) * sizeof(float));
  L.G = L.c + a256((size_t)((m + 1) * batch * (m + 1)) * sizeof(float));
  L.y = L.G + a256((size_t)(batch * (m + 1) * (m + 1)) * sizeof(float));
  L.cov = L.y + a256((size_t)(batch * (m + 1)) * sizeof(float));
  L.total = L.cov + cov_bytes;
  return L;
}


struct CgLayout {
  size_t r, z, d, ad, part, prr, scal, cov, total;
};

CgLayout cg_layout(int64_t n, int64_t batch, size_t cov_bytes, int64_t parts) {
  CgLayout L;
  const size_t vec = a256((size_t)(n * batch) * sizeof(float));
  L.r = 0;
  L.z = L.r + vec;
  L.d = L.z + vec;
  L.ad = L.d + vec;
  L.part = L.ad + vec;
  L.prr = L.part + a256((size_t)((parts + 1) * batch) * sizeof(float));
  L.scal = L.prr + a256((size_t)((cg_parts(n) + 1) * batch) * sizeof(float));
  L.cov = L.scal + a256((size_t)batch * 2 * sizeof(CgScal));
  L.total = L.cov + cov_bytes;
  return L;
}

}  // namespace
}  // namespace es

using namespace es;

extern "C" {

size_t es_tikhonov_pcg_workspace_bytes(int ndim, const int64_t* shape, int64_t batch, int order, int levels) {
  if (batch < 1 || ndim < 1 || ndim > 3 || !shape) return 0;
  int64_t n = 1;
  for (int k = 0; k < ndim; ++k) n *= shape[k];
  const size_t cov = es_workspace_bytes(ndim, shape, batch, order, levels, ES_OP_COV);
  return cg_layout(n, batch, cov, std::max(cg_parts(n), cov_dot_partials_max(ndim, shape))).total;
}

es_status es_tikhonov_pcg(int ndim, const int64_t* shape, int64_t batch, int order, int levels, double s, double alpha,
                          const float* p, const float* mask, float* x, int32_t max_iter, double rtol,
                          int32_t check_every, int32_t* iterations, float* rel_residual, void* ws, size_t ws_bytes,
                          void* stream) {
  char msg[256];
  if (ndim < 1 || ndim > 3 || !shape) return report_error(ES_EINVAL, "ndim must be 1..3 and shape non-NULL");
  if (batch < 0) return report_error(ES_EINVAL, "batch must be >= 0");
  if (!(alpha > 0) || !std::isfinite(alpha)) return report_error(ES_EINVAL, "alpha must be positive and finite");
  if (!(rtol >= 0) || !std::isfinite(rtol)) return report_error(ES_EINVAL, "rtol must be finite and >= 0");
  if (max_iter < 0) return report_error(ES_EINVAL, "max_iter must be >= 0");
  if (check_every < 1) check_every = 1;
  if (iterations) *iterations = 0;
  if (batch == 0) return ES_OK;
  if (batch > 0x7fffffffll) return report_error(ES_EINVAL, "batch too large");
  int64_t n = 1;
  for (int k = 0; k < ndim; ++k) {
    if (shape[k] < 1) return report_error(ES_EINVAL, "shape entries must be positive");
    n *= shape[k];
  }
  const int64_t per = cg_parts(n);
  if (per * batch > 0x7fffffffll) return report_error(ES_EINVAL, "problem too large");
  // validates the operator arguments (order, levels, divisibility) through the workspace query
  const size_t cov = es_workspace_bytes(ndim, shape, batch, order, levels, ES_OP_COV);
  if (cov == 0 && levels > 1) return report_error(ES_EINVAL, "invalid operator arguments (order, levels, shape)");
  // partial sums: per-chunk (element-wise kernels) or per-tile (the fused operator steps)
  const int64_t parts = std::max(per, cov_dot_partials_max(ndim, shape));
  const CgLayout L = cg_layout(n, batch, cov, parts);
  if (!p || !mask || !x || !rel_residual) return report_error(ES_EINVAL, "p, mask, x and rel_residual must be non-NULL");
  if (((uintptr_t)p | (uintptr_t)mask | (uintptr_t)x) & 15) return report_error(ES_EINVAL, "p, mask and x must be 16-byte aligned");
  if (!ws || ws_bytes < L.total) {
    snprintf(msg, sizeof msg, "workspace of %zu bytes required", L.total);
    return report_error(ES_EWORKSPACE, msg);
  }
  if ((uintptr_t)ws & 255) return report_error(ES_EINVAL, "workspace must be 256-byte aligned");
  const size_t vb = (size_t)(n * batch) * sizeof(float);
  auto ov = [](const void* a, size_t na, const void* b, size_t nb) {
    return (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
  };
  if (ov(x, vb, p, vb) || ov(x, vb, mask, vb) || ov(ws, L.total, x, vb) || ov(ws, L.total, p, vb) ||
      ov(ws, L.total, mask, vb))
    return report_error(ES_EINVAL, "x must not overlap p, mask or the workspace; the workspace must not overlap p or mask");
  es_status st = device_check();
  if (st != ES_OK) return st;

  char* w = (char*)ws;
  float* r = (float*)(w + L.r);
  float* z = (float*)(w + L.z);
  float* d = (float*)(w + L.d);
  float* ad = (float*)(w + L.ad);
  float* part = (float*)(w + L.part);  // d . ad and r . z, then one reduced value per instance
  float* prr = (float*)(w + L.prr);    // r . r, likewise
  CgScal* sc = (CgScal*)(w + L.scal);
  void* cws = cov ? (void*)(w + L.cov) : nullptr;
  const hipStream_t hs = (hipStream_t)stream;
  const dim3 grid((unsigned)(per * batch)), blk(kCgThreads);
  const float frtol = (float)rtol;
  auto ok = [&](const char* what) -> es_status {
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return ES_OK;
    snprintf(msg, sizeof msg, "%s: %s", what, hipGetErrorString(e));
    return report_error(ES_EDEVICE, msg);
  };
  // partials as the next kernel takes them: as they are, or reduced to one per instance behind them
  auto reduced = [&](float* p, int64_t nparts, int64_t cap, Partials* q) -> es_status {
    *q = Partials{p, (int32_t)nparts};
    if (nparts <= kCgMaxParts) return ES_OK;
    float* one = p + cap * batch;
    hipLaunchKernelGGL(k_cg_reduce, dim3((unsigned)batch), blk, 0, hs, *q, one);
    *q = Partials{one, 1};
    return ok("CG reduction launch");
  };
  // Fused operator steps (2-D grids whose operator ends in the vector-path synthesis): the last
  // kernel of the operator also forms the mask term and the per-tile inner products, so the
  // separate update / inner-product passes over the vectors disappear.  Falls back to the
  // separate kernels when the schedule does not allow it.
  const char* fz = getenv("ESWAVE_CG_FUSED");  // 0: always the separate kernels (comparison)
  bool fused = cov_dot_partials_max(ndim, shape) > 0 && !(fz && *fz == '0');
  // the operators with their pairs of arrays, scheduled once: z = P r; ad = alpha Gamma^2 d + M d and
  // z = P r with the inner products
  CovApply op_z, op_ad, op_zdot;
  if ((st = op_z.prepare(ndim, shape, batch, order, levels, s, r, z, cws, cov)) != ES_OK) return st;
  if (fused) {
    st = op_ad.prepare_dot(ndim, shape, batch, order, levels, -s, d, ad, cws, cov, mask, 1.f, (float)alpha, part,
                           parts * batch);
    if (st == ES_OK)
      st = op_zdot.prepare_dot(ndim, shape, batch, order, levels, s, r, z, cws, cov, nullptr, 1.f, 1.f, part, parts * batch);
    if (st == ES_EUNSUPPORTED) fused = false;
    else if (st != ES_OK) return st;
  }
  if (!fused && (st = op_ad.prepare(ndim, shape, batch, order, levels, -s, d, ad, cws, cov)) != ES_OK) return st;

  // r = b = M p, x = 0, ||b||; z = P r, d = z, rz = r . z
  Partials rr, rz, dad;
  hipLaunchKernelGGL(k_cg_init, grid, blk, 0, hs, n, (int)per, p, mask, x, r, prr);
  if ((st = ok("CG init launch")) != ES_OK || (st = reduced(prr, per, per, &rr)) != ES_OK) return st;
  if ((st = op_z.run(hs)) != ES_OK) return st;
  hipLaunchKernelGGL(k_cg_dot, grid, blk, 0, hs, n, (int)per, r, z, d, part);
  if ((st = ok("CG dot launch")) != ES_OK || (st = reduced(part, per, parts, &rz)) != ES_OK) return st;
  hipLaunchKernelGGL(k_cg_start, dim3((unsigned)batch), blk, 0, hs, rr, rz, sc, frtol);
  if ((st = ok("CG start launch")) != ES_OK) return st;

  std::vector<CgScal> host((size_t)batch);
  auto read_scalars = [&](int it) -> es_status {
    hipError_t e = hipMemcpyAsync(host.data(), sc + (it & 1) * batch, host.size() * sizeof(CgScal), hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e == hipSuccess) return ES_OK;
    snprintf(msg, sizeof msg, "CG residual read: %s", hipGetErrorString(e));
    return report_error(ES_EDEVICE, msg);
  };
  int it = 0;
  bool done = false, read = false;  // read: host holds the scalars of iteration `it`
  while (it < max_iter && !done) {
    CgScal* cur = sc + (it & 1) * batch;
    CgScal* next = sc + ((it + 1) & 1) * batch;
    // ad = alpha Gamma^2 d + M d, d . ad
    if ((st = op_ad.run(hs)) != ES_OK) return st;
    if (!fused) {
      hipLaunchKernelGGL(k_cg_apply, grid, blk, 0, hs, n, (int)per, (float)alpha, mask, d, ad, part);
      if ((st = ok("CG operator update launch")) != ES_OK) return st;
    }
    if ((st = reduced(part, fused ? op_ad.parts() : per, parts, &dad)) != ES_OK) return st;
    // a = rz / (d . ad), r -= a ad, ||r||
    hipLaunchKernelGGL(k_cg_step, grid, blk, 0, hs, n, (int)per, dad, cur, r, (const float*)ad, prr);
    if ((st = ok("CG step launch")) != ES_OK || (st = reduced(prr, per, per, &rr)) != ES_OK) return st;
    // z = P r, r . z
    if ((st = (fused ? op_zdot : op_z).run(hs)) != ES_OK) return st;
    if (!fused) {
      hipLaunchKernelGGL(k_cg_dot, grid, blk, 0, hs, n, (int)per, r, z, (float*)nullptr, part);
      if ((st = ok("CG dot launch")) != ES_OK) return st;
    }
    if ((st = reduced(part, fused ? op_zdot.parts() : per, parts, &rz)) != ES_OK) return st;
    // rel = ||r|| / ||b||, beta = (r . z) / rz, x += a d, d = z + beta d
    hipLaunchKernelGGL(k_cg_dir, grid, blk, 0, hs, n, (int)per, rr, rz, (const CgScal*)cur, next, frtol, x, d,
                       (const float*)z);
    if ((st = ok("CG direction launch")) != ES_OK) return st;
    ++it;
    read = it % check_every == 0 || it == max_iter;
    if (read) {
      if ((st = read_scalars(it)) != ES_OK) return st;
      done = true;
      for (const CgScal& c : host) done = done && !(c.rel > frtol);
    }
  }
  if (!read && (st = read_scalars(it)) != ES_OK) return st;
  for (int64_t b = 0; b < batch; ++b) rel_residual[b] = host[(size_t)b].rel;
  if (iterations) *iterations = it;
  return ES_OK;
}


size_t es_tikhonov_gmres_workspace_bytes(int ndim, const int64_t* shape, int64_t batch, int order, int levels,
                                         int32_t restart) {
  if (batch < 1 || ndim < 1 || ndim > 3 || !shape || restart < 1 || restart > kGmMaxBasis) return 0;
  int64_t n = 1;
  for (int k = 0; k < ndim; ++k) n *= shape[k];
  const size_t cov = es_workspace_bytes(ndim, shape, batch, order, levels, ES_OP_COV);
  return gm_layout(n, batch, restart, cov, cg_parts(n)).total;
}

es_status es_tikhonov_gmres(int ndim, const int64_t* shape, int64_t batch, int order, int levels, double s,
                            double alpha, const float* p, const float* mask, float* x, int32_t restart,
                            int32_t max_iter, double rtol, int32_t* iterations, float* rel_residual, void* ws,
                            size_t ws_bytes, void* stream) {
  char msg[256];
  if (ndim < 1 || ndim > 3 || !shape) return report_error(ES_EINVAL, "ndim must be 1..3 and shape non-NULL");
  if (batch < 0) return report_error(ES_EINVAL, "batch must be >= 0");
  if (!(alpha > 0) || !std::isfinite(alpha)) return report_error(ES_EINVAL, "alpha must be positive and finite");
  if (!(rtol >= 0) || !std::isfinite(rtol)) return report_error(ES_EINVAL, "rtol must be finite and >= 0");
  if (max_iter < 0) return report_error(ES_EINVAL, "max_iter must be >= 0");
  if (restart < 1 || restart > kGmMaxBasis) return report_error(ES_EINVAL, "restart must be 1..64");
  if (iterations) *iterations = 0;
  if (batch == 0) return ES_OK;
  if (batch > 0x7fffffffll) return report_error(ES_EINVAL, "batch too large");
  int64_t n = 1;
  for (int k = 0; k < ndim; ++k) {
    if (shape[k] < 1) return report_error(ES_EINVAL, "shape entries must be positive");
    n *= shape[k];
  }
  const int64_t per = cg_parts(n);
  if (per * batch > 0x7fffffffll) return report_error(ES_EINVAL, "problem too large");
  const size_t cov = es_workspace_bytes(ndim, shape, batch, order, levels, ES_OP_COV);
  if (cov == 0 && levels > 1) return report_error(ES_EINVAL, "invalid operator arguments (order, levels, shape)");
  const int m = restart;
  const GmLayout L = gm_layout(n, batch, m, cov, per);
  if (!p || !mask || !x || !rel_residual) return report_error(ES_EINVAL, "p, mask, x and rel_residual must be non-NULL");
  if (((uintptr_t)p | (uintptr_t)mask | (uintptr_t)x) & 15) return report_error(ES_EINVAL, "p, mask and x must be 16-byte aligned");
  if (!ws || ws_bytes < L.total) {
    snprintf(msg, sizeof msg, "workspace of %zu bytes required", L.total);
    return report_error(ES_EWORKSPACE, msg);
  }
  if ((uintptr_t)ws & 255) return report_error(ES_EINVAL, "workspace must be 256-byte aligned");
  const size_t vb = (size_t)(n * batch) * sizeof(float);
  auto ov = [](const void* a, size_t na, const void* b, size_t nb) {
    return (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
  };
  if (ov(x, vb, p, vb) || ov(x, vb, mask, vb) || ov(ws, L.total, x, vb) || ov(ws, L.total, p, vb) ||
      ov(ws, L.total, mask, vb))
    return report_error(ES_EINVAL, "x must not overlap p, mask or the workspace; the workspace must not overlap p or mask");
  es_status st = device_check();
  if (st != ES_OK) return st;

  char* wsc = (char*)ws;
  float* V = (float*)(wsc + L.V);
  float* bv = (float*)(wsc + L.b);
  float* w = (float*)(wsc + L.w);
  float* t = (float*)(wsc + L.t);
  float* part = (float*)(wsc + L.part);
  float* hg = (float*)(wsc + L.hg);
  // row 0: the cycle's start norm; row k + 1: the column of Arnoldi step k.  A row holds ld = m + 1
  // floats per instance: the coefficients c_0 .. c_k, and ||w||^2 last
  float* cd = (float*)(wsc + L.c);
  float* Gd = (float*)(wsc + L.G);
  float* yd = (float*)(wsc + L.y);
  void* cws = cov ? (void*)(wsc + L.cov) : nullptr;
  const int64_t vs = L.vs;
  const int ld = m + 1;
  const int64_t row = batch * ld;
  const hipStream_t hs = (hipStream_t)stream;
  const dim3 grid((unsigned)(per * batch)), blk(kCgThreads);
  const int nblk = (int)(per * batch);
  auto ok = [&](const char* what) -> es_status {
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) return ES_OK;
    snprintf(msg, sizeof msg, "%s: %s", what, hipGetErrorString(e));
    return report_error(ES_EDEVICE, msg);
  };
  auto to_host = [&](void* dst, const void* src, size_t bytes) -> es_status {
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e == hipSuccess) return ES_OK;
    snprintf(msg, sizeof msg, "GMRES coefficient read: %s", hipGetErrorString(e));
    return report_error(ES_EDEVICE, msg);
  };
  // the partial sums of `nv` vectors, as the next kernel takes them: as they are, or reduced to one
  struct Parts {
    const float* p;
    int per, nblk;
  };
  auto reduced = [&](int nv, Parts* out) -> es_status {
    *out = Parts{part, (int)per, nblk};
    if (per <= kGmMaxParts) return ES_OK;
    hipLaunchKernelGGL(k_gm_final, dim3((unsigned)batch, (unsigned)nv), blk, 0, hs, (int)per, nblk, part, hg);
    *out = Parts{hg, 1, (int)batch};
    return ok("GMRES reduction launch");
  };
  auto normalise = [&](const float* src, float* v, float* norm_row) -> es_status {
    Parts q;
    es_status r = reduced(1, &q);
    if (r != ES_OK) return r;
    hipLaunchKernelGGL(k_gm_scale, grid, blk, 0, hs, n, (int)per, q.per, q.p, norm_row + m, ld, src, v, mask, t);
    return ok("GMRES scale launch");
  };
  // the operator with its two pairs of arrays, scheduled once
  CovApply op_b, op_w;
  if ((st = op_b.prepare(ndim, shape, batch, order, levels, s, t, bv, cws, cov)) != ES_OK) return st;
  if ((st = op_w.prepare(ndim, shape, batch, order, levels, s, t, w, cws, cov)) != ES_OK) return st;
  // w = b - A x and its norm's partials
  auto residual = [&]() -> es_status {
    hipLaunchKernelGGL(k_gm_mask, grid, blk, 0, hs, n, (int)per, 1, mask, x, t);
    es_status r = ok("GMRES mask launch");
    if (r == ES_OK) r = op_w.run(hs);
    if (r != ES_OK) return r;
    hipLaunchKernelGGL(k_gm_lin3, grid, blk, 0, hs, n, (int)per, 1.f, (const float*)bv, -1.f, (const float*)w,
                       (float)-alpha, x, w, part);
    return ok("GMRES update launch");
  };
  // host copies of the rows and the FP64 least-squares state per instance: R (upper triangle of the
  // rotated Hessenberg matrix, column-major m x m), rotations, right side g, ||b||, whether the
  // instance still takes steps, its steps this cycle
  std::vector<float> hb, yh, hn;
  std::vector<double> R, cs, sn, g, bn;
  std::vector<char> active;
  std::vector<int> kk;
  try {
    hb.resize((size_t)(row * ld));
    yh.assign((size_t)row, 0.f);
    hn.resize((size_t)batch);
    R.resize((size_t)batch * m * m);
    cs.resize((size_t)batch * m);
    sn.resize((size_t)batch * m);
    g.resize((size_t)row);
    bn.assign((size_t)batch, 0.0);
    active.resize((size_t)batch);
    kk.resize((size_t)batch);
  } catch (const std::bad_alloc&) {
    return report_error(ES_ENOMEM, "host memory for the GMRES coefficients of every instance");
  }

  // b = E_s^*(mask p), x = 0, v_0 = b / ||b||
  hipLaunchKernelGGL(k_gm_mask, grid, blk, 0, hs, n, (int)per, 0, mask, p, t);
  if ((st = ok("GMRES mask launch")) != ES_OK || (st = op_b.run(hs)) != ES_OK) return st;
  hipLaunchKernelGGL(k_gm_begin, grid, blk, 0, hs, n, (int)per, (const float*)bv, x, part);
  if ((st = ok("GMRES init launch")) != ES_OK || (st = normalise(bv, V, cd)) != ES_OK) return st;

  int it = 0;
  auto any_active = [&]() {
    for (char a : active)
      if (a) return true;
    return false;
  };
  bool have_bn = false;
  auto start_norms = [&]() {  // row 0 of hb: the cycle's start norms (the first cycle's: ||b||)
    for (int64_t b = 0; b < batch; ++b) {
      const double beta = std::sqrt((double)hb[b * ld + m]);
      if (!have_bn) {
        bn[b] = beta;
        active[b] = beta > 0 && 1.0 > rtol;
      } else if (active[b] && !(beta / bn[b] > rtol)) {
        active[b] = 0;
      }
      std::fill(g.begin() + b * ld, g.begin() + (b + 1) * ld, 0.0);
      g[b * ld] = beta;
      kk[b] = 0;
    }
    have_bn = true;
  };
  // Column k of the Hessenberg matrix of every active instance: rotations, residual estimate.
  auto take_column = [&](int k) {
    for (int64_t b = 0; b < batch; ++b) {
      if (!active[b]) continue;
      const float* hc = hb.data() + (size_t)(k + 1) * row + b * ld;
      double col[kGmMaxBasis + 1];
      for (int j = 0; j <= k; ++j) col[j] = (double)hc[j];
      col[k + 1] = std::sqrt((double)hc[m]);
      double* c = cs.data() + b * m;
      double* sv = sn.data() + b * m;
      for (int i = 0; i < k; ++i) {  // earlier rotations
        const double u = col[i], v = col[i + 1];
        col[i] = c[i] * u + sv[i] * v;
        col[i + 1] = -sv[i] * u + c[i] * v;
      }
      const double r = std::hypot(col[k], col[k + 1]);
      c[k] = r > 0 ? col[k] / r : 1.0;
      sv[k] = r > 0 ? col[k + 1] / r : 0.0;
      col[k] = r;
      double* gb = g.data() + b * ld;
      gb[k + 1] = -sv[k] * gb[k];
      gb[k] = c[k] * gb[k];
      for (int j = 0; j <= k; ++j) R[(size_t)b * m * m + (size_t)k * m + j] = col[j];
      kk[b] = k + 1;
      if (!(std::fabs(gb[k + 1]) / bn[b] > rtol) || r == 0) active[b] = 0;
    }
  };
  // Steps are enqueued without waiting; the host reads the columns where the residual may have
  // reached rtol.  Small problems (a step of ~50 us, a wait of ~25 us): after two steps, then where
  // the rate of the steps seen so far would reach 80 % of the way; a step past the end changes
  // nothing but the time.  Problems whose step outweighs the wait: after every step.
  const bool lag = n * batch <= (int64_t)1 << 22;
  const int coef_threads = launch_fits(batch, kGmCoefThreads) ? kGmCoefThreads : kGmCoefThreadsMany;
  while (1.0 > rtol && it < max_iter) {
    const int steps = std::min(m, max_iter - it);
    int K = 0, read = 0, next = lag ? (rtol > 0 ? std::min(2, steps) : steps) : 1;
    double seen = 1.0;
    bool stop = false;
    for (int k = 0; k < steps && !stop; ++k) {
      if ((st = op_w.run(hs)) != ES_OK) return st;
      // Gram-Schmidt against v_0 .. v_k: one pass of inner products (with w and with v_k), the
      // CGS2 coefficients from the Gram matrix, one update pass
      if (cg_chunk(n) == kCgChunkSmall)
        hipLaunchKernelGGL((k_gm_dots<kCgChunkSmall / kCgThreads>), grid, blk, 0, hs, n, (int)per, k + 1, (const float*)V, vs,
                           (float)alpha, w, part);
      else
        hipLaunchKernelGGL((k_gm_dots<kCgChunkLarge / kCgThreads>), grid, blk, 0, hs, n, (int)per, k + 1, (const float*)V, vs,
                           (float)alpha, w, part);
      Parts q;
      if ((st = ok("GMRES inner-product launch")) != ES_OK || (st = reduced(2 * (k + 1), &q)) != ES_OK) return st;
      float* col = cd + (int64_t)(k + 1) * row;
      hipLaunchKernelGGL(k_gm_coef, dim3((unsigned)batch), dim3((unsigned)coef_threads), 0, hs, k, q.per, q.nblk, q.p, Gd, ld, col, ld);
      if ((st = ok("GMRES coefficient launch")) != ES_OK) return st;
      hipLaunchKernelGGL(k_gm_sub, grid, blk, 0, hs, n, (int)per, k + 1, (const float*)V, vs, (const float*)col, ld, w, part);
      if ((st = ok("GMRES update launch")) != ES_OK || (st = normalise(w, V + (int64_t)(k + 1) * vs, col)) != ES_OK) return st;
      if (k + 1 < next && k + 1 < steps) continue;
      // rows not read yet (row 0 with the first ones)
      const int r0 = read == 0 ? 0 : read + 1;
      if ((st = to_host(hb.data() + (size_t)r0 * row, cd + (size_t)r0 * row,
                        (size_t)(k + 2 - r0) * row * sizeof(float))) != ES_OK)
        return st;
      if (read == 0) start_norms();
      const int from = read;
      for (; read <= k && any_active(); ++read) {
        take_column(read);
        ++it;
        ++K;
      }
      stop = !any_active();
      if (lag && !stop && rtol > 0) {
        double rel = 0;
        for (int64_t b = 0; b < batch; ++b)
          if (active[b]) rel = std::max(rel, std::fabs(g[b * ld + read]) / bn[b]);
        const double rate = std::log(rel / seen) / (read - from);  // per step, negative
        const double need = rate < 0 ? 0.8 * std::log(rtol / rel) / rate : 1;
        next = k + 1 + (int)std::max(1.0, std::min(need, (double)m));
        seen = rel;
      } else {
        next = lag ? steps : k + 2;
      }
    }
    if (K == 0) break;
    // x += V y, y = R^{-1} g over each instance's steps of this cycle
    for (int64_t b = 0; b < batch; ++b) {
      const int nk = kk[b];
      const double* Rb = R.data() + (size_t)b * m * m;
      double yv[kGmMaxBasis];
      for (int i = nk - 1; i >= 0; --i) {
        double v = g[b * ld + i];
        for (int j = i + 1; j < nk; ++j) v -= Rb[(size_t)j * m + i] * yv[j];
        yv[i] = Rb[(size_t)i * m + i] != 0 ? v / Rb[(size_t)i * m + i] : 0.0;
      }
      for (int j = 0; j < ld; ++j) yh[b * ld + j] = j < nk ? (float)yv[j] : 0.f;
    }
    hipError_t e = hipMemcpyAsync(yd, yh.data(), yh.size() * sizeof(float), hipMemcpyHostToDevice, hs);
    if (e == hipSuccess) e = hipStreamSynchronize(hs);
    if (e != hipSuccess) {
      snprintf(msg, sizeof msg, "GMRES coefficient write: %s", hipGetErrorString(e));
      return report_error(ES_EDEVICE, msg);
    }
    hipLaunchKernelGGL(k_gm_combine, grid, blk, 0, hs, n, (int)per, K, (const float*)V, vs, (const float*)yd, ld, x);
    if ((st = ok("GMRES combine launch")) != ES_OK) return st;
    if (!any_active() || it >= max_iter) break;
    // restart from the true residual r = b - A x: v_0 = r / ||r||
    if ((st = residual()) != ES_OK || (st = normalise(w, V, cd)) != ES_OK) return st;
  }
  if (!have_bn) {  // no step taken
    if ((st = to_host(hb.data(), cd, (size_t)row * sizeof(float))) != ES_OK) return st;
    start_norms();
  }
  // true relative residual of the final iterate
  if ((st = residual()) != ES_OK) return st;
  hipLaunchKernelGGL(k_gm_final, dim3((unsigned)batch, 1), blk, 0, hs, (int)per, nblk, part, hg);
  if ((st = ok("GMRES reduction launch")) != ES_OK || (st = to_host(hn.data(), hg, hn.size() * sizeof(float))) != ES_OK)
    return st;
  for (int64_t b = 0; b < batch; ++b)
    rel_residual[b] = bn[b] > 0 ? (float)(std::sqrt((double)hn[b]) / bn[b]) : 0.f;
  if (iterations) *iterations = it;
  return ES_OK;
}

}  // extern "C"
