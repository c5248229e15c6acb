// 2-D low-pass launches that hold instances of every filter length (plans of different instances).  A
// launch that is too small to fill the chip takes 4-5 us whatever it does, and a plan ran one per phase
// and filter length; here each work-group branches on its task's length to the body that the one-length
// kernels run, so the bits are theirs.  Registers and LDS are those of 16 taps (the tile of 16 x 64: 73
// registers, 26.8 KB, five work-groups a CU), which costs the shorter filters less than their own launches.
// Plans of 2 filter lengths with and without, us: 4 x 1024^2 80 -> 54, 32 x 1024^2 175 -> 143, 64 x 512^2
// 111 -> 86, 64 x 256^2 65 -> 63 (never slower, so there is no limit); 48 instances of mixed sizes, three
// lengths and some cubes 298 -> 218, 36 of them 226 -> 149, 8 of them 137 -> 81 (calls one after the other;
// a call alone, from its submission to a synchronisation, is 256, 181 and 103).

#include "kcommon.h"
#include "lowpass.h"

namespace es {

namespace {

#define ES_EACH_TAPS(M) M(2) M(4) M(6) M(8) M(10) M(12) M(14) M(16)

template <int T1, int T2>
__global__ void __launch_bounds__(kThreads) k_mixed_down(TaskArgs args, FilterBank bank) {
  __shared__ __attribute__((aligned(16))) unsigned char sm[sizeof(LpDownSmem<2, kMaxTaps, 1, T1, T2>)];
  const int wg = logical_wg(args.total_wg, args.reverse);
  if (wg < 0) return;
  const Task t = pick_task<Task>(args, wg);
  switch (__builtin_amdgcn_readfirstlane(t.taps)) {
#define ES_CASE(L)                                                                                                  \
  case L: {                                                                                                         \
    using S = LpDownSmem<2, L, 1, T1, T2>;                                                                          \
    static_assert(sizeof(S) <= sizeof(sm), "the longest filter's tile is the largest");                             \
    lp_down_tile<2, L, 1, T1, T2, kThreads, true>(t, wg, bank.f[L / 2 - 1], *reinterpret_cast<S*>(sm));             \
    break;                                                                                                          \
  }
    ES_EACH_TAPS(ES_CASE)
#undef ES_CASE
  }
}

template <int U1, int U2, bool VEC>
__global__ void __launch_bounds__(kThreads) k_mixed_up(TaskArgs args, FilterBank bank) {
  __shared__ __attribute__((aligned(16))) unsigned char sm[sizeof(LpUpSmem<2, kMaxTaps, 1, U1, U2>)];
  const int wg = logical_wg(args.total_wg, args.reverse);
  if (wg < 0) return;
  const Task t = pick_task<Task>(args, wg);
  switch (__builtin_amdgcn_readfirstlane(t.taps)) {
#define ES_CASE(L)                                                                                                  \
  case L: {                                                                                                         \
    using S = LpUpSmem<2, L, 1, U1, U2>;                                                                            \
    static_assert(sizeof(S) <= sizeof(sm), "the longest filter's tile is the largest");                             \
    lp_up_tile<2, L, 1, U1, U2, kThreads, VEC>(t, wg, bank.f[L / 2 - 1], *reinterpret_cast<S*>(sm));                \
    break;                                                                                                          \
  }
    ES_EACH_TAPS(ES_CASE)
#undef ES_CASE
  }
}

template <int CMAX>
__global__ void __launch_bounds__(coarse_threads(CMAX)) k_mixed_coarse(TailArgs args, FilterBank bank) {
  __shared__ __attribute__((aligned(16))) float sm[coarse_lds_floats(2, CMAX)];
  const int wg = logical_wg(args.total_wg);
  if (wg < 0) return;
  int lo = 0, hi = args.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (args.table[mid].tile_begin <= wg) lo = mid;
    else hi = mid - 1;
  }
  const TailTask* tp = args.table + lo;
  switch (__builtin_amdgcn_readfirstlane(tp->taps)) {
#define ES_CASE(L) \
  case L: lp_coarse_block<2, L, CMAX, coarse_threads(CMAX)>(tp, wg - tp->tile_begin, bank.f[L / 2 - 1], sm); break;
    ES_EACH_TAPS(ES_CASE)
#undef ES_CASE
  }
}

template <int V>
void launch_v(int kind, bool vec, const TaskArgs& a, int grid, const FilterBank& b, hipStream_t s) {
  constexpr Shape3 dn = shape_of(K_LP_DOWN, 2, V, kMaxTaps), up = shape_of(K_LP_UP, 2, V, kMaxTaps);
  if (kind == K_LP_DOWN)
    hipLaunchKernelGGL((k_mixed_down<dn.b, dn.c>), dim3(grid), dim3(kThreads), 0, s, a, b);
  else if (vec)
    hipLaunchKernelGGL((k_mixed_up<up.b, up.c, true>), dim3(grid), dim3(kThreads), 0, s, a, b);
  else
    hipLaunchKernelGGL((k_mixed_up<up.b, up.c, false>), dim3(grid), dim3(kThreads), 0, s, a, b);
}

}  // namespace

hipError_t launch_mixed_level(int kind, int variant, const TaskArgs& args, int grid, const FilterBank& bank,
                              hipStream_t s) {
  const bool vec = args.vec != 0;
  if (args.table == nullptr || (kind != K_LP_DOWN && kind != K_LP_UP) || (kind == K_LP_DOWN && !vec))
    return hipErrorInvalidValue;
  TaskArgs a = args;
  a.bank = nullptr;
  if (variant == 0) launch_v<0>(kind, vec, a, grid, bank, s);
  else if (variant == 2) launch_v<2>(kind, vec, a, grid, bank, s);
  else launch_v<1>(kind, vec, a, grid, bank, s);
  return hipGetLastError();
}

hipError_t launch_mixed_coarse(const TailArgs& args, int grid, size_t lds_bytes, const FilterBank& bank, hipStream_t s) {
  if (args.table == nullptr) return hipErrorInvalidValue;
  TailArgs a = args;
  a.bank = nullptr;
  if (lds_bytes <= sizeof(float) * coarse_lds_floats(2, kCoarseMaxBlock))
    hipLaunchKernelGGL((k_mixed_coarse<kCoarseMaxBlock>), dim3(grid), dim3(coarse_threads(kCoarseMaxBlock)), 0, s, a, bank);
  else
    hipLaunchKernelGGL((k_mixed_coarse<kCoarseMaxBlockBig>), dim3(grid), dim3(coarse_threads(kCoarseMaxBlockBig)), 0, s, a, bank);
  return hipGetLastError();
}

}  // namespace es
