// Composite low-pass filters of the coarsest levels, folded to short axes: compile-time device tables.
#pragma once

#include <utility>

#include "internal.h"

namespace es {

// Low-pass taps of db1 .. db8 as es_filter derives them (a host test compares the two).
constexpr double kDaubechies[kMaxTaps / 2][kMaxTaps] = {
    {0.70710678118654757, 0.70710678118654757},
    {0.48296291314453416, 0.83651630373780794, 0.22414386804201339, -0.12940952255126037},
    {0.33267055295008263, 0.80689150931109255, 0.45987750211849154, -0.13501102001025458, -0.085441273882026658,
     0.035226291885709533},
    {0.23037781330889651, 0.71484657055291567, 0.63088076792985892, -0.027983769416859854, -0.18703481171909309,
     0.030841381835560764, 0.032883011666885197, -0.010597401785069032},
    {0.16010239797419293, 0.60382926979718965, 0.72430852843777294, 0.13842814590132074, -0.24229488706638203,
     -0.032244869584638375, 0.077571493840045719, -0.0062414902127982744, -0.012580751999081999,
     0.0033357252854737712},
    {0.11154074335010947, 0.49462389039845306, 0.75113390802109536, 0.31525035170919763, -0.22626469396543983,
     -0.12976686756726194, 0.097501605587323043, 0.027522865530305727, -0.03158203931748603,
     0.00055384220116149613, 0.0047772575109455108, -0.0010773010853084796},
    {0.077852054085009184, 0.39653931948191729, 0.72913209084623509, 0.46978228740519312, -0.14390600392856498,
     -0.22403618499387498, 0.071309219266830259, 0.080612609151083078, -0.038029936935014413,
     -0.016574541630666881, 0.01255099855609984, 0.00042957797292136651, -0.0018016407040474908,
     0.00035371379997452024},
    {0.054415842243104008, 0.31287159091429995, 0.67563073629728976, 0.58535468365420673, -0.015829105256349306,
     -0.28401554296154691, 0.00047248457391328285, 0.12874742662047847, -0.017369301001807547,
     -0.044088253930794755, 0.013981027917398282, 0.0087460940474057766, -0.0048703529934515741,
     -0.00039174037337694705, 0.00067544940645056933, -0.00011747678412476953}};

constexpr int kDenseSide = 32;   // longest axis of a block whose levels run as matrix products
constexpr int kDenseLevels = 4;  // levels below such a block: the coarsest one is never visited, so 2 divides its sides too

// Level of row r of an axis of length n that stacks the rows of every level, finest first: the distance n - r from
// the end lies in (n / 2^i, n / 2^(i-1)] for level i.  Above the number of levels for rows past the last one's.
constexpr int dense_level(int n, int r) {
  int level = 1;
  for (int q = 1; q <= kDenseLevels; ++q) level += n - r <= (n >> q);
  return level;
}

// c[n / 2][i - 1]: C_i with a_i[k] = sum_j C_i[j] x[(j + 2^i k) mod n], the i-level low-pass analysis of a
// periodic axis of even length n <= 32 that 2^i divides; formed in FP64, rounded once.
struct CompositeTable {
  float c[kDenseSide / 2 + 1][kDenseLevels][kDenseSide];
};

template <int L, int N>
constexpr void composite_of_length(CompositeTable& r) {
  double cur[N] = {1.0};
  for (int i = 1; i <= kDenseLevels && N % (1 << i) == 0; ++i) {
    double next[N] = {};
    for (int u = 0; u < L; ++u)
      for (int j = 0; j < N; ++j) next[(j + (u << (i - 1))) % N] += kDaubechies[L / 2 - 1][u] * cur[j];
    for (int j = 0; j < N; ++j) {
      cur[j] = next[j];
      r.c[N / 2][i - 1][j] = (float)next[j];
    }
  }
}

template <int L, int... H>
constexpr CompositeTable make_composite(std::integer_sequence<int, H...>) {
  CompositeTable r{};
  (composite_of_length<L, 2 * H + 2>(r), ...);
  return r;
}

// In device memory with the code, so that neither a launch's arguments (host memory) nor a first call
// carries them.
template <int L>
__device__ const CompositeTable kComposite = make_composite<L>(std::make_integer_sequence<int, kDenseSide / 2>{});

}  // namespace es
