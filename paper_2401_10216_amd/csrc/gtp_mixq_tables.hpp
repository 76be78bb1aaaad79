// Sphere quadrature and operand images of the sample-domain channel mixing
// (gtp_mixq.hip), made on the host.
//
// Degree L = 1..8: Gauss-Legendre nodes in cos(theta) (3 L / 2 + 1) times 3 L +
// 1 uniform phi, exact for the triple products' degree 3 L; the Q points are
// numbered in TILES tiles of 16 (the last one's rest is padding, zero in every
// image), T tiles to a wave and NWQ waves to a batch entry.  Images of
// v_mfma_f32_16x16x32_bf16 operands in three bf16 parts (gtp_split.hpp), eight
// values per lane 16 g + i:
//   YS[tile][step][part]     column i = point 16 tile + i, contraction indices
//        = coefficients 32 step + 8 g + j: Y_k(point)
//   YA[ktile][wave][s][part] column i = coefficient 16 ktile + i, contraction
//        indices = points 16 (T wave + j) + 4 s + g, j < T: w Y_k(point)
#pragma once

#include <cmath>
#include <cstdint>
#include <utility>
#include <vector>

namespace gtp {

template <int L>
struct MixqGeo {
  static_assert(L >= 1 && L <= 8, "degrees of the sample-domain channel mixing");
  static constexpr int K = (L + 1) * (L + 1), NTH = 3 * L / 2 + 1, NPH = 3 * L + 1, Q = NTH * NPH;
  static constexpr int TILES = (Q + 15) / 16;
  // waves per batch entry and tiles per wave; at the smallest degrees a wave
  // takes several batch entries, so that a weight operand serves four tiles or more
  static constexpr int NWQ = L <= 4 ? 1 : L <= 6 ? 2 : 4;
  static constexpr int T = (TILES + NWQ - 1) / NWQ, NB = L == 1 ? 4 : L == 2 ? 2 : 1;
  static constexpr int KS = (K + 31) / 32, KT = (K + 15) / 16;
  static constexpr int FR = 64 * 8;  // values of an image
  static constexpr int YS = 0, YA = YS + NWQ * T * KS * 3 * FR, HALVES = YA + KT * NWQ * 4 * 3 * FR;
};

// Contractions per 16 points and 16 outputs with C channels as the
// contraction index (the call gives C1 the role that costs less).
inline int64_t mixq_steps(int64_t C) { return C <= 16 ? 3 : 6 * ((C + 31) / 32); }

// Whether the sample domain is the faster way for B entries of C1 x C2 -> Co
// channels at degree L, against the pair products (k_mix_fused, nct tiles of 16
// outputs).  Sampling costs per channel, again for every 32 outputs and, the
// other input's, every 32 contracted channels; so it pays where each sample
// serves many pairs and outputs: 8192 entries of 32 x 32 -> 32 at L = 6 521 us
// against 1029, but 2048 of 256 x 2 -> 32 at L = 1 102 against 35, 16384 of 16 x 16
// -> 128 at L = 7 2.6 times the pairs'.  Both times in us from per-degree constants
// fitted to 3792 sizes measured both ways (128 to 4096 pairs, 8 to 128 outputs, 16
// to 16384 entries) within 30 %: a fixed part, which a small batch pays, and one
// per entry.  By this rule those sizes take 1.02 times the faster way's time in
// the geometric mean.  Under 4 channels in one input (padded to 16 or 32) the
// pair products were the faster everywhere.
inline bool mixq_pays(int L, int64_t B, int64_t C1, int64_t C2, int64_t Co, int nct) {
  struct Cost {
    double chunk_us, chunk, tile;     // pairs: 256 of them, fixed; per entry (ns), and per 16 outputs
    double base, channels, products;  // samples per entry (ns): all, 16 channels, 100 steps
  };
  static constexpr Cost kCost[8] = {
      {3.8, 0.4, 2.4, 1.6, 0.6, 1.3},   {4.5, 1.4, 2.6, 1.7, 0.8, 2.2},  {4.6, 4.0, 2.8, 1.6, 1.1, 4.1},
      {6.4, 8.8, 4.0, 2.2, 1.6, 6.0},   {8.3, 15.5, 4.6, 8.0, 2.7, 9.2}, {12.7, 24.5, 4.9, 7.3, 3.1, 12.9},
      {19.6, 41.0, 5.6, 16.0, 5.4, 16.0}, {28.2, 110.0, 11.5, 25.0, 8.7, 22.2}};
  if (L < 1 || L > 8 || C1 < 4 || C2 < 4) return false;
  if (mixq_steps(C2) * C1 < mixq_steps(C1) * C2) std::swap(C1, C2);
  const Cost& k = kCost[L - 1];
  const double n = 1e-3 * double(B);  // ns an entry to us
  const double chunks = double(C1) * double(C2) <= 256.0 ? 1.0 : std::ceil(double(C1) * double(C2) / 256.0);
  const double pairs =
      std::fmax(8.5 + chunks * (k.chunk_us + 1.5 * nct), n * chunks * (k.chunk + k.tile * nct));
  const double turns = C1 <= 16 ? 1.0 : double((C1 + 31) / 32);  // of 16 or 32 contracted channels
  const double sampled = turns * ((C1 <= 16 ? 1.0 : 2.0) + 2.0 * double((C2 + 31) / 32));
  const double steps = 0.01 * double(mixq_steps(C1)) * double(C2) * (Co <= 16 ? 1.0 : 2.0);
  const double fixed = 20.0 + 1.5 * sampled + 4.0 * steps;
  const double each = n * double((Co + 31) / 32) * (k.base + k.channels * sampled + k.products * steps);
  // (the larger of the two, a little more where they are alike)
  return 1.05 * std::sqrt(std::hypot(fixed * fixed, each * each)) < pairs;
}

// bf16 bits of a double (round to nearest even; normal range).
uint16_t bf16_bits(double v);
double bf16_value(uint16_t b);

// The images of degree L (1..8).
std::vector<uint16_t> build_mixq_images(int L);

}  // namespace gtp
