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

#include <cstdint>
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

// bf16 bits of a double (round to nearest even; normal range).
uint16_t bf16_bits(double v);
double bf16_value(uint16_t b);

// The images of degree L (1..8).
std::vector<uint16_t> build_mixq_images(int L);

}  // namespace gtp
