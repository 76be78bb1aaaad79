#include "gtp_mixq_tables.hpp"

#include <cmath>
#include <cstring>

#include "gtp_tables.hpp"

namespace gtp {

namespace {

const double kPiQ = 3.14159265358979323846264338327950288;

template <int L>
std::vector<uint16_t> images() {
  using G = MixqGeo<L>;
  std::vector<double> z, w;
  gauss_legendre(G::NTH, z, w);
  std::vector<double> Y(size_t(G::Q) * G::K), wq(G::Q), th(ntri(L));
  for (int a = 0; a < G::NTH; ++a) {
    theta_factors(L, std::acos(z[a]), th.data());
    for (int b = 0; b < G::NPH; ++b) {
      const int q = a * G::NPH + b;
      wq[q] = w[a] * 2.0 * kPiQ / G::NPH;
      for (int l = 0; l <= L; ++l)
        for (int m = -l; m <= l; ++m) {
          const double ph = 2.0 * kPiQ * double((std::abs(m) * b) % G::NPH) / G::NPH;
          const double v = th[tri(l, std::abs(m))] * (m < 0 ? std::sin(ph) : std::cos(ph));
          Y[size_t(q) * G::K + l * l + l + m] = v;
        }
    }
  }
  auto part_of = [](double x, int part) {
    for (; part > 0; --part) x -= bf16_value(bf16_bits(x));
    return bf16_bits(x);
  };
  std::vector<uint16_t> v(G::HALVES, 0);
  for (int lane = 0; lane < 64; ++lane) {
    const int g = lane / 16, i = lane % 16;
    for (int j = 0; j < 8; ++j)
      for (int part = 0; part < 3; ++part) {
        auto put = [&](int base, int frag, double x) {
          v[size_t(base) + (size_t(frag * 3 + part) * 64 + lane) * 8 + j] = part_of(x, part);
        };
        for (int tile = 0; tile < G::NWQ * G::T; ++tile)
          for (int s = 0; s < G::KS; ++s) {
            const int q = 16 * tile + i, k = 32 * s + 8 * g + j;
            put(G::YS, tile * G::KS + s, q < G::Q && k < G::K ? Y[size_t(q) * G::K + k] : 0.0);
          }
        for (int kt = 0; kt < G::KT; ++kt)
          for (int ws = 0; ws < G::NWQ * 4; ++ws) {
            const int q = 16 * (G::T * (ws / 4) + j) + 4 * (ws % 4) + g, k = 16 * kt + i;
            const bool in = j < G::T && q < G::Q && k < G::K;
            put(G::YA, kt * G::NWQ * 4 + ws, in ? wq[q] * Y[size_t(q) * G::K + k] : 0.0);
          }
      }
  }
  return v;
}

}  // namespace

uint16_t bf16_bits(double v) {
  // (through fp32: where that makes a tie either neighbour will do, the rest
  // goes into the next part)
  const float f = float(v);
  uint32_t u;
  std::memcpy(&u, &f, 4);
  return uint16_t((u + 0x7fffu + (u >> 16 & 1)) >> 16);
}

double bf16_value(uint16_t b) {
  const uint32_t u = uint32_t(b) << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

std::vector<uint16_t> build_mixq_images(int L) {
  switch (L) {
    case 1: return images<1>();
    case 2: return images<2>();
    case 3: return images<3>();
    case 4: return images<4>();
    case 5: return images<5>();
    case 6: return images<6>();
    case 7: return images<7>();
    case 8: return images<8>();
    default: break;
  }
  return {};
}

}  // namespace gtp
