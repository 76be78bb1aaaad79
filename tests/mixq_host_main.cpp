// Host check of the sample-domain channel mixing (test infrastructure, run by
// tests/test_mix_tables.py): the operand images' three bf16 parts through the
// kernel's own index arithmetic, against the spherical harmonics and their
// orthonormality, and the rule that chooses between it and the pair products.
#include <cmath>
#include <cstdio>
#include <vector>

#include "gtp_mixq_tables.hpp"
#include "gtp_tables.hpp"

namespace {

int fails = 0;
void check(bool ok, const char* what, int a = 0, int b = 0) {
  if (!ok && fails++ < 10) std::printf("FAIL %s %d %d\n", what, a, b);
}

template <int L>
void degree() {
  using G = gtp::MixqGeo<L>;
  const std::vector<uint16_t> im = gtp::build_mixq_images(L);
  check(int(im.size()) == G::HALVES, "size", L);
  auto parts = [&](int base, int frag, int lane, int j) {
    double v[3];
    for (int p = 0; p < 3; ++p) v[p] = gtp::bf16_value(im[base + ((frag * 3 + p) * 64 + lane) * 8 + j]);
    check(std::fabs(v[1]) <= std::ldexp(std::fabs(v[0]), -8) && std::fabs(v[2]) <= std::ldexp(std::fabs(v[1]), -8),
          "parts", L);
    return v[0] + v[1] + v[2];
  };
  const int NQ = 16 * G::NWQ * G::T;
  std::vector<double> ys(NQ * G::K), ya(NQ * G::K);
  for (int lane = 0; lane < 64; ++lane)
    for (int j = 0; j < 8; ++j) {
      const int g = lane / 16, i = lane % 16;
      for (int tile = 0; tile < G::NWQ * G::T; ++tile)
        for (int s = 0; s < G::KS; ++s) {
          const int k = 32 * s + 8 * g + j, q = 16 * tile + i;
          const double v = parts(G::YS, tile * G::KS + s, lane, j);
          if (k < G::K) ys[q * G::K + k] = v;
          check((k < G::K && q < G::Q) || v == 0.0, "padding of the values", q, k);
        }
      for (int kt = 0; kt < G::KT; ++kt)
        for (int ws = 0; ws < 4 * G::NWQ; ++ws) {
          const int k = 16 * kt + i, q = 16 * (G::T * (ws / 4) + j) + 4 * (ws % 4) + g;
          const double v = parts(G::YA, kt * 4 * G::NWQ + ws, lane, j);
          if (j < G::T && k < G::K) ya[q * G::K + k] = v;
          check((j < G::T && k < G::K && q < G::Q) || v == 0.0, "padding of the weighted values", q, k);
        }
    }
  // the values: the l = 1 triple of each point is a direction, in which the
  // zonal sum over each degree has its known value; and the weighted ones
  // integrate products to the identity
  const double pi = 3.14159265358979323846;
  for (int q = 0; q < G::Q; ++q)
    for (int l = 0; l <= L; ++l) {
      double s = 0.0;
      for (int k = l * l; k < (l + 1) * (l + 1); ++k) s += ys[q * G::K + k] * ys[q * G::K + k];
      check(std::fabs(s - (2 * l + 1) / (4 * pi)) <= 1e-6, "addition theorem", q, l);
    }
  for (int a = 0; a < G::K; ++a)
    for (int b = 0; b < G::K; ++b) {
      double s = 0.0;
      for (int q = 0; q < G::Q; ++q) s += ya[q * G::K + a] * ys[q * G::K + b];
      check(std::fabs(s - (a == b)) <= 1e-6, "orthonormality", a, b);
    }
}

void rule() {
  auto pays = [](int L, int64_t B, int64_t C1, int64_t C2, int64_t Co) {
    int nct = 1;
    while (16 * nct < Co) nct *= 2;
    // (either input may take either role where both cost the same)
    if (gtp::mixq_steps(C1) * C2 != gtp::mixq_steps(C2) * C1)
      check(gtp::mixq_pays(L, B, C1, C2, Co, nct) == gtp::mixq_pays(L, B, C2, C1, Co, nct), "rule's symmetry", L);
    return gtp::mixq_pays(L, B, C1, C2, Co, nct);
  };
  for (int L = 1; L <= 8; ++L) {
    // one, two or three channels against many: the pair products measured up to 2.9 times faster
    for (int64_t B : {1, 16, 256, 2048, 16384})
      for (int64_t Co : {8, 32, 64, 128})
        for (auto c : {std::pair<int64_t, int64_t>{256, 2}, {64, 2}, {128, 1}, {43, 3}})
          check(!pays(L, B, c.first, c.second, Co), "few channels", L, int(B));
    check(pays(L, 8192, 32, 32, 32) && pays(L, 2000, 64, 64, 64), "many channels", L);
  }
  check(!pays(7, 16384, 16, 16, 128) && !pays(1, 16, 64, 32, 32) && !pays(6, 2048, 16, 16, 64) &&
            !pays(7, 2048, 64, 8, 128), "measured slower");
  check(pays(8, 16, 32, 32, 32) && pays(6, 16384, 16, 16, 8) && pays(8, 16384, 32, 4, 8), "measured faster");
}

}  // namespace

int main() {
  check(gtp::bf16_bits(1.0) == 0x3f80 && gtp::bf16_bits(1.0 + std::ldexp(1.0, -8)) == 0x3f80 &&
            gtp::bf16_bits(1.0 + 3 * std::ldexp(1.0, -8)) == 0x3f82 && gtp::bf16_bits(-2.0) == 0xc000,
        "bf16 rounding");
  degree<1>();
  degree<2>();
  degree<3>();
  degree<4>();
  degree<5>();
  degree<6>();
  degree<7>();
  degree<8>();
  rule();
  std::printf(fails ? "failed %d\n" : "ok\n", fails);
  return fails != 0;
}
