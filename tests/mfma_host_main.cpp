// Host check of the split-operand matrix-core kernel's images (test
// infrastructure, run by tests/test_mfma_product.py): the half conversion over
// every finite half, the two-part tables against the plan's fp64 ones through
// the kernel's own index arithmetic, and the index images' bounds.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "gtp_mfma_tables.hpp"

namespace {

int fails = 0;
void check(bool ok, const char* what) {
  if (!ok && fails++ < 10) std::printf("FAIL %s\n", what);
}

template <int L>
void degree() {
  using G = gtp::MfmaGeo<L>;
  const gtp::Tables t = gtp::build_tables(L, L, L);
  const gtp::MfmaImages im = gtp::build_mfma_images(t);
  check(int(im.f.size()) == G::FLOATS && int(im.h.size()) == G::HALVES, "sizes");
  auto half = [&](int base, int frag, int lane, int j) { return gtp::half_value(im.h[base + (frag * 64 + lane) * 8 + j]); };
  auto S = [&](int l, int m, int j) { return t.S[size_t(gtp::tri(l, m)) * t.NJ + j]; };
  const double wscale = std::ldexp(1.0, im.kw);
  // every order of 1..L in exactly one quad; every coefficient in one step
  int seen[L + 1] = {0}, coeff[L + 1][L + 1] = {{0}};
  for (int q = 0; q < G::NQ; ++q)
    for (int mi = 0; mi < 4; ++mi) {
      const int m = G::order(q, mi);
      ++seen[m];
      for (int par = 0; par < 2; ++par)
        for (int s = 0; s < G::steps(mi); ++s)
          for (int g = 0; g < 4; ++g) {
            const int l = m + par + 2 * (4 * s + g), f = G::step0(mi, par) + s;
            if (l <= L) ++coeff[l][m];
            for (int tile = 0; tile < G::NPT; ++tile)
              for (int i = 0; i < 16; ++i) {
                const double v = im.f[G::SA + ((size_t(tile * G::NQ + q) * G::SAV + f / 4) * 64 + 16 * g + i) * 4 + f % 4];
                check(v == (l <= L ? S(l, m, 16 * tile + i + 1) : 0.0), "theta synthesis entry");
              }
          }
      // theta analysis: the two parts of W within 2^-22 of the entry (or half a
      // subnormal step)
      for (int par = 0; par < 2; ++par)
        for (int i = 0; i < 16; ++i)
          for (int pair = 1; pair <= L; ++pair) {
            const int l = m + par + 2 * i, c = q * 8 + 2 * mi + par, g = (pair - 1) / 8, j = (pair - 1) % 8;
            const double w = l <= L ? wscale * t.W[size_t(gtp::tri(l, m)) * t.NJ + pair] / (G::PHI * G::PHI * G::PHI) : 0.0;
            const double v = L == 16 ? half(G::WC, c, 16 * g + i, j) + half(G::WC, c, 16 * (g + 2) + i, j)
                                     : half(G::WC, c * 2, 16 * g + i, j) + half(G::WC, c * 2 + 1, 16 * g + i, j);
            check(std::fabs(v - w) <= std::fmax(std::ldexp(std::fabs(w), -22), std::ldexp(1.0, -25)), "analysis entry");
          }
    }
  for (int m = 1; m <= L; ++m) check(seen[m] == 1, "order");
  for (int l = 1; l <= L; ++l)
    for (int m = 1; m <= l; ++m) check(coeff[l][m] == 1, "coefficient");
  // the phi tables' parts: the even and odd cosines and sines of every order, and
  // the rms of what the parts leave of them (at L = 16 below fp32's rounding, 1.4e-8)
  double left = 0.0;
  int entries = 0;
  for (int type = 0; type < 4; ++type)
    for (int mb = 0; mb < G::NMB; ++mb)
      for (int lane = 0; lane < (L == 16 ? 32 : 64); ++lane)
        for (int j = 0; j < 4; ++j) {
          const int k = 16 * mb + lane % 16, q = (type & 1 ? 0 : G::NSL) + lane / 16, m = G::order(q, j);
          if (k > G::Q) continue;
          const double a = 6.283185307179586476925286766559 * ((m * k) % G::NP) / G::NP;
          const double v = type >= 2 ? std::sin(a) : std::cos(a);
          const double h = half(G::TP, type * G::NMB + mb, lane, j) +
                           (L == 16 ? half(G::TP, type * G::NMB + mb, lane + 32, j) : half(G::TP, type * G::NMB + mb, lane, j + 4));
          check(std::fabs(h / G::PHI - v) <= std::ldexp(1.0, -24), "phi table entry");
          left += (h / G::PHI - v) * (h / G::PHI - v);
          ++entries;
        }
  check(std::sqrt(left / entries) <= (L == 16 ? 1.0e-8 : 3.0e-8), "phi tables' rms");
  // index images: within the stage and the output image, every output once
  const int cases[][3] = {{L, L, L}, {L - 3, 2, 2 * L}, {1, L, 5}, {0, L, L}};
  for (const auto& c : cases) {
    const int K = gtp::nsh(L), k1 = gtp::nsh(c[0]), k2 = gtp::nsh(c[1]), ko = gtp::nsh(c[2]), kk = ko < K ? ko : K;
    const auto v = gtp::build_mfma_index(L, k1, k2, ko);
    check(v.size() == size_t(G::NTH) * (G::GATHER + 2 * G::SCATTER), "index size");
    std::vector<int> in(8 * K + 1, 0), out(4 * K + 1, 0);
    for (int tid = 0; tid < G::NTH; ++tid) {
      const int wave = tid / 64;
      for (int f = 0; f < G::NSTEP + G::NS0; ++f) {
        const int e = v[size_t(tid) * G::GATHER + f];
        check(e % 4 == 0 && e / 4 <= 8 * K, "gather bound");
        if (f < G::NSTEP || wave < 2) ++in[e / 4];
      }
      const uint16_t* o = &v[size_t(G::NTH) * G::GATHER + size_t(tid) * 2 * G::SCATTER];
      for (int j = 0; j < (wave < G::NPART ? 17 : 16); ++j) {
        check(o[j] % 4 == 0 && o[j] / 4 <= 4 * K, "scatter bound");
        ++out[o[j] / 4];
      }
    }
    for (int p = 0; p < 4; ++p) {
      for (int k = 0; k < k1; ++k) check(in[p * k1 + k] == 1, "x1 coefficient");
      for (int k = 0; k < k2; ++k) check(in[4 * K + p * k2 + k] == 1, "x2 coefficient");
      for (int k = 0; k < kk; ++k) check(out[p * kk + k] == 1, "output coefficient");
    }
  }
}

}  // namespace

int main() {
  for (int h = 0; h < 0x10000; ++h)
    if ((h & 0x7c00) != 0x7c00) check(gtp::half_bits(gtp::half_value(uint16_t(h))) == h, "half round trip");
  // ties to even, and the binades' edges
  check(gtp::half_bits(1.0 + std::ldexp(1.0, -11)) == 0x3c00 && gtp::half_bits(1.0 + 3 * std::ldexp(1.0, -11)) == 0x3c02, "ties");
  check(gtp::half_bits(std::ldexp(1.0, -25)) == 0 && gtp::half_bits(std::ldexp(1.5, -25)) == 1, "subnormal ties");
  check(gtp::half_bits(2.0 - std::ldexp(1.0, -12)) == 0x4000 && gtp::half_bits(65519.0) == 0x7bff, "carry");
  degree<16>();
  degree<32>();
  std::printf(fails ? "failed %d\n" : "ok\n", fails);
  return fails != 0;
}
