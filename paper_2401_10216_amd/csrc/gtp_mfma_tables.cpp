#include "gtp_mfma_tables.hpp"

#include <cmath>

namespace gtp {

namespace {

const double kTwoPi = 6.283185307179586476925286766559;

template <int L>
std::vector<uint16_t> index_images(int k1, int k2, int ko) {
  using G = MfmaGeo<L>;
  constexpr int K = (L + 1) * (L + 1);
  const int kk = ko < K ? ko : K;
  std::vector<uint16_t> v(size_t(G::NTH) * (G::GATHER + 2 * G::SCATTER), 0);
  for (int tid = 0; tid < G::NTH; ++tid) {
    const int q = tid / 64, g = tid % 64 / 16, i = tid % 16;
    const int p = i >> 2, ti = (i >> 1) & 1, cs = i & 1, kr = ti ? k2 : k1;
    auto element = [&](int l, int ms) {
      const int k = l * l + l + ms;
      return uint16_t(4 * (l <= L && k < kr ? (ti ? 4 * K + p * k2 : p * k1) + k : 8 * K));
    };
    auto result = [&](int l, int ms) {
      const int k = l * l + l + ms;
      return uint16_t(4 * (l <= L && k < kk ? g * kk + k : 4 * K));
    };
    uint16_t* const a = &v[size_t(tid) * G::GATHER];
    uint16_t* const o = &v[size_t(G::NTH) * G::GATHER + size_t(tid) * 2 * G::SCATTER];
    for (int mi = 0; mi < 4; ++mi)
      for (int par = 0; par < 2; ++par) {
        const int m = G::order(q, mi), c = 2 * mi + par, l = m + par + 2 * i;
        for (int s = 0; s < G::steps(mi); ++s)
          a[G::step0(mi, par) + s] = element(m + par + 2 * (4 * s + g), cs ? -m : m);
        o[2 * c] = result(l, m);
        o[2 * c + 1] = result(l, -m);
      }
    // m = 0: no sin part
    for (int s = 0; s < G::NS0; ++s)
      a[G::NSTEP + s] = cs ? uint16_t(4 * 8 * K) : element(2 * (4 * s + g) + q % 2, 0);
    const int x = q < G::NPART ? q : G::NPART - 1;
    o[16] = result(x < G::NE0 ? 2 * (16 * x + i) : 2 * (16 * (x - G::NE0) + i) + 1, 0);
  }
  return v;
}

template <int L>
MfmaImages images(const Tables& t) {
  using G = MfmaGeo<L>;
  MfmaImages r;
  r.f.assign(G::FLOATS, 0.0);
  r.h.assign(G::HALVES, 0);
  auto part_of = [](double x, int part) {
    const uint16_t h1 = half_bits(x);
    return part == 0 ? h1 : half_bits(x - half_value(h1));
  };
  auto S = [&](int l, int m, int j) { return l <= L ? t.S[size_t(tri(l, m)) * t.NJ + j] : 0.0; };
  constexpr double kW = 1.0 / (G::PHI * G::PHI * G::PHI);
  auto W = [&](int l, int m, int j) { return l <= L ? kW * t.W[size_t(tri(l, m)) * t.NJ + j] : 0.0; };
  double wmax = 0.0;
  for (int l = 0; l <= L; ++l)
    for (int m = 0; m <= l; ++m)
      for (int j = 1; j <= L; ++j) wmax = std::fmax(wmax, std::fabs(W(l, m, j)));
  int ex = 0;
  std::frexp(wmax, &ex);  // wmax in [2^(ex - 1), 2^ex)
  r.kw = 11 - ex;
  const double wscale = std::ldexp(1.0, r.kw);
  auto trig = [&](bool sine, int m, int k) {
    const double a = kTwoPi * double((int64_t(m) * k) % G::NP) / G::NP;
    return G::PHI * (sine ? std::sin(a) : std::cos(a));
  };
  for (int lane = 0; lane < 64; ++lane) {
    const int g = lane / 16, i = lane % 16;
    for (int tile = 0; tile < G::NPT; ++tile)
      for (int q = 0; q < G::NQ; ++q)
        for (int mi = 0; mi < 4; ++mi)
          for (int par = 0; par < 2; ++par)
            for (int s = 0; s < G::steps(mi); ++s) {
              const int f = G::step0(mi, par) + s, m = G::order(q, mi);
              r.f[G::SA + ((size_t(tile * G::NQ + q) * G::SAV + f / 4) * 64 + lane) * 4 + f % 4] =
                  S(m + par + 2 * (4 * s + g), m, 16 * tile + i + 1);
            }
    for (int task = 0; task < G::NT0; ++task)
      for (int s = 0; s < G::NS0; ++s) {
        const int l = 2 * (4 * s + g) + task % 2;
        const bool pole = task >= 2 * G::NPT;
        r.f[G::S0 + ((size_t(task) * G::S0V + s / 4) * 64 + lane) * 4 + s % 4] =
            pole ? (i == 0 ? S(l, 0, 0) : 0.0) : G::PHI * S(l, 0, 16 * (task / 2) + i + 1);
      }
    for (int j = 0; j < 8; ++j) {
      auto put = [&](int base, int frag, uint16_t h) { r.h[size_t(base) + (size_t(frag) * 64 + lane) * 8 + j] = h; };
      for (int type = 0; type < 4; ++type) {
        const bool sine = type >= 2, odd = type & 1;
        for (int mb = 0; mb < G::NMB; ++mb) {
          const int k = 16 * mb + i;
          const int slot = L == 16 ? g & 1 : g, part = L == 16 ? g >> 1 : j / 4;
          const int m = G::order(odd ? slot : G::NSL + slot, j % 4);
          put(G::TP, type * G::NMB + mb, k <= G::Q ? part_of(trig(sine, m, k), part) : 0);
        }
        for (int im = 0; im < G::TAI; ++im) {
          const int k = L == 16 ? 4 * g + j % 4 : 16 * (j / 4) + 4 * g + j % 4;
          const int part = L == 16 ? j / 4 : im, a = i / 4, b = i % 4;
          int m = 2 * (4 * b + a) + (odd ? 1 : 2);
          if (L == 16 && b >= 2) m = (i == 2 && type == 0) ? 0 : L + 1;
          const double w = (k == 0 || k == G::Q) ? 0.5 : 1.0;
          put(G::TA, type * G::TAI + im, (m <= L && k <= G::Q) ? part_of(w * trig(sine, m, k), part) : 0);
        }
      }
      for (int im = 0; im < G::WPARTS; ++im) {
        const int pair = (L == 16 ? 8 * (g & 1) : 8 * g) + j + 1, part = L == 16 ? g >> 1 : im;
        for (int q = 0; q < G::NQ; ++q)
          for (int c = 0; c < 8; ++c) {
            const int m = G::order(q, c / 2);
            put(G::WC, (q * 8 + c) * G::WPARTS + im, part_of(wscale * W(m + c % 2 + 2 * i, m, pair), part));
          }
        for (int x = 0; x < G::NPART; ++x) {
          const int l = x < G::NE0 ? 2 * (16 * x + i) : 2 * (16 * (x - G::NE0) + i) + 1;
          put(G::W0, x * G::WPARTS + im, part_of(wscale * W(l, 0, pair), part));
        }
      }
    }
  }
  return r;
}

}  // namespace

uint16_t half_bits(double v) {
  const uint16_t sign = std::signbit(v) ? 0x8000 : 0;
  const double a = std::fabs(v);
  if (a == 0.0) return sign;
  if (!(a < 65520.0)) return uint16_t(sign | 0x7c00);
  int ex = 0;
  std::frexp(a, &ex);                       // a in [2^(ex - 1), 2^ex)
  const int e = ex - 1 < -14 ? -14 : ex - 1;  // exponent of the format's binade (subnormals: -14)
  const double q = std::nearbyint(std::ldexp(a, 10 - e));  // multiples of 2^(e - 10), ties to even
  // q = 1024 .. 2048 (normal) or 0 .. 1024 (subnormal binade); a carry moves
  // into the exponent by itself
  const int bits = int(q) + (e + 14) * 1024;
  return uint16_t(sign | uint16_t(bits));
}

double half_value(uint16_t h) {
  const int e = (h >> 10) & 31, f = h & 1023;
  const double a = e == 0 ? std::ldexp(double(f), -24) : std::ldexp(double(f + 1024), e - 25);
  return (h & 0x8000) ? -a : a;
}

MfmaImages build_mfma_images(const Tables& t) {
  if (t.L1 != t.L2 || t.L1 != t.Lout) return {};
  if (t.L1 == 16) return images<16>(t);
  if (t.L1 == 32) return images<32>(t);
  return {};
}

std::vector<uint16_t> build_mfma_index(int L, int k1, int k2, int ko) {
  return L == 16 ? index_images<16>(k1, k2, ko) : index_images<32>(k1, k2, ko);
}

}  // namespace gtp
