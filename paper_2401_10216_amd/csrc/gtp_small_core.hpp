// The thread-per-product core of small degrees (gtp_small.hip, gtp_wbwd.hip):
// one lane's Gaunt tensor product from its input accessors into its
// registers, and the loads and stores of a wave's rows.
#pragma once

#include <type_traits>
#include <utility>

#include "gtp_ct.hpp"
#include "gtp_device.hpp"

// Scheduling fence between the per-node stages: keeps the two mirror nodes
// from being interleaved (which costs registers) and keeps the table
// prefetch behind the LDS reads it would otherwise make wait.
#define GTP_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

namespace gtp {
namespace {

constexpr int ctri(int l, int m) { return l * (l + 1) / 2 + m; }
// degree of coefficient index i = l*l + l + m
constexpr int cdeg(int i) {
  int l = 0;
  while ((l + 1) * (l + 1) <= i) ++l;
  return l;
}
constexpr int csh(int L) { return (L + 1) * (L + 1); }
constexpr int cmin(int a, int b) { return a < b ? a : b; }
constexpr int cmax(int a, int b) { return a > b ? a : b; }
// LDS row stride of K-float rows that each lane reads or writes as its own
// row: odd, so that one column of the 64 lanes' rows falls in 64 distinct
// banks.  K = (L + 1)^2 is even (a multiple of 4) for odd L, where a stride
// of K put every lane's element i in one bank.
constexpr int lds_stride(int k) { return k | 1; }

// Coefficient accessors of one lane's input vector: in registers, or a row of
// the workgroup's LDS tile.  touch() makes the LDS row offset opaque so the
// reads stay inside the node loop instead of being hoisted into registers.
template <int K>
struct RegX {
  float (&a)[K];
  template <class I>
  __device__ __forceinline__ float operator()(I) const { return a[I::value]; }
  __device__ __forceinline__ void touch() {}
};
struct LdsX {
  const float* tile;
  int off;
  template <class I>
  __device__ __forceinline__ float operator()(I) const { return tile[off + I::value]; }
  __device__ __forceinline__ void touch() { asm volatile("" : "+v"(off)); }
};

__device__ __forceinline__ float ld_in(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ld_in(const uint16_t* p, int64_t i) {
  return __uint_as_float(uint32_t(p[i]) << 16);
}

// phi grid p_k = 2 pi k / NP with NP = 4Q.  The points k, -k, 2Q + k, 2Q - k
// share |cos(m p)| and |sin(m p)|, with signs set by the parity of m, so both
// transforms work on the quarter 0 <= k <= Q and fan out.

// a += s x, or a = s x for the first term of a sum: a multiply-add onto a
// zero cannot drop the addend (signed zeros), and its three-operand form
// cannot carry a literal constant.  The first product is kept out of
// multiply-add fusion for the same reason (x s - y needs that form too).
template <bool FIRST>
__device__ __forceinline__ void mac(float& a, float s, float x) {
  if constexpr (FIRST) {
#pragma clang fp contract(off)
    a = s * x;
  } else {
    a = fmaf(s, x, a);
  }
}

// Whether m is the first degree of its parity (m >= 1) with a non-zero
// cos (S = false) or sin (S = true) twiddle at sample k: the first term of a
// phi-synthesis partial sum.
constexpr bool first_m(int m, long long k, int NP, bool S) {
  for (int mm = (m % 2 == 0) ? 2 : 1; mm < m; mm += 2) {
    const float v = S ? ct_round(ct_sin2pi(mm * k, NP)) : ct_round(ct_cos2pi(mm * k, NP));
    if (v != 0.0f) return false;
  }
  return true;
}
// Whether k is the first sample with a non-zero cos / sin twiddle of degree
// m: the first term of a phi-analysis sum.
constexpr bool first_k(int m, int k, int NP, bool S) {
  for (int kk = 0; kk < k; ++kk) {
    const float v = S ? ct_round(ct_sin2pi((long long)m * kk, NP)) : ct_round(ct_cos2pi((long long)m * kk, NP));
    if (v != 0.0f) return false;
  }
  return true;
}

// F[k] = A0 + sum_m A[2m-1] cos(m p_k) + A[2m] sin(m p_k), k < NP, for a
// function of phi-degree <= M.
template <int M, int NP>
__device__ __forceinline__ void phi_synth(const float (&A)[2 * M + 1], float (&F)[NP]) {
  static_assert(NP % 4 == 0, "phi grid size must be a multiple of 4");
  constexpr int Q = NP / 4;
  cfor<0, Q + 1>([&](auto KK) {
    constexpr int k = decltype(KK)::value;
    // partial sums over even / odd m of the cos and sin parts
    float pe = A[0], po = 0.0f, qe = 0.0f, qo = 0.0f;
    cfor<1, M + 1>([&](auto MM) {
      constexpr int m = decltype(MM)::value;
      constexpr float c = ct_round(ct_cos2pi((long long)m * k, NP));
      constexpr float sn = ct_round(ct_sin2pi((long long)m * k, NP));
      if constexpr (m % 2 == 0) {
        if constexpr (c != 0.0f) pe = fmaf(A[2 * m - 1], c, pe);
        if constexpr (sn != 0.0f) mac<first_m(m, k, NP, true)>(qe, sn, A[2 * m]);
      } else {
        if constexpr (c != 0.0f) mac<first_m(m, k, NP, false)>(po, c, A[2 * m - 1]);
        if constexpr (sn != 0.0f) mac<first_m(m, k, NP, true)>(qo, sn, A[2 * m]);
      }
    });
    if constexpr (k == 0) {
      F[0] = pe + po;
      F[2 * Q] = pe - po;
    } else if constexpr (k == Q) {
      F[Q] = pe + qo;  // cos(odd m pi/2) = sin(even m pi/2) = 0
      F[3 * Q] = pe - qo;
    } else if constexpr (M == 1) {
      // two roundings a sample where the class sums take four: with so few terms
      // the powers of L = 1 show it (fourth power to Lout = 3 against 64 bits
      // 1.63e-7 -> 1.61e-7, with ipow's FINE 1.578e-7; the generic kernel 1.583e-7)
      constexpr float c = ct_round(ct_cos2pi(k, NP)), sn = ct_round(ct_sin2pi(k, NP));
      const float a = fmaf(c, A[1], A[0]), b = fmaf(-c, A[1], A[0]);
      F[k] = fmaf(sn, A[2], a);
      F[NP - k] = fmaf(-sn, A[2], a);
      F[2 * Q + k] = fmaf(-sn, A[2], b);
      F[2 * Q - k] = fmaf(sn, A[2], b);
    } else {
      const float s1 = pe + po, d1 = pe - po, s2 = qe + qo, d2 = qe - qo;
      F[k] = s1 + s2;
      F[NP - k] = s1 - s2;
      F[2 * Q + k] = d1 + d2;
      F[2 * Q - k] = d1 - d2;
    }
  });
}

// C[0] = sum_k F_k, C[2m-1] = sum_k F_k cos(m p_k), C[2m] = sum_k F_k sin(m p_k), m <= MO.
template <int MO, int NP>
__device__ __forceinline__ void phi_analysis(const float (&F)[NP], float (&C)[2 * MO + 1]) {
  static_assert(NP % 4 == 0, "phi grid size must be a multiple of 4");
  constexpr int Q = NP / 4;
  cfor<0, 2 * MO + 1>([&](auto I) { C[decltype(I)::value] = 0.0f; });
  cfor<0, Q + 1>([&](auto KK) {
    constexpr int k = decltype(KK)::value;
    // even-m / odd-m folds of the four points sharing this quarter angle
    float ce, co, se = 0.0f, so = 0.0f;
    if constexpr (k == 0) {
      ce = F[0] + F[2 * Q];
      co = F[0] - F[2 * Q];
    } else if constexpr (k == Q) {
      ce = F[Q] + F[3 * Q];
      co = 0.0f;
      so = F[Q] - F[3 * Q];
    } else {
      const float a = F[k] + F[NP - k], b = F[2 * Q + k] + F[2 * Q - k];
      const float d = F[k] - F[NP - k], e = F[2 * Q + k] - F[2 * Q - k];
      ce = a + b;
      co = a - b;
      se = d + e;
      so = d - e;
    }
    cfor<0, MO + 1>([&](auto MM) {
      constexpr int m = decltype(MM)::value;
      constexpr float c = ct_round(ct_cos2pi((long long)m * k, NP));
      constexpr float sn = ct_round(ct_sin2pi((long long)m * k, NP));
      constexpr int ic = m == 0 ? 0 : 2 * m - 1;
      if constexpr (c != 0.0f) mac<first_k(m, k, NP, false)>(C[ic], c, (m % 2 == 0) ? ce : co);
      if constexpr (m > 0 && sn != 0.0f) mac<first_k(m, k, NP, true)>(C[2 * m], sn, (m % 2 == 0) ? se : so);
    });
  });
}

// Theta synthesis at the mirror pair (t_j, t_{NT-j}) of one input of degree
// L: even-parity and odd-parity (l + m) partial sums give both nodes.  x(I)
// returns coefficient I; ST row j holds Theta_lm(t_j) for all (l, m).
template <int L, typename X, typename T>
__device__ __forceinline__ void theta_synth_pair(X x, const T& Sj, float (&Aj)[2 * L + 1],
                                                 float (&Ajp)[2 * L + 1]) {
  cfor<0, L + 1>([&](auto MM) {
    constexpr int m = decltype(MM)::value;
    float ec = 0.0f, oc = 0.0f, es = 0.0f, os = 0.0f;
    cfor<m, L + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      const float sv = Sj[ctri(l, m)];
      if constexpr ((l + m) % 2 == 0) {
        mac<l == m>(ec, sv, x(std::integral_constant<int, l * l + l + m>{}));
        if constexpr (m > 0) mac<l == m>(es, sv, x(std::integral_constant<int, l * l + l - m>{}));
      } else {
        mac<l == m + 1>(oc, sv, x(std::integral_constant<int, l * l + l + m>{}));
        if constexpr (m > 0) mac<l == m + 1>(os, sv, x(std::integral_constant<int, l * l + l - m>{}));
      }
    });
    if constexpr (m == 0) {
      Aj[0] = ec + oc;
      Ajp[0] = ec - oc;
    } else {
      Aj[2 * m - 1] = ec + oc;
      Ajp[2 * m - 1] = ec - oc;
      Aj[2 * m] = es + os;
      Ajp[2 * m] = es - os;
    }
  });
}

// Theta synthesis at one node of the mirror pair: MIRROR = false gives t_j,
// MIRROR = true gives t_{NT-j} (Theta_lm picks up (-1)^(l+m)).
template <int L, bool MIRROR, typename X, typename T>
__device__ __forceinline__ void theta_synth_node(X x, const T& Sj, float (&A)[2 * L + 1]) {
  cfor<0, L + 1>([&](auto MM) {
    constexpr int m = decltype(MM)::value;
    float ec = 0.0f, es = 0.0f;
    cfor<m, L + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      const float sv = (MIRROR && (l + m) % 2) ? -Sj[ctri(l, m)] : Sj[ctri(l, m)];
      mac<l == m>(ec, sv, x(std::integral_constant<int, l * l + l + m>{}));
      if constexpr (m > 0) mac<l == m>(es, sv, x(std::integral_constant<int, l * l + l - m>{}));
    });
    if constexpr (m == 0) {
      A[0] = ec;
    } else {
      A[2 * m - 1] = ec;
      A[2 * m] = es;
    }
  });
}

// acc += W(t_j) * C for the moments C of one node; MIRROR uses the weights of
// t_{NT-j}, which are (-1)^(l+m) times those of t_j.  FIRST: the first node
// with m > 0 terms (acc holds only the poles' m = 0 terms).
template <int LE, bool MIRROR, typename T, bool FIRST = false>
__device__ __forceinline__ void theta_analysis_node(const T& Wj, const float (&C)[2 * LE + 1],
                                                    float (&acc)[(LE + 1) * (LE + 1)]) {
  cfor<0, LE + 1>([&](auto MM) {
    constexpr int m = decltype(MM)::value;
    cfor<m, LE + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      const float w = (MIRROR && (l + m) % 2) ? -Wj[ctri(l, m)] : Wj[ctri(l, m)];
      mac<(FIRST && m > 0)>(acc[l * l + l + m], w, C[m == 0 ? 0 : 2 * m - 1]);
      if constexpr (m > 0) mac<FIRST>(acc[l * l + l - m], w, C[2 * m]);
    });
  });
}

// Theta synthesis at the equator (only even l + m survive).
template <int L, typename X>
__device__ __forceinline__ void theta_synth_eq(X x, const float* __restrict__ Sj, float (&A)[2 * L + 1]) {
  cfor<0, L + 1>([&](auto MM) {
    constexpr int m = decltype(MM)::value;
    float ec = 0.0f, es = 0.0f;
    cfor<m, L + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      if constexpr ((l + m) % 2 == 0) {
        const float sv = Sj[ctri(l, m)];
        ec = fmaf(sv, x(std::integral_constant<int, l * l + l + m>{}), ec);
        if constexpr (m > 0) es = fmaf(sv, x(std::integral_constant<int, l * l + l - m>{}), es);
      }
    });
    if constexpr (m == 0) {
      A[0] = ec;
    } else {
      A[2 * m - 1] = ec;
      A[2 * m] = es;
    }
  });
}

// v^NU; FINE: the fourth power takes the square's rounding along.
template <int NU, bool FINE = false>
__device__ __forceinline__ float ipow(float v) {
  if constexpr (NU == 1) {
    return v;
  } else if constexpr (NU == 4 && FINE) {
    const float h = v * v, e = fmaf(v, v, -h);
    return fmaf(h + h, e, h * h);
  } else if constexpr (NU % 2 == 0) {
    const float h = ipow<NU / 2>(v);
    return h * h;
  } else {
    return v * ipow<NU - 1>(v);
  }
}

// Quarter-angle class sums of a function of phi-degree <= M at sample k:
// pe / po = sum over even / odd m of A_cos(m) cos(m p_k) (pe with A0), qe / qo
// the same for the sin parts.  The samples at k, NP - k, 2Q + k, 2Q - k are
// pe + po +- (qe + qo) and pe - po +- (qe - qo).
template <int M, int NP, int k>
__device__ __forceinline__ void phi_classes(const float (&A)[2 * M + 1], float& pe, float& po, float& qe,
                                            float& qo) {
  pe = A[0];
  po = qe = qo = 0.0f;
  cfor<1, M + 1>([&](auto MM) {
    constexpr int m = decltype(MM)::value;
    constexpr float c = ct_round(ct_cos2pi((long long)m * k, NP));
    constexpr float sn = ct_round(ct_sin2pi((long long)m * k, NP));
    if constexpr (m % 2 == 0) {
      if constexpr (c != 0.0f) pe = fmaf(A[2 * m - 1], c, pe);
      if constexpr (sn != 0.0f) mac<first_m(m, k, NP, true)>(qe, sn, A[2 * m]);
    } else {
      if constexpr (c != 0.0f) mac<first_m(m, k, NP, false)>(po, c, A[2 * m - 1]);
      if constexpr (sn != 0.0f) mac<first_m(m, k, NP, true)>(qo, sn, A[2 * m]);
    }
  });
}

// One node, product of two functions: the phi moments m <= LE of f g from
// the class sums of f and g.  Summed over the four points of a quarter angle
// (the grid's p -> -p, pi -+ p symmetry), f g folds to
//   even-m cos: 4 (pe pe' + po po' + qe qe' + qo qo'),
//   odd-m cos:  4 (pe po' + po pe' + qe qo' + qo qe'),
//   even-m sin: 4 (pe qe' + po qo' + qe pe' + qo po'),
//   odd-m sin:  4 (pe qo' + po qe' + qe po' + qo pe')
// (2 and two points at k = 0 and k = Q), so no sample is formed; the factor
// goes into the analysis twiddles.
template <int L1, int L2, int LE, int NP>
__device__ __forceinline__ void node_product_cls(const float (&A)[2 * L1 + 1], const float (&B)[2 * L2 + 1],
                                                 float (&C)[2 * LE + 1]) {
  static_assert(NP % 4 == 0, "phi grid size must be a multiple of 4");
  constexpr int Q = NP / 4;
  cfor<0, 2 * LE + 1>([&](auto I) { C[decltype(I)::value] = 0.0f; });
  cfor<0, Q + 1>([&](auto KK) {
    constexpr int k = decltype(KK)::value;
    float pe, po, qe, qo, pf, pg, qf, qg;  // f: pe po qe qo; g: pf pg qf qg
    phi_classes<L1, NP, k>(A, pe, po, qe, qo);
    phi_classes<L2, NP, k>(B, pf, pg, qf, qg);
    float ce, co = 0.0f, se = 0.0f, so = 0.0f;
    constexpr float fac = (k == 0 || k == Q) ? 2.0f : 4.0f;
    if constexpr (k == 0) {
      ce = fmaf(po, pg, pe * pf);
      co = fmaf(po, pf, pe * pg);
    } else if constexpr (k == Q) {
      ce = fmaf(qo, qg, pe * pf);
      so = fmaf(qo, pf, pe * qg);
    } else {
      ce = fmaf(qo, qg, fmaf(qe, qf, fmaf(po, pg, pe * pf)));
      co = fmaf(qo, qf, fmaf(qe, qg, fmaf(po, pf, pe * pg)));
      se = fmaf(qo, pg, fmaf(qe, pf, fmaf(po, qg, pe * qf)));
      so = fmaf(qo, pf, fmaf(qe, pg, fmaf(po, qf, pe * qg)));
    }
    cfor<0, LE + 1>([&](auto MM) {
      constexpr int m = decltype(MM)::value;
      constexpr float c = ct_round(ct_cos2pi((long long)m * k, NP));
      constexpr float sn = ct_round(ct_sin2pi((long long)m * k, NP));
      constexpr int ic = m == 0 ? 0 : 2 * m - 1;
      if constexpr (c != 0.0f) mac<first_k(m, k, NP, false)>(C[ic], fac * c, (m % 2 == 0) ? ce : co);
      if constexpr (m > 0 && sn != 0.0f) mac<first_k(m, k, NP, true)>(C[2 * m], fac * sn, (m % 2 == 0) ? se : so);
    });
  });
}

// One node: the phi moments m <= LE of the product of two functions (from
// their class sums), or of a power of one function (through its samples).
template <int L1, int L2, int LE, int NP, int NU>
__device__ __forceinline__ void node_product(const float (&A)[2 * L1 + 1], const float (&B)[2 * L2 + 1],
                                             float (&C)[2 * LE + 1]) {
  if constexpr (NU == 0) {
    node_product_cls<L1, L2, LE, NP>(A, B, C);
  } else {
    float F[NP];
    phi_synth<L1, NP>(A, F);
    cfor<0, NP>([&](auto KK) { F[decltype(KK)::value] = ipow<NU, L1 == 1>(F[decltype(KK)::value]); });
    phi_analysis<LE, NP>(F, C);
  }
}

// Degree bookkeeping of one product stage.  NU = 0: x1 (deg L1) times x2
// (deg L2); NU >= 2: x1^NU (L2 unused).
template <int L1, int L2, int LO, int NU>
struct Geo {
  static constexpr int U = NU == 0 ? L1 + L2 : NU * L1;
  static constexpr int LE = cmin(LO, U);
  static constexpr int NT = U + 1;
  static constexpr int NJ = NT + 1;
  static constexpr int NP = (U + LE + 1 + 3) / 4 * 4;  // same rule as the host tables
  static constexpr int KE = csh(LE);
};

// Compile-time copies of the node-major S and W rows of the equal-degree
// triples L1 = L2 = Lout = 1..8 (SmallConsts<L>::S[j][tri(l, m)], ::W[j][..]),
// generated at build time from the same fp64 builder and fp32 rounding as a
// plan's device tables.  Read with constant indices they become instruction
// literals: a VALU instruction with a literal operand issues at the rate of
// an all-VGPR one, one with a scalar-register operand at about half of it.
#include "gtp_small_consts.inc"

template <int L, int J, bool IS_W>
struct LitRow {
  __device__ __forceinline__ constexpr float operator[](int i) const {
    return IS_W ? SmallConsts<L>::W[J][i] : SmallConsts<L>::S[J][i];
  }
};

template <int L1, int L2, int LO, int NU>
constexpr bool lit_tables() {
  return NU == 0 && L1 == L2 && L2 == LO && L1 >= 1 && L1 <= 8;
}

// gtp_core for L1 = L2 = Lout = L with the tables as literals: the node-pair
// loop is unrolled at compile time (NT = 2 L + 1 is odd: no equator node).
template <int L, typename XA, typename XB>
__device__ __forceinline__ void gtp_core_lit(XA xa, XB xb, float (&acc)[(L + 1) * (L + 1)]) {
  using G = Geo<L, L, L, 0>;
  constexpr int NT = G::NT, NP = G::NP;
  static_assert(NT % 2 == 1, "equal degrees give an odd node count");
  cfor<0, G::KE>([&](auto I) { acc[decltype(I)::value] = 0.0f; });
  {
    // poles: only m = 0 is non-zero and all phi samples are equal
    constexpr LitRow<L, 0, false> S0{};
    constexpr LitRow<L, 0, true> W0{};
    float ae = 0.0f, ao = 0.0f, be = 0.0f, bo = 0.0f;
    cfor<0, L + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      if constexpr (l % 2 == 0) {
        mac<l == 0>(ae, S0[ctri(l, 0)], xa(std::integral_constant<int, l * l + l>{}));
        mac<l == 0>(be, S0[ctri(l, 0)], xb(std::integral_constant<int, l * l + l>{}));
      } else {
        mac<l == 1>(ao, S0[ctri(l, 0)], xa(std::integral_constant<int, l * l + l>{}));
        mac<l == 1>(bo, S0[ctri(l, 0)], xb(std::integral_constant<int, l * l + l>{}));
      }
    });
    const float fn = (ae + ao) * (be + bo), fs = (ae - ao) * (be - bo);
    const float ce = float(NP) * (fn + fs), co = float(NP) * (fn - fs);
    cfor<0, L + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      acc[l * l + l] = W0[ctri(l, 0)] * ((l % 2 == 0) ? ce : co);
    });
  }
  cfor<1, (NT + 1) / 2>([&](auto JJ) {
    constexpr int j = decltype(JJ)::value;
    constexpr LitRow<L, j, false> Sj{};
    constexpr LitRow<L, j, true> Wj{};
    xa.touch();
    xb.touch();
    float Aj[2 * L + 1], Ajp[2 * L + 1], Bj[2 * L + 1];
    theta_synth_pair<L>(xa, Sj, Aj, Ajp);
    theta_synth_node<L, false>(xb, Sj, Bj);
    GTP_SCHED_FENCE();
    {
      float C[2 * L + 1];
      node_product<L, L, L, NP, 0>(Aj, Bj, C);
      theta_analysis_node<L, false, LitRow<L, j, true>, j == 1>(Wj, C, acc);
    }
    GTP_SCHED_FENCE();
    {
      theta_synth_node<L, true>(xb, Sj, Bj);
      float C[2 * L + 1];
      node_product<L, L, L, NP, 0>(Ajp, Bj, C);
      theta_analysis_node<L, true>(Wj, C, acc);
    }
    GTP_SCHED_FENCE();
  });
}

// acc (degree <= LE) = product of xa and xb (or xa^NU) for one lane.
// xa(I), xb(I) return input coefficient I; ST / WT are the node-major
// synthesis and analysis tables with row lengths ntS / ntW (for equal degrees
// 1..8 the compile-time copies are used instead).
template <int L1, int L2, int LO, int NU, typename XA, typename XB>
__device__ __forceinline__ void gtp_core(XA xa, XB xb, float (&acc)[Geo<L1, L2, LO, NU>::KE],
                                         const float* __restrict__ ST, int ntS, const float* __restrict__ WT,
                                         int ntW) {
  if constexpr (lit_tables<L1, L2, LO, NU>()) {
    gtp_core_lit<L1>(xa, xb, acc);
    return;
  }
  using G = Geo<L1, L2, LO, NU>;
  constexpr int LE = G::LE, NT = G::NT, NP = G::NP;
  cfor<0, G::KE>([&](auto I) { acc[decltype(I)::value] = 0.0f; });

  // Poles (t = 0 and t = pi): only m = 0 is non-zero; the phi samples are all
  // equal, so the m = 0 moment is NP times the product value.
  {
    float ae = 0.0f, ao = 0.0f, be = 0.0f, bo = 0.0f;
    cfor<0, L1 + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      const float sv = ST[ctri(l, 0)];
      if constexpr (l % 2 == 0) ae = fmaf(sv, xa(std::integral_constant<int, l * l + l>{}), ae);
      else ao = fmaf(sv, xa(std::integral_constant<int, l * l + l>{}), ao);
    });
    float fn, fs;
    if constexpr (NU == 0) {
      cfor<0, L2 + 1>([&](auto LL) {
        constexpr int l = decltype(LL)::value;
        const float sv = ST[ctri(l, 0)];
        if constexpr (l % 2 == 0) be = fmaf(sv, xb(std::integral_constant<int, l * l + l>{}), be);
        else bo = fmaf(sv, xb(std::integral_constant<int, l * l + l>{}), bo);
      });
      fn = (ae + ao) * (be + bo);
      fs = (ae - ao) * (be - bo);
    } else {
      fn = ipow<NU, L1 == 1>(ae + ao);
      fs = ipow<NU, L1 == 1>(ae - ao);
    }
    const float ce = float(NP) * (fn + fs), co = float(NP) * (fn - fs);
    cfor<0, LE + 1>([&](auto LL) {
      constexpr int l = decltype(LL)::value;
      const float w = WT[ctri(l, 0)];
      acc[l * l + l] = fmaf(w, (l % 2 == 0) ? ce : co, acc[l * l + l]);
    });
  }

  // Interior mirror pairs (j, NT - j), 1 <= j < NT / 2 (runtime tables:
  // degree triples without compile-time constants).
  // The node-pair tables are software-pipelined through scalar registers:
  // S of pair j + 1 and W of pair j are requested after the first LDS reads
  // of pair j (LDS reads share the scalar loads' wait counter) and arrive
  // while the phi transforms of pair j run.
  constexpr int NS = ctri(cmax(L1, L2), cmax(L1, L2)) + 1;
  constexpr int NW = ctri(LE, LE) + 1;
  float scur[NS];
  cfor<0, NS>([&](auto I) { scur[decltype(I)::value] = ST[ntS + decltype(I)::value]; });
  for (int j = 1; 2 * j < NT; ++j) {
    xa.touch();
    xb.touch();
    // x1 at both mirror nodes from shared even / odd partial sums; x2 node by
    // node (fewer live registers), its first node before the table prefetch
    float Aj[2 * L1 + 1], Ajp[2 * L1 + 1];
    float Bj[2 * L2 + 1];
    theta_synth_pair<L1>(xa, scur, Aj, Ajp);
    if constexpr (NU == 0) theta_synth_node<L2, false>(xb, scur, Bj);
    GTP_SCHED_FENCE();
    float sb[NS];
    cfor<0, NS>([&](auto I) { sb[decltype(I)::value] = scur[decltype(I)::value]; });
    // row j + 1 always exists (j + 1 <= NT), even when it is not used
    const float* Sn = ST + (j + 1) * ntS;
    cfor<0, NS>([&](auto I) { scur[decltype(I)::value] = Sn[decltype(I)::value]; });
    const float* Wj = WT + j * ntW;
    float wcur[NW];
    cfor<0, NW>([&](auto I) { wcur[decltype(I)::value] = Wj[decltype(I)::value]; });
    GTP_SCHED_FENCE();
    {
      float C[2 * LE + 1];
      node_product<L1, L2, LE, NP, NU>(Aj, Bj, C);
      theta_analysis_node<LE, false>(wcur, C, acc);
    }
    GTP_SCHED_FENCE();
    {
      if constexpr (NU == 0) theta_synth_node<L2, true>(xb, sb, Bj);
      float C[2 * LE + 1];
      node_product<L1, L2, LE, NP, NU>(Ajp, Bj, C);
      theta_analysis_node<LE, true>(wcur, C, acc);
    }
    GTP_SCHED_FENCE();
  }

  // Equator node when NT is even.
  if constexpr (NT % 2 == 0) {
    constexpr int j = NT / 2;
    const float* Sj = ST + j * ntS;
    const float* Wj = WT + j * ntW;
    float A[2 * L1 + 1], B[2 * L2 + 1];
    theta_synth_eq<L1>(xa, Sj, A);
    if constexpr (NU == 0) theta_synth_eq<L2>(xb, Sj, B);
    float Cq[2 * LE + 1];
    node_product<L1, L2, LE, NP, NU>(A, B, Cq);
    cfor<0, LE + 1>([&](auto MM) {
      constexpr int m = decltype(MM)::value;
      cfor<m, LE + 1>([&](auto LL) {
        constexpr int l = decltype(LL)::value;
        if constexpr ((l + m) % 2 == 0) {
          const float w = Wj[ctri(l, m)];
          acc[l * l + l + m] = fmaf(w, Cq[m == 0 ? 0 : 2 * m - 1], acc[l * l + l + m]);
          if constexpr (m > 0) acc[l * l + l - m] = fmaf(w, Cq[2 * m], acc[l * l + l - m]);
        }
      });
    });
  }
}

constexpr int kTile = 64;  // products per workgroup (one wave)
// Waves per SIMD the register budget is sized for: x1 and the accumulators
// stay in registers, so the budget shrinks with the degree.
constexpr int small_waves(int L1, int L2, int LO) { return (L1 > 6 || L2 > 6 || LO > 6) ? 2 : 3; }

// Row tid (product p0 + tid, the last one for lanes past the end) of x into
// registers, each lane loading its own row.
template <int K, typename TIn>
__device__ __forceinline__ void load_rows(const TIn* __restrict__ x, int64_t p0, int cnt, float (&r)[K]) {
  const int tid = threadIdx.x;
  const TIn* const xr = x + (p0 + (tid < cnt ? tid : cnt - 1)) * K;
  cfor<0, K>([&](auto I) { r[decltype(I)::value] = ld_in(xr, decltype(I)::value); });
}

template <int KO, int KE>
__device__ __forceinline__ void store_rows(float* __restrict__ y, int64_t p0, int cnt, float* tile,
                                           const float (&acc)[KE], int tid = threadIdx.x) {
  constexpr int SO = lds_stride(KO);
  cfor<0, KO>([&](auto I) {
    constexpr int i = decltype(I)::value;
    tile[tid * SO + i] = (i < KE) ? acc[i < KE ? i : 0] : 0.0f;
  });
  __syncthreads();
  float* out = y + p0 * KO;
  typedef float sv4 __attribute__((ext_vector_type(4)));
  if (cnt == kTile && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    // a full workgroup's rows are 64 KO floats, a whole number of 16-byte
    // runs: 16-byte non-temporal stores (the outputs are not read again:
    // 1.6 % faster at L = 6 than plain stores; non-temporal loads of the
    // input rows, by contrast, measured 1.5x slower)
    constexpr int N4 = kTile * KO / 4;
    if constexpr (SO == KO) {
      // compact rows: the tile (16-byte aligned) is the output's layout
      for (int i = tid; i < N4; i += kTile)
        __builtin_nontemporal_store(reinterpret_cast<const sv4*>(tile)[i], reinterpret_cast<sv4*>(out) + i);
    } else {
      // padded rows; KO is a multiple of 4, so no 16-byte run crosses a row
      static_assert(KO % 4 == 0, "even row lengths are (2m)^2");
      for (int i = tid; i < N4; i += kTile) {
        const int r = (4 * i) / KO, c = 4 * i - r * KO;
        const float* const t = tile + r * SO + c;
        __builtin_nontemporal_store(sv4{t[0], t[1], t[2], t[3]}, reinterpret_cast<sv4*>(out) + i);
      }
    }
  } else {
    for (int i = tid; i < cnt * KO; i += kTile) {
      const int r = i / KO;
      out[i] = tile[r * SO + (i - r * KO)];
    }
  }
}

// Per-degree weights of one lane's product (WGT = true): scale the K values
// at(I) (degrees <= L) by wrow[degree].
template <int L, int K, typename V>
__device__ __forceinline__ void scale_by_degree(const float* __restrict__ wrow, V&& at) {
  float wl[L + 1];
  cfor<0, L + 1>([&](auto LL) { wl[decltype(LL)::value] = wrow[decltype(LL)::value]; });
  cfor<0, K>([&](auto I) { at(I) *= wl[cdeg(decltype(I)::value)]; });
}

// Row tid of a workgroup's products (xr: this lane's row, the last product's
// for lanes past the end) into the LDS tile, row stride lds_stride(K); each
// lane later reads only its own row.  fp32 rows of degree 5..7 with a compact
// tile: when the workgroup is full and the slab is 16-byte aligned (dma), the
// whole slab x + p0 K by coalesced 16-byte loads straight into LDS (lane
// q 64 + tid carries floats 4 (q 64 + tid) .. + 3, no registers on the way;
// the slab is a whole number of 16-byte runs, 64 K floats).  (Measured: 2.4 %
// faster at L = 6; at L = 4 4 % and at L = 8 1 % slower than the per-lane
// loads, so degrees 5..7 only.  Staging x1 the same way, through the tile
// before x2, measured 1 % slower at L = 6.)
template <int L, bool ALLOW_DMA, typename T>
__device__ __forceinline__ void stage_tile_rows(float* tile, const T* __restrict__ x, const T* __restrict__ xr,
                                                int64_t p0, int cnt, int tid, int dma) {
  constexpr int K = csh(L), S = lds_stride(K);
  bool staged = false;
  if constexpr (std::is_same<T, float>::value && ALLOW_DMA && L >= 5 && L <= 7 && S == K) {
    if (dma && cnt == kTile) {
      typedef __attribute__((address_space(3))) void lds_void;
      typedef const __attribute__((address_space(1))) void glb_void;
      constexpr int NF = kTile * K, NQ = (NF + 255) / 256;
      const float* const slab = x + p0 * K;
      cfor<0, NQ>([&](auto Q) {
        constexpr int q = decltype(Q)::value;
        const int e = (q * 64 + tid) * 4;
        if (q + 1 < NQ || e < NF)
          __builtin_amdgcn_global_load_lds((glb_void*)(slab + e), (lds_void*)(tile + q * 256), 16, 0, 0);
      });
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the whole wave's rows are in LDS
      staged = true;
    }
  }
  if (!staged) cfor<0, K>([&](auto I) { tile[tid * S + decltype(I)::value] = ld_in(xr, decltype(I)::value); });
}

}  // namespace
}  // namespace gtp
