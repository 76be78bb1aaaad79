// Fused Gaunt tensor product on the matrix cores with split operands, for
// L1 = L2 = Lout = L in {16, 32} and every triple padded to them (gfx950).
//
// The sampled pipeline of Sec. 3.2 (convolution theorem, theta nodes in
// mirror pairs, 4-fold phi symmetry) with every transform a matrix
// contraction.  The theta synthesis runs on v_mfma_f32_16x16x4_f32; the phi
// transforms and the theta analysis on v_mfma_f32_16x16x32_f16 with split
// operands: a value enters as h1 + h2 (h1 = fp16(v), h2 = fp16(v - h1)), which
// leave at most max(2^-23 |v|, 2^-25) of it: 2^-23 of the value itself from 2^-2
// up, and below it 2^-31 of its input's norm (theta values: 2^-25 against norms
// 2^SE1, 2^SE2), far under the rounding of the sums it enters; against
// tables split the same way, the products accumulating in fp32; everything
// between the contractions stays fp32.  Three or four 16x16x32 fp16
// contractions of 16 cycles replace eight 16x16x4 fp32 ones of 32.  The theta
// values are brought to inputs of norm [1/2, 1) by a power of two, which
// bounds every later intermediate (|F| <= sqrt(K / 4 pi) |x|, the addition
// theorem) within the half type's range, and the output is scaled back.
//
// A workgroup takes four products at a time (the sixteen rows of a theta
// contraction are 4 products x 2 inputs x cos / sin):
//   A  theta synthesis: wave q owns the four orders m of quad q; even and odd
//      degrees apart give the node (sum) and its mirror (difference), split
//      and written to LDS as the phi stage's operand (16 bytes per lane);
//   B  phi stage, wave = (product, 16 node pairs): synthesis of both inputs
//      at the nodes, then at their mirrors, sample products (class sums, no
//      sample formed), analysis; the accumulator layout of the synthesis is
//      the operand layout of the analysis; moments of the pairs (sum,
//      difference) to LDS;
//   C  theta analysis: wave q its quad's orders again, columns = degrees.
// Theta tables are read once per four products, where one wave per product
// read them for each; x comes in by 16-byte loads straight into LDS, the next
// group's issued after B.
//
// Bound: issue of matrix and vector instructions (of the SIMDs' cycles, by
// counters: degree 32 27 % matrix, 42 % vector at four cycles each; 16 and 12 21 to
// 22 % and 56 %), the two seldom at once on a SIMD; the rest is latency between
// the five barriers of a turn, with two (L = 32) and three (L = 16) waves per
// SIMD.  Measured against the fp32 one-wave-per-product kernel it replaced
// (theta stages on the VALU, table reads per product): 262144 products of
// degree 32 3.58 -> 2.59 ms, 2.1M bf16 products of degree 16 5.20 -> 4.60 ms, 191904
// of degree 12 0.479 -> 0.402 ms; error against fp64 (2-norm) 1.67e-7 -> 1.38e-7 at
// 32, 1.35e-7 -> 1.29e-7 at 16, 1.18e-7 -> 1.11e-7 at 12 (1.38e-7 and 1.19e-7 with
// phi tables at scale 1).  (The theta synthesis by split fp16 too measured slower
// at L = 16, its operands' split and scaling costing more than the contractions
// saved, and less exact.)
#include <type_traits>
#include <utility>

#include "gtp_ct.hpp"
#include "gtp_device.hpp"
#include "gtp_mfma_tables.hpp"
#include "gtp_split.hpp"

// Bounds what the scheduler hoists (operand reads hold registers from their
// issue on).
#define GTP_FENCE() __builtin_amdgcn_sched_barrier(0)

namespace gtp {
namespace {

// A slab of n elements into LDS at `to` by the NTH threads of the workgroup,
// straight from memory (no registers on the way), WIDTH bytes per lane and
// load, dividing the slab's size and both addresses.  In assembly: the
// compiler would wait for the loads at the next LDS access of any kind; here
// the caller waits (vmcnt) before the barrier that publishes the slab.  M0
// holds the wave's LDS address, lane l's data go to M0 + WIDTH l.  (M0 is reserved:
// the compiler sets it right before an instruction that needs it, keeps nothing
// in it and takes it in no clobber list; this file's kernels use it nowhere else.)
template <int WIDTH, int NTH, int TRIPS, typename T>
__device__ __forceinline__ void slab_to_lds(const T* s, unsigned char* to, int n, int tid, int wave) {
  typedef __attribute__((address_space(3))) unsigned char lds_char;
  const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((lds_char*)to)) + wave * 64 * WIDTH;
  const int units = n * int(sizeof(T)) / WIDTH;
#pragma unroll
  for (int r = 0; r < TRIPS; ++r) {
    const int u = r * NTH + tid;
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(base + r * NTH * WIDTH), off = u * WIDTH;
    if (u < units) {
      if constexpr (WIDTH == 16) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(off), "s"(s)
                     : "memory");
      } else {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(m0), "v"(off), "s"(s)
                     : "memory");
      }
    }
  }
}
// Any alignment and length: element loads through registers.
template <int NTH, typename T>
__device__ __forceinline__ void slab_by_element(const T* s, unsigned char* to, int n, int tid) {
  for (int e = tid; e < n; e += NTH) reinterpret_cast<T*>(to)[e] = s[e];
}
__device__ __forceinline__ float stage_value(const float* p, int k) { return p[k]; }
__device__ __forceinline__ float stage_value(const uint16_t* p, int k) { return __uint_as_float(uint32_t(p[k]) << 16); }

template <int L>
struct KGeo {
  using G = MfmaGeo<L>;
  static constexpr int NPT = G::NPT, NW = 4 * NPT, NTH = 64 * NW, K = (L + 1) * (L + 1);
  static_assert(G::NQ == NW, "one quad of orders per wave");
  // Powers of two.  The theta values stand for inputs of norm [1/2, 1) 2^SE1 and
  // 2^SE2, so that |F1 F2| stays below the half type's largest value; the
  // moments, sums of up to 2 (Q + 1) products, come down by another 2^-MS.
  static constexpr int SE1 = L == 16 ? 6 : 5, SE2 = SE1 - 1, MS = L == 16 ? 5 : 6;
  static constexpr int LOGK = L == 16 ? 5 : 6;  // 2^LOGK > sqrt(K)
  // LDS (bytes).  V: [mirror][tile][product][input][type][slot][node][16];
  // the x stage, the moments and the output image take its place in turn.
  static constexpr int TYB = G::NSL * 256, VP = 8 * TYB, V = 2 * NPT * 4 * VP;
  static constexpr int ST = 2 * 4 * K * 4 + 16;           // x stage (at 0): two slabs of four rows, a slot of zeros
  // moments: blocks [par][order] of 16 rows of L halves; the orders of one parity
  // follow each other, odd ones first, then 0 (blocks 32 bytes apart in banks:
  // the four lane groups write four blocks next to each other)
  static constexpr int MOB = 16 * L * 2 + 32, MOP = (L + 1) * MOB;
  static constexpr int MO = ST, YO = MO + 2 * MOP, Y = 4 * K * 4 + 16;  // output image + a spare slot
  static_assert(YO + Y <= V && YO % 16 == 0, "x stage, moments and output image in V's place");
  static constexpr int V0 = V, V0B = NPT * 16 * 16 * 4;  // m = 0: [tile][product][input][par][pair], fp32
  static constexpr int POLE = V0 + V0B, POLEB = 16 * 4;  // and the poles: [product][input][par]
  static constexpr int RED = POLE + POLEB, REDB = 2 * NW * 16 * 4;  // per wave and row: sum of squares; largest value
  static constexpr int EX = RED + REDB, LDS = EX + 32;              // [product][input] exponents
  // workgroups a CU holds: at L = 16 three by registers (four, 128 registers
  // with 20 spilled, measured the same), at L = 32 one by LDS
  static constexpr int WGS = L == 16 ? 3 : 1;
};

template <int L, typename T1, typename T2, bool WGT>
__global__ __launch_bounds__(KGeo<L>::NTH) __attribute__((amdgpu_waves_per_eu(L == 16 ? 3 : 2))) void k_full_mfma(
    const T1* __restrict__ x1, const T2* __restrict__ x2, float* __restrict__ y, int64_t n, int64_t ngroups,
    int64_t nwg, DevTables t, DegWeights wt, int k1, int k2, int ko, int vecx, int vecy) {
  using G = MfmaGeo<L>;
  using KG = KGeo<L>;
  constexpr int NPT = KG::NPT, NTH = KG::NTH, K = KG::K, NMB = G::NMB, NPART = G::NPART;
  __shared__ __align__(16) unsigned char lds[KG::LDS];
  lds_poison(reinterpret_cast<float*>(lds), KG::LDS / 4);
  float* const yimg = reinterpret_cast<float*>(lds + KG::YO);
  float* const pole = reinterpret_cast<float*>(lds + KG::POLE);
  float* const red = reinterpret_cast<float*>(lds + KG::RED);
  int* const ebuf = reinterpret_cast<int*>(lds + KG::EX);
  const u4* const img = reinterpret_cast<const u4*>(t.MF);  // an fp16 image is 64 of these
  const f4* const simg = reinterpret_cast<const f4*>(t.MS);
  const u4* const idx = reinterpret_cast<const u4*>(t.MFX);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int even = wave / G::NSL, jq = wave % G::NSL;  // this wave's quad: orders (L / 4) mi + 2 jq + 1 (odd) or + 2
  const int task = wave < G::NT0 ? wave : G::NT0 - 1;  // its m = 0 task (waves past the last repeat it)
  const int kk = ko < K ? ko : K;                      // output coefficients per row that may be non-zero

  // phi operands of phase B, held across the groups
  u4 tp[4][NMB];
  uint32_t ta[4][4 * G::TAI];
  const int lane0 = threadIdx.x & 63;
  cfor<0, 4>([&](auto TY) {
    constexpr int ty = decltype(TY)::value;
    cfor<0, NMB>([&](auto MB) {
      constexpr int mb = decltype(MB)::value;
      tp[ty][mb] = img[G::TP / 8 + (ty * NMB + mb) * 64 + lane0];
    });
    cfor<0, G::TAI>([&](auto P) {
      constexpr int p = decltype(P)::value;
      const u4 v = img[G::TA / 8 + (ty * G::TAI + p) * 64 + lane0];
      cfor<0, 4>([&](auto E) { ta[ty][4 * p + decltype(E)::value] = v[decltype(E)::value]; });
    });
  });

  // Lane-derived indices come from an opaque copy of the thread id in every
  // phase: recomputed there, not held (or spilled) across the phases.
  auto fresh = [] {
    int v = threadIdx.x;
    asm volatile("" : "+v"(v));
    return v;
  };
  // a group's rows into the stage: x1's four rows of k1, then x2's of k2, as
  // they lie in memory.  Rows past the batch's end keep what was there: each
  // product's results come from its own rows alone.
  unsigned char* const st1 = lds;
  unsigned char* const st2 = st1 + 4 * K * sizeof(T1);
  constexpr int W1 = sizeof(T1) == 4 ? 16 : 4, W2 = sizeof(T2) == 4 ? 16 : 4;
  auto fetch = [&](int64_t p0) {
    const int cnt = int(n - p0 < 4 ? n - p0 : 4), tid = fresh();
    if (vecx && cnt == 4) {
      slab_to_lds<W1, NTH, (4 * K * int(sizeof(T1)) / W1 + NTH - 1) / NTH>(x1 + p0 * k1, st1, 4 * k1, tid, wave);
      slab_to_lds<W2, NTH, (4 * K * int(sizeof(T2)) / W2 + NTH - 1) / NTH>(x2 + p0 * k2, st2, 4 * k2, tid, wave);
    } else {
      slab_by_element<NTH>(x1 + p0 * k1, st1, cnt * k1, tid);
      slab_by_element<NTH>(x2 + p0 * k2, st2, cnt * k2, tid);
    }
    // the slot of zeros follows the slabs (mixed types: one of each width)
    if (tid < 4) {
      if constexpr (sizeof(T1) != sizeof(T2)) reinterpret_cast<uint32_t*>(lds + 24 * K)[tid] = 0;
      reinterpret_cast<uint32_t*>(lds + (sizeof(T1) == 2 ? 16 : 32) * K)[tid] = 0;
    }
  };
  // theta-synthesis tables (of tile 0 for the next group) and this thread's
  // operand offsets
  f4 sa[G::SAV], s0[G::S0V];
  u4 gx[G::GATHER / 8];
  auto load_sa = [&](int tile, int lane) {
    cfor<0, G::SAV>([&](auto V) {
      constexpr int v = decltype(V)::value;
      sa[v] = simg[G::SA / 4 + ((tile * G::NQ + wave) * G::SAV + v) * 64 + lane];
    });
  };
  auto load_gx = [&](int tid) {
    cfor<0, G::GATHER / 8>([&](auto J) {
      gx[decltype(J)::value] = idx[tid * (G::GATHER / 8) + decltype(J)::value];
    });
  };
  // The stage is complete at the barrier after every wave's own loads are:
  // the wait comes before the next tables are requested.
  auto stage_done = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int lane = fresh() & 63;
    load_sa(0, lane);
    cfor<0, G::S0V>([&](auto V) {
      constexpr int v = decltype(V)::value;
      s0[v] = simg[G::S0 / 4 + (task * G::S0V + v) * 64 + lane];
    });
    __syncthreads();
  };
  int64_t w = blockIdx.x;
  if (w >= ngroups) return;  // whole-workgroup exit
  // the workgroup's groups follow each other at equal steps (their number is
  // a multiple of 8 or there is one group each; see xcd_product)
  int64_t p0 = xcd_product(w, ngroups) * 4;
  const int64_t pstep = nwg / 8 * 4;
  fetch(p0);
  load_gx(fresh());
  stage_done();
  for (; w < ngroups; w += nwg, p0 += pstep) {
    const int cnt = int(n - p0 < 4 ? n - p0 : 4);
    int tid = fresh(), lane = tid & 63, g = lane >> 4, i = lane & 15;
    auto again = [&] {
      tid = fresh();
      lane = tid & 63;
      g = lane >> 4;
      i = lane & 15;
    };
    // ---- this lane's row of the theta contractions (product i / 4, input
    // (i / 2) % 2, cos or sin part): the steps' operands, then the m = 0 task's
    constexpr int NX = G::NSTEP + G::NS0;
    float xv[NX];
    {
      float ss = 0.0f;
      uint32_t bits = 0;
      const int ti = (i >> 1) & 1;
      const float* wrow = nullptr;
      if constexpr (WGT) {
        const float* const wb = ti ? wt.w2 : wt.w1;
        const int p = i >> 2;
        if (wb) wrow = wb + weight_row(wt, p0 + (p < cnt ? p : cnt - 1)) * (L + 1);
      }
      auto get = [&](auto F, auto degree) {
        constexpr int f = decltype(F)::value;
        const uint32_t pk = gx[f / 8][f / 2 % 4], off = f % 2 ? pk >> 16 : pk & 0xffffu;
        float v;
        if constexpr (sizeof(T1) == 4 && sizeof(T2) == 4) {
          v = *reinterpret_cast<const float*>(lds + off);
        } else if constexpr (sizeof(T1) == 2 && sizeof(T2) == 2) {
          v = stage_value(reinterpret_cast<const uint16_t*>(lds + (off >> 1)), 0);
        } else {
          // x2's slab holds 2-byte elements from 16 K on: byte off / 2 + 8 K
          const uint32_t o2 = ti ? off / 2 + 8 * K : off;
          const uint32_t b = *reinterpret_cast<const uint32_t*>(lds + (o2 & ~3u));
          v = __uint_as_float(ti ? (o2 & 2 ? b & 0xffff0000u : b << 16) : b);
        }
        if constexpr (WGT) {
          const int l = degree();
          if (wrow) v *= wrow[l <= L ? l : 0];
        }
        xv[f] = v;
        return v;
      };
      cfor<0, 4>([&](auto MI) {
        cfor<0, 2>([&](auto PA) {
          cfor<0, G::steps(decltype(MI)::value)>([&](auto S) {
            constexpr int mi = decltype(MI)::value, pa = decltype(PA)::value, st = decltype(S)::value;
            const float v = get(std::integral_constant<int, G::step0(mi, pa) + st>{}, [&] {
              return (L / 4) * mi + 2 * jq + (even ? 2 : 1) + pa + 2 * (4 * st + g);
            });
            ss = fmaf(v, v, ss);
            bits |= __float_as_uint(v);
          });
        });
      });
      float s2 = 0.0f;
      cfor<0, G::NS0>([&](auto S) {
        constexpr int st = decltype(S)::value;
        const float v = get(std::integral_constant<int, G::NSTEP + st>{}, [&] { return 2 * (4 * st + g) + wave % 2; });
        s2 = fmaf(v, v, s2);
        bits |= __float_as_uint(v);
      });
      ss += wave < 2 ? s2 : 0.0f;  // (the other waves repeat m = 0 for other tiles and the poles)
      // a sum of zero stands for coefficients of zero below; where only their
      // squares vanished, for a value that is not fine
      if (ss == 0.0f && (bits << 1) != 0) ss = 1e-38f;
      ss = add_rows(ss);
      if (g == 0) red[wave * 16 + i] = ss;
    }

    // ---- A. theta synthesis, even and odd degrees apart: rows 4 g + r =
    // (product g, input r / 2, cos or sin), columns = node pairs
    f4 ev[NPT][4], od[NPT][4], z0 = {0.0f, 0.0f, 0.0f, 0.0f};
    cfor<0, NPT>([&](auto TT) {
      constexpr int tile = decltype(TT)::value;
      cfor<0, 4>([&](auto MI) {
        constexpr int mi = decltype(MI)::value;
        f4 e = {0.0f, 0.0f, 0.0f, 0.0f}, o = e;
        cfor<0, G::steps(mi)>([&](auto S) {
          constexpr int fe = G::step0(mi, 0) + decltype(S)::value, fo = G::step0(mi, 1) + decltype(S)::value;
          e = mfma32(xv[fe], sa[fe / 4][fe % 4], e);
          o = mfma32(xv[fo], sa[fo / 4][fo % 4], o);
        });
        ev[tile][mi] = e;
        od[tile][mi] = o;
      });
      if constexpr (tile + 1 < NPT) load_sa(tile + 1, lane);
    });
    cfor<0, G::NS0>([&](auto S) {
      constexpr int st = decltype(S)::value;
      z0 = mfma32(xv[G::NSTEP + st], s0[st / 4][st % 4], z0);
    });
    __syncthreads();  // the sums of squares are complete, the stage is dead

    again();
    float sc[2];  // of product g: the powers of two of its inputs
    {
      f4 ss = {0.0f, 0.0f, 0.0f, 0.0f};
      cfor<0, KG::NW>([&](auto R) { ss += *reinterpret_cast<const f4*>(red + decltype(R)::value * 16 + 4 * g); });
      const float s[2] = {ss[0] + ss[1], ss[2] + ss[3]};
      auto fine = [](float v) { return (v > 1e-30f && v < 1e37f) || v == 0.0f; };
      // norm in [2^(e - 1), 2^e)
      int e[2] = {(__builtin_amdgcn_frexp_expf(s[0]) + 1) >> 1, (__builtin_amdgcn_frexp_expf(s[1]) + 1) >> 1};
      if (__any(!(fine(s[0]) && fine(s[1])))) {
        // (every wave sees the same sums and takes the same way)  Where a sum
        // of squares leaves fp32's range: from the largest coefficient
        float mx = 0.0f;
        cfor<0, NX>([&](auto F) { mx = fmaxf(mx, fabsf(xv[decltype(F)::value])); });
        mx = max_rows(mx);
        if (g == 0) red[(KG::NW + wave) * 16 + i] = mx;
        __syncthreads();
        f4 m = {0.0f, 0.0f, 0.0f, 0.0f};
        cfor<0, KG::NW>([&](auto R) {
          const f4 v = *reinterpret_cast<const f4*>(red + (KG::NW + decltype(R)::value) * 16 + 4 * g);
          cfor<0, 4>([&](auto E) { m[decltype(E)::value] = fmaxf(m[decltype(E)::value], v[decltype(E)::value]); });
        });
        cfor<0, 2>([&](auto TI) {
          constexpr int ti = decltype(TI)::value;
          const float v = fmaxf(m[2 * ti], m[2 * ti + 1]);
          if (!fine(s[ti])) e[ti] = v > 0.0f ? __builtin_amdgcn_frexp_expf(v) + KG::LOGK : 0;
          // the scale's part that one factor cannot carry
          const int up = (ti ? KG::SE2 : KG::SE1) - e[ti], over = up > 126 ? up - 126 : up < -126 ? up + 126 : 0;
          cfor<0, NPT>([&](auto TT) {
            cfor<0, 8>([&](auto C) {
              constexpr int c = decltype(C)::value, tile = decltype(TT)::value, r = 2 * ti + c % 2;
              ev[tile][c / 2][r] = ldexpf(ev[tile][c / 2][r], over);
              od[tile][c / 2][r] = ldexpf(od[tile][c / 2][r], over);
            });
          });
          z0[2 * ti] = ldexpf(z0[2 * ti], over);
          sc[ti] = ldexpf(1.0f, up - over);
        });
      } else {
        sc[0] = ldexpf(1.0f, KG::SE1 - e[0]);
        sc[1] = ldexpf(1.0f, KG::SE2 - e[1]);
      }
      if (wave == 0 && i == 0) {
        ebuf[2 * g] = e[0];
        ebuf[2 * g + 1] = e[1];
      }
    }
    // the node (sum) and its mirror (difference), split, to V
    cfor<0, NPT>([&](auto TT) {
      constexpr int tile = decltype(TT)::value;
      cfor<0, 4>([&](auto R) {
        constexpr int r = decltype(R)::value;  // input r / 2, type: cos or sin (r % 2), even or odd m
        float nd[4], mr[4];
        cfor<0, 4>([&](auto MI) {
          constexpr int mi = decltype(MI)::value;
          const float o = sc[r / 2] * od[tile][mi][r];
          nd[mi] = fmaf(sc[r / 2], ev[tile][mi][r], o);
          mr[mi] = fmaf(sc[r / 2], ev[tile][mi][r], -o);
        });
        unsigned char* const vb =
            lds + (tile * 4 + g) * KG::VP + ((r / 2) * 4 + (r % 2) * 2 + (even ? 0 : 1)) * KG::TYB + jq * 256 + i * 16;
        *reinterpret_cast<u4*>(vb) = split4(nd[0], nd[1], nd[2], nd[3]);
        *reinterpret_cast<u4*>(vb + NPT * 4 * KG::VP) = split4(mr[0], mr[1], mr[2], mr[3]);
      });
    });
    if (wave < 2 * NPT) {
      float* const v0 = reinterpret_cast<float*>(lds + KG::V0) + ((wave / 2 * 8 + 2 * g) * 2 + wave % 2) * 16 + i;
      v0[0] = sc[0] * z0[0];
      v0[32] = sc[1] * z0[2];
    } else if (wave < G::NT0 && i == 0) {
      pole[4 * g + wave % 2] = sc[0] * z0[0];
      pole[4 * g + 2 + wave % 2] = sc[1] * z0[2];
    }
    __syncthreads();

    again();
    // ---- B. phi stage of product bp at the pairs of tile bt
    const int bp = wave & 3, bt = wave >> 2;
    f4 o[2][4];  // [mirror][type]
    float zz[2] = {0.0f, 0.0f};
    float ce0[2], co0[2];  // m = 0 values: even and odd degrees, per input
    cfor<0, 2>([&](auto TI) {
      constexpr int ti = decltype(TI)::value;
      const float* const v0 = reinterpret_cast<const float*>(lds + KG::V0) + (bt * 8 + 2 * bp + ti) * 32 + i;
      ce0[ti] = v0[0];
      co0[ti] = v0[16];
    });
    cfor<0, 2>([&](auto NM) {
      constexpr int nm = decltype(NM)::value;
      const unsigned char* const vb =
          lds + ((nm * NPT + bt) * 4 + bp) * KG::VP + (L == 16 ? g & 1 : g) * 256 + i * 16;
      f4 acc[2][NMB][4];
      cfor<0, 4>([&](auto TY) {
        constexpr int ty = decltype(TY)::value;
        cfor<0, 2>([&](auto TI) {
          constexpr int ti = decltype(TI)::value;
          const u4 d = *reinterpret_cast<const u4*>(vb + (ti * 4 + ty) * KG::TYB);
          const float c = nm ? ce0[ti] - co0[ti] : ce0[ti] + co0[ti];
          cfor<0, NMB>([&](auto MB) {
            constexpr int mb = decltype(MB)::value;
            f4 a = ty == 0 ? f4{c, c, c, c} : f4{0.0f, 0.0f, 0.0f, 0.0f};  // m = 0 enters every even cos sum
            const u4 tq = tp[ty][mb];
            if constexpr (L == 16) {
              a = mfma(tq, d, a);
            } else {
              a = mfma(u4{tq[2], tq[3], tq[2], tq[3]}, d, a);
              a = mfma(u4{tq[0], tq[1], tq[0], tq[1]}, d, a);
            }
            acc[ti][mb][ty] = a;
          });
        });
        GTP_FENCE();
      });
      // sample products folded over the four points of a quarter angle, from
      // the class sums of the two inputs (the factor 4 in the output scale)
      cfor<0, NMB>([&](auto MB) {
        constexpr int mb = decltype(MB)::value;
        const f4 pe1 = acc[0][mb][0], po1 = acc[0][mb][1], qe1 = acc[0][mb][2], qo1 = acc[0][mb][3];
        const f4 pe2 = acc[1][mb][0], po2 = acc[1][mb][1], qe2 = acc[1][mb][2], qo2 = acc[1][mb][3];
        acc[0][mb][0] = pe1 * pe2 + po1 * po2 + qe1 * qe2 + qo1 * qo2;
        acc[0][mb][1] = pe1 * po2 + po1 * pe2 + qe1 * qo2 + qo1 * qe2;
        acc[0][mb][2] = pe1 * qe2 + po1 * qo2 + qe1 * pe2 + qo1 * po2;
        acc[0][mb][3] = pe1 * qo2 + po1 * qe2 + qe1 * po2 + qo1 * pe2;
      });
      if constexpr (L == 32) {
        // m = 0 moment (at L = 16 a row of the analysis): samples 16 mb + 4 g + r
        float z = 0.0f;
        cfor<0, NMB>([&](auto MB) {
          cfor<0, 4>([&](auto R) {
            constexpr int mb = decltype(MB)::value, r = decltype(R)::value;
            const int k = 16 * mb + 4 * g + r;
            const float wk = k > G::Q ? 0.0f : (k == 0 || k == G::Q) ? 0.5f : 1.0f;
            z = fmaf(wk, acc[0][mb][0][r], z);
          });
        });
        zz[nm] = add_rows(z);
      }
      cfor<0, 4>([&](auto TY) {
        constexpr int ty = decltype(TY)::value;
        const f4 a = acc[0][0][ty];
        f4 s = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (L == 16) {
          const u4 d = split4(a[0], a[1], a[2], a[3]);
          s = mfma(u4{ta[ty][2], ta[ty][3], ta[ty][2], ta[ty][3]}, d, s);
          s = mfma(u4{ta[ty][0], ta[ty][1], ta[ty][0], ta[ty][1]}, d, s);
        } else {
          const f4 b = acc[0][NMB - 1][ty];
          const u4 d = split4(a[0], a[1], a[2], a[3]), e = split4(b[0], b[1], b[2], b[3]);
          const u4 h1 = {d[0], d[1], e[0], e[1]}, h2 = {d[2], d[3], e[2], e[3]};
          const u4 t1 = {ta[ty][0], ta[ty][1], ta[ty][2], ta[ty][3]}, t2 = {ta[ty][4], ta[ty][5], ta[ty][6], ta[ty][7]};
          s = mfma(t2, h2, s);
          s = mfma(t2, h1, s);
          s = mfma(t1, h2, s);
          s = mfma(t1, h1, s);
        }
        o[nm][ty] = s;
        GTP_FENCE();
      });
    });
    again();
    // theta-analysis tables of this wave's orders, in flight across the barriers
    u4 wc[8][G::WPARTS], w0[G::WPARTS];
    cfor<0, G::WPARTS>([&](auto P) {
      constexpr int p = decltype(P)::value;
      cfor<0, 8>([&](auto C) {
        constexpr int c = decltype(C)::value;
        wc[c][p] = img[G::WC / 8 + ((wave * 8 + c) * G::WPARTS + p) * 64 + lane];
      });
      w0[p] = img[G::W0 / 8 + ((wave < NPART ? wave : 0) * G::WPARTS + p) * 64 + lane];
    });
    u4 sx[3];  // this thread's output offsets
    cfor<0, 3>([&](auto J) { sx[decltype(J)::value] = idx[NTH * (G::GATHER / 8) + tid * 3 + decltype(J)::value]; });
    __syncthreads();  // every wave is done with V
    if (w + nwg < ngroups) fetch(p0 + pstep);  // in flight until the next turn
    again();
    // moments of the pairs: sum (par 0) and difference (par 1) of the node and
    // its mirror, parts 1 and 2 to rows (product, cos or sin, part)
    {
      // two neighbouring lanes share their words: even lanes write the sums of
      // both pairs, odd lanes the differences (half the stores of one each)
      unsigned char* const mo =
          lds + KG::MO + g * KG::MOB + (i & 1) * KG::MOP + (bp * 4) * (L * 2) + (16 * bt + (i & 14)) * 2;
      const uint32_t pick = i & 1 ? 0x03020706u : 0x05040100u;
      constexpr float ms = 1.0f / float(1 << KG::MS);
      auto pair_word = [&](uint32_t own) {
        const uint32_t nb = __builtin_amdgcn_mov_dpp(own, 0xb1 /* quad_perm 1, 0, 3, 2 */, 0xf, 0xf, true);
        return __builtin_amdgcn_perm(nb, own, pick);
      };
      auto put = [&](unsigned char* b, float vn, float vm) {
        const float a = ms * vn;
        uint32_t p, r;
        split2(fmaf(ms, vm, a), fmaf(-ms, vm, a), p, r);
        *reinterpret_cast<uint32_t*>(b) = pair_word(p);
        *reinterpret_cast<uint32_t*>(b + L * 2) = pair_word(r);
      };
      cfor<0, 4>([&](auto TY) {
        constexpr int ty = decltype(TY)::value;
        cfor<0, L / 8>([&](auto R) {
          constexpr int r = decltype(R)::value;  // order number 4 r + g of its parity
          put(mo + ((ty % 2 ? 0 : L / 2) + 4 * r) * KG::MOB + (ty / 2) * 2 * (L * 2), o[0][ty][r], o[1][ty][r]);
        });
      });
      // m = 0: a row of the analysis at L = 16
      if (g == 0) {
        if constexpr (L == 16) {
          put(mo + L * KG::MOB, o[0][0][2], o[1][0][2]);
        } else {
          put(mo + L * KG::MOB, zz[0], zz[1]);
        }
      }
    }
    __syncthreads();

    again();
    // ---- C. theta analysis: rows 4 g + r = (product g, cos or sin, part),
    // columns = degrees l = m + par + 2 i
    {
      const int ex = ebuf[2 * g] + ebuf[2 * g + 1] + (2 + KG::MS - KG::SE1 - KG::SE2) - t.mf_kw;
      const float* worow = nullptr;
      if constexpr (WGT) {
        if (wt.wo) worow = wt.wo + weight_row(wt, p0 + (g < cnt ? g : cnt - 1)) * (L + 1);
      }
      const unsigned char* const mo = lds + KG::MO + i * (L * 2) + (L == 16 ? g & 1 : g) * 16;
      auto sums = [&](int blk, int pa, const u4 (&tw)[G::WPARTS]) {
        const u4 d = *reinterpret_cast<const u4*>(mo + blk * KG::MOB + pa * KG::MOP);
        f4 s = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (G::WPARTS == 2) s = mfma(d, tw[1], s);
        return mfma(d, tw[0], s);
      };
      auto put = [&](uint32_t off, int l, float v) {
        v = ldexpf(v, ex);
        if constexpr (WGT) {
          if (worow) v *= worow[l <= L ? l : 0];
        }
        *reinterpret_cast<float*>(lds + KG::YO + off) = v;
      };
      cfor<0, 8>([&](auto C) {
        constexpr int c = decltype(C)::value, pa = c % 2;
        const int num = (L / 8) * (c / 2) + jq;  // of its parity: order 2 num + 1 (odd), + 2 (even)
        const int l = 2 * num + (even ? 2 : 1) + pa + 2 * i;
        const f4 s = sums((even ? L / 2 : 0) + num, pa, wc[c]);
        const uint32_t off = sx[c / 4][c % 4];
        put(off & 0xffffu, l, s[0] + s[1]);
        put(off >> 16, l, s[2] + s[3]);
      });
      if (wave < NPART) {
        const int pa = wave < G::NE0 ? 0 : 1, l = 2 * (16 * (wave - (pa ? G::NE0 : 0)) + i) + pa;
        const f4 s = sums(L, pa, w0);
        // the poles' part: equal phi samples there; sum and difference of the
        // two poles' products, in the contraction's scale
        const f4 q = *reinterpret_cast<const f4*>(pole + 4 * g);  // x1 even, odd, x2 even, odd degrees
        const float pp = pa ? q[0] * q[3] + q[1] * q[2] : q[0] * q[2] + q[1] * q[3];
        const float wp = t.WT[l <= L ? l * (l + 1) / 2 : 0] * ldexpf(2.0f * float(G::NP), t.mf_kw - 2 - KG::MS);
        put(sx[2][0] & 0xffffu, l, fmaf(wp, pp, s[0] + s[1]));
      }
    }
    load_gx(tid);
    if (w + nwg < ngroups) {
      stage_done();
    } else {
      __syncthreads();
    }
    again();
    // ---- the four rows out (zeros above the kernel's degree)
    float* const out = y + p0 * ko;
    if (vecy && cnt == 4) {
      for (int u = tid; u < kk; u += NTH)
        __builtin_nontemporal_store(reinterpret_cast<const f4*>(yimg)[u], reinterpret_cast<f4*>(out) + u);
    } else if (kk == ko) {
      for (int e = tid; e < cnt * ko; e += NTH) out[e] = yimg[e];
    } else {
      for (int p = 0; p < cnt; ++p)
        for (int e = tid; e < ko; e += NTH) out[int64_t(p) * ko + e] = e < kk ? yimg[p * kk + e] : 0.0f;
    }
  }
}

template <int L, typename T1, typename T2, bool WGT>
hipError_t launch_typed(const DevTables& t, const void* x1, const void* x2, int64_t n, float* y, const DegWeights& wt,
                        hipStream_t s, int k1, int k2, int ko) {
  using KG = KGeo<L>;
  // at most 2^28 groups per launch
  constexpr int64_t kMost = int64_t(1) << 30;
  for (int64_t p0 = 0; p0 < n; p0 += kMost) {
    const int64_t nn = n - p0 < kMost ? n - p0 : kMost, ng = (nn + 3) / 4;
    const T1* const a = static_cast<const T1*>(x1) + size_t(p0) * k1;
    const T2* const b = static_cast<const T2*>(x2) + size_t(p0) * k2;
    float* const yy = y + size_t(p0) * ko;
    DegWeights w = wt;
    w.pbase += p0;
    // a group's slab starts 4 k elements after the last: aligned with the base
    // (fp32 slabs move by 16 bytes, bf16 slabs, 8 k bytes apart, by 4)
    const int vecx = reinterpret_cast<uintptr_t>(a) % (sizeof(T1) == 4 ? 16 : 4) == 0 &&
                     reinterpret_cast<uintptr_t>(b) % (sizeof(T2) == 4 ? 16 : 4) == 0;
    const int vecy = reinterpret_cast<uintptr_t>(yy) % 16 == 0 && ko <= KG::K;
    // as many workgroups as MI355X's 256 CUs hold (a multiple of 8; any number works)
    constexpr int64_t most = 256 * KG::WGS;
    hipLaunchKernelGGL((k_full_mfma<L, T1, T2, WGT>), dim3(unsigned(ng < most ? ng : most)), dim3(KG::NTH), 0, s, a, b,
                       yy, nn, ng, ng < most ? ng : most, t, w, k1, k2, ko, vecx, vecy);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int L>
hipError_t launch_one(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n, float* y,
                      const DegWeights& wt, hipStream_t s, bool* supported, int k1, int k2, int ko) {
  constexpr int K = KGeo<L>::K;
  if (ko == 0) k1 = k2 = ko = K;
  if (k1 > K || k2 > K || k1 < 1 || k2 < 1 || (wt.on && (k1 != K || k2 != K || ko != K))) {
    *supported = false;
    return hipSuccess;
  }
  if (wt.on) {
    if (it1 == IN_F32 && it2 == IN_F32) return launch_typed<L, float, float, true>(t, x1, x2, n, y, wt, s, k1, k2, ko);
    if (it1 == IN_BF16 && it2 == IN_BF16)
      return launch_typed<L, uint16_t, uint16_t, true>(t, x1, x2, n, y, wt, s, k1, k2, ko);
  } else {
    if (it1 == IN_F32 && it2 == IN_F32)
      return launch_typed<L, float, float, false>(t, x1, x2, n, y, wt, s, k1, k2, ko);
    if (it1 == IN_BF16 && it2 == IN_BF16)
      return launch_typed<L, uint16_t, uint16_t, false>(t, x1, x2, n, y, wt, s, k1, k2, ko);
    if (it1 == IN_F32 && it2 == IN_BF16)
      return launch_typed<L, float, uint16_t, false>(t, x1, x2, n, y, wt, s, k1, k2, ko);
  }
  *supported = false;
  return hipSuccess;
}

}  // namespace

hipError_t launch_full_mfma(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n, float* y,
                            const DegWeights& wt, hipStream_t s, bool* supported, int k1, int k2, int ko) {
  *supported = true;
  if (t.MS && t.MF && t.MFX && t.waveL == 16) return launch_one<16>(t, x1, it1, x2, it2, n, y, wt, s, supported, k1, k2, ko);
  if (t.MS && t.MF && t.MFX && t.waveL == 32) return launch_one<32>(t, x1, it1, x2, it2, n, y, wt, s, supported, k1, k2, ko);
  *supported = false;
  return hipSuccess;
}

}  // namespace gtp
