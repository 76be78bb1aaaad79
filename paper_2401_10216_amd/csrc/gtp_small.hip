// Thread-per-product fused Gaunt tensor product for small degrees (gfx950).
//
// One lane owns one (b, c) product.  The three steps of Sec. 3.2 run with the
// convolution theorem: the 2D Fourier series of each input is sampled on a
// uniform (theta, phi) torus grid (the inverse transforms, with step 1 folded
// into the theta part: table S), the samples are multiplied pointwise, and the
// forward transforms followed by step 3 (table W) give the SH coefficients.
// The theta transforms use the grid's mirror symmetry t <-> pi - t (Theta_lm
// has parity (-1)^(l+m)), the phi transforms use p <-> -p and pi -+ p: they
// are unrolled direct DFTs with compile-time twiddles, and the pointwise
// product is taken, already folded over each quarter angle's four points,
// from the two inputs' quarter-angle class sums.  For equal degrees the S
// and W rows are compile-time constants too.  Nothing but x and y touches
// HBM.
#include "gtp_small.hpp"
#include "gtp_small_core.hpp"

namespace gtp {
namespace {

template <int L1, int L2, int LO, int NU, typename T1, typename T2, bool WGT, bool OUT>
__global__ __launch_bounds__(kTile) __attribute__((amdgpu_waves_per_eu(small_waves(L1, L2, LO)))) void k_full_small(const T1* __restrict__ x1, const T2* __restrict__ x2,
                                                      float* __restrict__ y, int64_t n,
                                                      const float* __restrict__ ST, int ntS,
                                                      const float* __restrict__ WT, int ntW, DegWeights wt,
                                                      PairIdx pi, int dma) {
  using G = Geo<L1, L2, LO, NU>;
  constexpr int K1 = csh(L1), K2 = NU == 0 ? csh(L2) : 1, KO = csh(LO);
  constexpr int S2 = lds_stride(K2);
  constexpr int KT = cmax(S2, lds_stride(KO));
  __shared__ __align__(16) float tile[kTile * KT];
  lds_poison(tile, kTile * KT);
  const int tid = threadIdx.x;
  const int64_t p0 = int64_t(blockIdx.x) * kTile;
  const int cnt = int((n - p0) < kTile ? (n - p0) : kTile);
  float xa[K1];
  float acc[G::KE];
  if constexpr (NU == 0) {
    // each lane loads its own two rows, x1 into registers and x2 into its
    // tile row (row-major, odd row stride: conflict-free reads); a wave's
    // rows are contiguous, so every cache line still comes from HBM once.
    // Lanes past the end repeat the last product.  Outer-product indexing
    // (pair products of channel mixing) takes rows b C1 + c1 and b C2 + c2.
    const int64_t p = p0 + (tid < cnt ? tid : cnt - 1);
    int64_t r1 = p, r2 = p;
    if constexpr (OUT) pair_rows(pi, p, r1, r2);
    const T1* const xr1 = x1 + r1 * K1;
    const T2* const xr2 = x2 + r2 * K2;
    cfor<0, K1>([&](auto I) { xa[decltype(I)::value] = ld_in(xr1, decltype(I)::value); });
    // x2 into its tile rows (the pair products' rows are not one slab)
    stage_tile_rows<L2, !OUT>(tile, x2, xr2, p0, cnt, tid, dma);
    if constexpr (WGT) {
      // each lane scales its own product: x1 in registers, x2 in its tile row
      const int64_t row = weight_row(wt, p0 + tid);
      if (wt.w1)
        scale_by_degree<L1, K1>(wt.w1 + row * (L1 + 1), [&](auto I) -> float& { return xa[decltype(I)::value]; });
      if (wt.w2)
        scale_by_degree<L2, K2>(wt.w2 + row * (L2 + 1),
                                [&](auto I) -> float& { return tile[tid * S2 + decltype(I)::value]; });
    }
    RegX<K1> A{xa};
    LdsX B{tile, tid * S2};
    gtp_core<L1, L2, LO, NU>(A, B, acc, ST, ntS, WT, ntW);
    if constexpr (WGT) {
      // outputs above degree LE are zeros and stay zeros
      if (wt.wo) {
        // the row index from an opaque copy of the lane id (not held across the core)
        int tq = threadIdx.x;
        asm volatile("" : "+v"(tq));
        scale_by_degree<G::LE, G::KE>(wt.wo + weight_row(wt, p0 + tq) * (LO + 1),
                                      [&](auto I) -> float& { return acc[decltype(I)::value]; });
      }
    }
    __syncthreads();
  } else {
    load_rows<K1>(x1, p0, cnt, xa);
    RegX<K1> A{xa};
    gtp_core<L1, L2, LO, NU>(A, A, acc, ST, ntS, WT, ntW);
  }
  store_rows<KO, G::KE>(y, p0, cnt, tile, acc);
}

// Both input gradients of an equal-degree product (the backward of Sec. 3.1's
// product, L1 = L2 = Lout = L <= 8): dx1 = P_L(GTP(dy, x2)) and then
// dx2 = P_L(GTP(dy, x1)), each the forward product on the compile-time
// tables of (L, L, L).  Each lane's dy row is read once and stays in
// registers for both products; x2, then x1, pass through the one LDS tile,
// and each gradient leaves through it as the forward's output does.  Against
// two forward launches this saves dy's second read: five rows move per
// product instead of six.  The two products run as a loop that is not
// unrolled, so the core's code is not duplicated.
template <int L, typename TX>
__global__ __launch_bounds__(kTile) __attribute__((amdgpu_waves_per_eu(small_waves(L, L, L)))) void k_bwd_small(
    const float* __restrict__ dy, const TX* __restrict__ x1, const TX* __restrict__ x2, float* __restrict__ dx1,
    float* __restrict__ dx2, int64_t n, int dma) {
  constexpr int K = csh(L), S = lds_stride(K);
  __shared__ __align__(16) float tile[kTile * S];
  lds_poison(tile, kTile * S);
  const int64_t p0 = int64_t(blockIdx.x) * kTile;
  const int cnt = int((n - p0) < kTile ? (n - p0) : kTile);
  float xd[K], acc[K];
  {
    const int tid = threadIdx.x;
    const float* const dr = dy + (p0 + (tid < cnt ? tid : cnt - 1)) * K;
    cfor<0, K>([&](auto I) { xd[decltype(I)::value] = dr[decltype(I)::value]; });
  }
#pragma unroll 1
  for (int g = 0; g < 2; ++g) {
    // dy's values opaque to the compiler in each product (its node
    // syntheses, the same in both, are not hoisted out of the loop and held:
    // that would take more registers than the core has), and the lane's row
    // addresses rebuilt from an opaque copy of the lane id in each product
    // rather than held across it
#pragma unroll
    for (int i = 0; i < K; ++i) asm volatile("" : "+v"(xd[i]));
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int64_t p = p0 + (tid < cnt ? tid : cnt - 1);
    const TX* const x = g == 0 ? x2 : x1;  // dx1 pairs dy with x2, dx2 with x1
    float* const out = g == 0 ? dx1 : dx2;
    stage_tile_rows<L, true>(tile, x, x + p * K, p0, cnt, tid, dma);
    gtp_core_lit<L>(RegX<K>{xd}, LdsX{tile, tid * S}, acc);
    __syncthreads();
    store_rows<K, K>(out, p0, cnt, tile, acc, tid);
    __syncthreads();  // the stores' tile reads are done before the next rows land there
  }
}

// Degree-padded product: a plan of degrees (a, b, c) whose padded degree
// L = max(a, b, min(c, a + b)) is at most 8 runs on the equal-degree core of
// degree L (compile-time tables).  The inputs are read as degree-L vectors
// whose coefficients above their own degrees are zero (rows of k1 = (a+1)^2
// and k2 = (b+1)^2 values), and the first ko = (c+1)^2 outputs are written
// (zeros above degree L when c > L).  Exact: the degree-L sampling grid
// integrates the product of any two degree-L functions exactly, and
// zero-padding or truncating the coefficient vectors changes nothing else.
template <int L, typename T1, typename T2>
__global__ __launch_bounds__(kTile) __attribute__((amdgpu_waves_per_eu(small_waves(L, L, L)))) void k_full_small_pad(
    const T1* __restrict__ x1, const T2* __restrict__ x2, float* __restrict__ y, int64_t n, int k1, int k2, int ko) {
  constexpr int K = csh(L), S = lds_stride(K);
  __shared__ __align__(16) float tile[kTile * S];
  lds_poison(tile, kTile * S);
  const int tid = threadIdx.x;
  const int64_t p0 = int64_t(blockIdx.x) * kTile;
  const int cnt = int((n - p0) < kTile ? (n - p0) : kTile);
  const int64_t p = p0 + (tid < cnt ? tid : cnt - 1);
  const int row = tid < cnt ? tid : cnt - 1;
  // The workgroup's rows of each input are one contiguous slab: coalesced
  // loads of the slab into the tile (compact rows of k floats), then each
  // lane takes its own row out of LDS, zero-padded to degree L.
  auto slab_to_tile = [&](auto src, int k) {
    const int tot = cnt * k;
    int e = tid;
    for (; e + 3 * kTile < tot; e += 4 * kTile) {
      const float v0 = ld_in(src, e), v1 = ld_in(src, e + kTile), v2 = ld_in(src, e + 2 * kTile),
                  v3 = ld_in(src, e + 3 * kTile);
      tile[e] = v0;
      tile[e + kTile] = v1;
      tile[e + 2 * kTile] = v2;
      tile[e + 3 * kTile] = v3;
    }
    for (; e < tot; e += kTile) tile[e] = ld_in(src, e);
    __syncthreads();
  };
  float xa[K];
  slab_to_tile(x1 + p0 * k1, k1);
  cfor<0, K>([&](auto I) {
    constexpr int i = decltype(I)::value;
    const float v = tile[row * k1 + (i < k1 ? i : 0)];  // in-bounds index, then the select
    xa[i] = i < k1 ? v : 0.0f;
  });
  __syncthreads();
  {
    float xb[K];
    slab_to_tile(x2 + p0 * k2, k2);
    cfor<0, K>([&](auto I) {
      constexpr int i = decltype(I)::value;
      const float v = tile[row * k2 + (i < k2 ? i : 0)];
      xb[i] = i < k2 ? v : 0.0f;
    });
    __syncthreads();
    cfor<0, K>([&](auto I) { tile[tid * S + decltype(I)::value] = xb[decltype(I)::value]; });
  }
  float acc[K];
  RegX<K> A{xa};
  LdsX B{tile, tid * S};
  gtp_core<L, L, L, 0>(A, B, acc, nullptr, 0, nullptr, 0);
  __syncthreads();
  if (ko <= K) {
    cfor<0, K>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if (i < ko) tile[tid * ko + i] = acc[i];
    });
    __syncthreads();
    float* const out = y + p0 * ko;
    for (int i = tid; i < cnt * ko; i += kTile) out[i] = tile[i];
  } else if (tid < cnt) {
    float* const out = y + p * ko;
    cfor<0, K>([&](auto I) { out[decltype(I)::value] = acc[decltype(I)::value]; });
    for (int i = K; i < ko; ++i) out[i] = 0.0f;
  }
}

// Stepwise many-body chain: B_2 = P_LO(A A), B_{k+1} = P_LO(B_k A).
template <int L, int LO, typename TIn>
__global__ __launch_bounds__(kTile) void k_self_stepwise_small(const TIn* __restrict__ x, float* __restrict__ y,
                                                               int64_t n, int nu, DevTables t1, DevTables t2) {
  constexpr int K = csh(L), KO = csh(LO);
  using G1 = Geo<L, L, LO, 0>;
  using G2 = Geo<LO, L, LO, 0>;
  constexpr int KT = lds_stride(KO);  // the output rows (store_rows)
  __shared__ __align__(16) float tile[kTile * KT];
  lds_poison(tile, kTile * KT);
  const int64_t p0 = int64_t(blockIdx.x) * kTile;
  const int cnt = int((n - p0) < kTile ? (n - p0) : kTile);
  float a[K];
  load_rows<K>(x, p0, cnt, a);
  float b[KO];
  {
    float acc[G1::KE];
    RegX<K> A{a};
    gtp_core<L, L, LO, 0>(A, A, acc, t1.ST, t1.ntS, t1.WT, t1.ntW);
    cfor<0, KO>([&](auto I) {
      constexpr int i = decltype(I)::value;
      b[i] = i < G1::KE ? acc[i < G1::KE ? i : 0] : 0.0f;
    });
  }
  for (int step = 2; step < nu; ++step) {
    float acc[G2::KE];
    RegX<K> A{a};
    RegX<KO> Bv{b};
    gtp_core<LO, L, LO, 0>(Bv, A, acc, t2.ST, t2.ntS, t2.WT, t2.ntW);
    cfor<0, KO>([&](auto I) {
      constexpr int i = decltype(I)::value;
      b[i] = i < G2::KE ? acc[i < G2::KE ? i : 0] : 0.0f;
    });
  }
  store_rows<KO, KO>(y, p0, cnt, tile, b);
}

template <int L1, int L2, int LO, int NU, typename T1, typename T2, bool WGT, bool OUT = false>
hipError_t launch_typed(const DevTables& t, const void* x1, const void* x2, int64_t n, float* y,
                        const DegWeights& wt, hipStream_t s, const PairIdx& pi = PairIdx{0, 0}) {
  const dim3 grid(unsigned((n + kTile - 1) / kTile)), block(kTile);
  const int dma = (reinterpret_cast<uintptr_t>(x2) % 16) == 0;  // 16-byte runs straight into LDS
  hipLaunchKernelGGL((k_full_small<L1, L2, LO, NU, T1, T2, WGT, OUT>), grid, block, 0, s, static_cast<const T1*>(x1),
                     static_cast<const T2*>(x2), y, n, t.ST, t.ntS, t.WT, t.ntW, wt, pi, dma);
  return hipGetLastError();
}

// Input types: both fp32, both bf16, or (equal degrees only) fp32 x1 with
// bf16 x2, the pairing of a backward pass (fp32 output gradient times a bf16
// input).  Per-degree weights: equal degrees, equal input types.  Other
// combinations are not instantiated (*supported = false).
template <int L1, int L2, int LO, int NU>
hipError_t launch_one(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n, float* y,
                      const DegWeights& wt, hipStream_t s, bool* supported) {
  constexpr bool equal = L1 == L2 && L2 == LO && NU == 0;
  if (wt.on) {
    if constexpr (equal) {
      if (it1 == IN_BF16 && it2 == IN_BF16)
        return launch_typed<L1, L2, LO, NU, uint16_t, uint16_t, true>(t, x1, x2, n, y, wt, s);
      if (it1 == IN_F32 && it2 == IN_F32) return launch_typed<L1, L2, LO, NU, float, float, true>(t, x1, x2, n, y, wt, s);
    }
    *supported = false;
    return hipSuccess;
  }
  if (it1 == IN_BF16 && it2 == IN_BF16)
    return launch_typed<L1, L2, LO, NU, uint16_t, uint16_t, false>(t, x1, x2, n, y, wt, s);
  if (it1 == IN_F32 && it2 == IN_F32) return launch_typed<L1, L2, LO, NU, float, float, false>(t, x1, x2, n, y, wt, s);
  if constexpr (equal) {
    if (it1 == IN_F32 && it2 == IN_BF16)
      return launch_typed<L1, L2, LO, NU, float, uint16_t, false>(t, x1, x2, n, y, wt, s);
  }
  *supported = false;
  return hipSuccess;
}

// Outer-product pair products (channel mixing), equal degrees, equal types.
template <int L>
hipError_t launch_pairs_one(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n,
                            float* y, const PairIdx& pi, hipStream_t s, bool* supported) {
  const DegWeights nw{nullptr, nullptr, nullptr, 1, 0, 0, false};
  if (it1 == IN_F32 && it2 == IN_F32) return launch_typed<L, L, L, 0, float, float, false, true>(t, x1, x2, n, y, nw, s, pi);
  if (it1 == IN_BF16 && it2 == IN_BF16)
    return launch_typed<L, L, L, 0, uint16_t, uint16_t, false, true>(t, x1, x2, n, y, nw, s, pi);
  *supported = false;
  return hipSuccess;
}

// Fused channel mixing (the channel-mixing rule of the appendix, Implementation
// Details; equal degrees L, Kd = (L+1)^2):
//   y[b, co] = sum_p W[co, p] T[b, p],  T[b, p] = GTP(x1[b, c1], x2[b, c2]),
// p = c1 C2 + c2.  One workgroup (four waves) per batch entry, in rounds of
// 256 pairs: each lane takes one pair product with the thread-per-product
// core (x2 row in its LDS row), writes the product over that row, and after
// a barrier the waves mix the round's 256 products on the matrix cores,
//   y_b^T (Kd x Co) += T_round^T (Kd x 256) W^T_round (256 x Co),
// wave w taking the 16-coefficient row tiles w, w + 4, ... and every
// 16-channel column tile (v_mfma_f32_16x16x4f32: A[i][k] from lane 16 k + i,
// B[k][j] from lane 16 k + j, D register r of lane 16 g + i = row 4 g + r,
// column i).  K-step s of a round covers the pair slots 4 s + g; the weights
// come in the blocked layout WB[p / 16][co][g][s'] (p = 16 (p / 16) + 4 s' +
// g, zero past P and Co), so one 16-byte load gives a lane its B operands of
// four K-steps.  The partial y_b of each wave's tiles passes from one round
// to the next through y itself (each lane reads back what it wrote; the
// lines stay in L2), so no accumulator is live during the products.  Only
// x1, x2, W and y touch HBM.
// FINE (from 128 pairs): 32 pairs at a time are summed from zero, those sums to
// the round's, the rounds' to y, instead of every K-step rounding the whole sum
// so far: error against 64-bit results at L = 6 2.3e-7 -> 1.5e-7 at 128 pairs, 5.8e-7
// -> 1.6e-7 at 1024, 1.1e-6 -> 1.7e-7 at 4096, for 0 to 5 % of time (11 to 16 % at
// L <= 4 and 128 outputs; runs of 16 pairs took 30 % there, and an outer loop over
// runs 40 %).
typedef float mixv4 __attribute__((ext_vector_type(4)));
constexpr int kMixThreads = 256;
// waves per SIMD of the fused mix: the thread-per-product core's budget,
// except at L = 8 where the 81 KB tile admits one workgroup per CU anyway
constexpr int mix_waves(int L) { return L == 8 ? 1 : small_waves(L, L, L); }

template <int L, typename TIn, int NCT, bool FINE>
__global__ __launch_bounds__(kMixThreads) __attribute__((amdgpu_waves_per_eu(mix_waves(L)))) void k_mix_fused(
    const TIn* __restrict__ x1, const TIn* __restrict__ x2, const float* __restrict__ WB, float* __restrict__ y,
    int64_t C1, int64_t C2, int Co, int64_t P, const float* __restrict__ ST, int ntS, const float* __restrict__ WT,
    int ntW) {
  constexpr int Kd = csh(L);
  constexpr int NKT = (Kd + 15) / 16, KTW = (NKT + 3) / 4, CoB = 16 * NCT, KS = lds_stride(Kd);
  __shared__ float tile[kMixThreads * KS];
  lds_poison(tile, kMixThreads * KS);
  const int64_t b = blockIdx.x;
  const int64_t nround = (P + kMixThreads - 1) / kMixThreads;
  for (int64_t r = 0; r < nround; ++r) {
    // thread-derived indices from an opaque copy of the thread id each round
    // (recomputed, not held across the product)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wv = tid >> 6, g = lane >> 4, i = lane & 15;
    {
      // pair index split in 32 bits (the launcher takes C1 C2 < 2^31)
      const unsigned pl = unsigned(r) * kMixThreads + unsigned(tid);
      const unsigned pc = pl < unsigned(P) ? pl : unsigned(P) - 1u;
      const unsigned c1 = pc / unsigned(C2), c2 = pc - c1 * unsigned(C2);
      const TIn* const xr1 = x1 + (b * C1 + c1) * Kd;
      const TIn* const xr2 = x2 + (b * C2 + c2) * Kd;
      float xa[Kd], acc[Kd];
      cfor<0, Kd>([&](auto I) { xa[decltype(I)::value] = ld_in(xr1, decltype(I)::value); });
      cfor<0, Kd>([&](auto I) { tile[tid * KS + decltype(I)::value] = ld_in(xr2, decltype(I)::value); });
      RegX<Kd> A{xa};
      LdsX Bx{tile, tid * KS};
      gtp_core<L, L, L, 0>(A, Bx, acc, ST, ntS, WT, ntW);
      // over the lane's own row (its x2 reads are done).  Slots past P hold
      // a copy of the last pair's product; their weight rows are zero.
      cfor<0, Kd>([&](auto I) { tile[tid * KS + decltype(I)::value] = acc[decltype(I)::value]; });
    }
    // this wave's partial sums of the previous rounds (output rows k0 + 4 g +
    // rr of channel 16 ct + i) and its first weight block, requested before
    // the barrier so that they arrive while the other waves finish
    mixv4 macc[KTW][NCT], bw[KTW][NCT], yp[FINE ? KTW : 1][FINE ? NCT : 1];
    const float* const wb = WB + ((r * 16) * CoB + i) * 16 + g * 4;
    cfor<0, KTW>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      const int k0 = (wv + 4 * t) * 16;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const int co = ct * 16 + i;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int k = k0 + 4 * g + rr;
          const float v = (r > 0 && co < Co && k < Kd) ? y[(b * Co + co) * Kd + k] : 0.0f;
          macc[t][ct][rr] = FINE ? 0.0f : v;
          if constexpr (FINE) yp[t][ct][rr] = v;
        }
        bw[t][ct] = *reinterpret_cast<const mixv4*>(wb + ct * 256);
      }
    });
    __syncthreads();
    cfor<0, KTW>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      const int k0 = (wv + 4 * t) * 16;
      if (k0 < Kd) {  // wave-uniform
        const int ka = k0 + i < Kd ? k0 + i : Kd - 1;
        const bool kok = k0 + i < Kd;
        mixv4 bn[NCT];
        constexpr int RUN = 2;  // blocks of 16 pairs summed from zero (FINE)
        mixv4 run[FINE ? NCT : 1];
#pragma unroll 2
        for (int q = 0; q < 16; ++q) {
          float a[4];
#pragma unroll
          for (int sp = 0; sp < 4; ++sp) {
            const float v = tile[(16 * q + 4 * sp + g) * KS + ka];
            a[sp] = kok ? v : 0.0f;
          }
          const int qn = q + 1 < 16 ? q + 1 : q;
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct)
            bn[ct] = *reinterpret_cast<const mixv4*>(wb + int64_t(qn) * CoB * 16 + ct * 256);
#pragma unroll
          for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
              mixv4& s = FINE ? run[FINE ? ct : 0] : macc[t][ct];
              if (FINE && sp == 0 && q % RUN == 0) s = mixv4{0.0f, 0.0f, 0.0f, 0.0f};
              s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[sp], bw[t][ct][sp], s, 0, 0, 0);
            }
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            if (FINE && q % RUN == RUN - 1) macc[t][ct] += run[FINE ? ct : 0];
            bw[t][ct] = bn[ct];
          }
        }
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
          const int co = ct * 16 + i;
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const int k = k0 + 4 * g + rr;
            if constexpr (FINE) macc[t][ct][rr] += yp[t][ct][rr];
            if (co < Co && k < Kd) y[(b * Co + co) * Kd + k] = macc[t][ct][rr];
          }
        }
      }
    });
    __syncthreads();
  }
}

template <int L, typename TIn>
hipError_t launch_mix_fused_typed(const DevTables& t, const void* x1, const void* x2, const float* WB, float* y,
                                  int64_t B, int64_t C1, int64_t C2, int Co, int nct, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(B)), block(kMixThreads);
  const int64_t P = C1 * C2;
  const TIn* a = static_cast<const TIn*>(x1);
  const TIn* c = static_cast<const TIn*>(x2);
  const bool fine = P >= 128;  // shorter sums keep their order, and their bits
  switch (nct) {
    case 1:
      if (fine)
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 1, true>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      else
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 1, false>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      break;
    case 2:
      if (fine)
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 2, true>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      else
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 2, false>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      break;
    case 4:
      if (fine)
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 4, true>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      else
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 4, false>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      break;
    case 8:
      if (fine)
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 8, true>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      else
        hipLaunchKernelGGL((k_mix_fused<L, TIn, 8, false>), grid, block, 0, s, a, c, WB, y, C1, C2, Co, P, t.ST, t.ntS, t.WT, t.ntW);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int L>
hipError_t launch_mix_fused_one(const DevTables& t, const void* x1, const void* x2, int it, const float* WB, float* y,
                                int64_t B, int64_t C1, int64_t C2, int Co, int nct, hipStream_t s) {
  if (it == IN_BF16) return launch_mix_fused_typed<L, uint16_t>(t, x1, x2, WB, y, B, C1, C2, Co, nct, s);
  return launch_mix_fused_typed<L, float>(t, x1, x2, WB, y, B, C1, C2, Co, nct, s);
}

template <int L, int LO>
hipError_t launch_chain(const DevTables& t1, const DevTables& t2, int nu, const void* x, int in_type, int64_t n,
                        float* y, hipStream_t s) {
  const dim3 grid(unsigned((n + kTile - 1) / kTile)), block(kTile);
  if (in_type == IN_BF16)
    hipLaunchKernelGGL((k_self_stepwise_small<L, LO, uint16_t>), grid, block, 0, s,
                       static_cast<const uint16_t*>(x), y, n, nu, t1, t2);
  else
    hipLaunchKernelGGL((k_self_stepwise_small<L, LO, float>), grid, block, 0, s, static_cast<const float*>(x), y,
                       n, nu, t1, t2);
  return hipGetLastError();
}

}  // namespace

// (L1, L2, Lout) pair products, (L, nu, Lout) fused powers and (L, Lout) chains
// with a thread-per-product instantiation.  Everything else takes the generic
// path.  Powers and chains: every L and Lout in 1..3 (powers: nu in 2..4, the
// chain's nu is a loop), the degrees of the many-body features they are for.
// One launch of a lane per product against the generic kernel's workgroup per
// product (and per step of a chain, through a workspace), 64000 products fp32:
// chains of L = 3, nu = 2 / 3 / 4 to Lout = 2 574 / 1134 / 1687 -> 14 / 16 / 15
// us (launch-bound), fourth power of L = 3 to Lout = 3 583 -> 14 us; errors
// against 64-bit results 0.79 to 1.0 of the generic kernel's.
#define GTP_SMALL_PAIRS(X) \
  X(1, 1, 1) X(2, 2, 2) X(3, 3, 3) X(4, 4, 4) X(5, 5, 5) X(6, 6, 6) X(7, 7, 7) X(8, 8, 8) X(2, 2, 3) X(3, 2, 3) X(1, 2, 2) \
      X(2, 1, 3)
#define GTP_SMALL_POWERS_OF(X, a) \
  X(a, 2, 1) X(a, 2, 2) X(a, 2, 3) X(a, 3, 1) X(a, 3, 2) X(a, 3, 3) X(a, 4, 1) X(a, 4, 2) X(a, 4, 3)
#define GTP_SMALL_POWERS(X) GTP_SMALL_POWERS_OF(X, 1) GTP_SMALL_POWERS_OF(X, 2) GTP_SMALL_POWERS_OF(X, 3)
#define GTP_SMALL_CHAINS(X) X(1, 1) X(1, 2) X(1, 3) X(2, 1) X(2, 2) X(2, 3) X(3, 1) X(3, 2) X(3, 3)

hipError_t launch_full_small(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n,
                             float* y, int nu, const DegWeights& wt, hipStream_t s, bool* supported) {
  *supported = true;
  if (nu == 0) {
#define GTP_CASE(a, b, c) \
  if (t.L1 == a && t.L2 == b && t.Lout == c) return launch_one<a, b, c, 0>(t, x1, it1, x2, it2, n, y, wt, s, supported);
    GTP_SMALL_PAIRS(GTP_CASE)
#undef GTP_CASE
  } else {
    // power plans are built as (L, (nu - 1) L, Lout)
#define GTP_CASE(a, v, c) \
  if (nu == v && t.L1 == a && t.L2 == (v - 1) * a && t.Lout == c) \
    return launch_one<a, 0, c, v>(t, x1, it1, x1, it1, n, y, wt, s, supported);
    GTP_SMALL_POWERS(GTP_CASE)
#undef GTP_CASE
  }
  *supported = false;
  return hipSuccess;
}

template <int L>
hipError_t launch_pad_one(const void* x1, int it1, const void* x2, int it2, int64_t n, float* y, int k1, int k2,
                          int ko, hipStream_t s, bool* supported) {
  const dim3 grid(unsigned((n + kTile - 1) / kTile)), block(kTile);
  if (it1 == IN_F32 && it2 == IN_F32)
    hipLaunchKernelGGL((k_full_small_pad<L, float, float>), grid, block, 0, s, static_cast<const float*>(x1),
                       static_cast<const float*>(x2), y, n, k1, k2, ko);
  else if (it1 == IN_BF16 && it2 == IN_BF16)
    hipLaunchKernelGGL((k_full_small_pad<L, uint16_t, uint16_t>), grid, block, 0, s, static_cast<const uint16_t*>(x1),
                       static_cast<const uint16_t*>(x2), y, n, k1, k2, ko);
  else if (it1 == IN_F32 && it2 == IN_BF16)
    hipLaunchKernelGGL((k_full_small_pad<L, float, uint16_t>), grid, block, 0, s, static_cast<const float*>(x1),
                       static_cast<const uint16_t*>(x2), y, n, k1, k2, ko);
  else {
    *supported = false;
    return hipSuccess;
  }
  return hipGetLastError();
}

template <int L>
hipError_t launch_bwd_one(const float* dy, const void* x1, const void* x2, int it, int64_t n, float* dx1, float* dx2,
                          hipStream_t s, bool* supported) {
  const dim3 grid(unsigned((n + kTile - 1) / kTile)), block(kTile);
  // 16-byte runs straight into LDS when both input slabs are aligned
  const int dma = ((reinterpret_cast<uintptr_t>(x1) | reinterpret_cast<uintptr_t>(x2)) % 16) == 0;
  if (it == IN_F32)
    hipLaunchKernelGGL((k_bwd_small<L, float>), grid, block, 0, s, dy, static_cast<const float*>(x1),
                       static_cast<const float*>(x2), dx1, dx2, n, dma);
  else if (it == IN_BF16)
    hipLaunchKernelGGL((k_bwd_small<L, uint16_t>), grid, block, 0, s, dy, static_cast<const uint16_t*>(x1),
                       static_cast<const uint16_t*>(x2), dx1, dx2, n, dma);
  else {
    *supported = false;
    return hipSuccess;
  }
  return hipGetLastError();
}

hipError_t launch_bwd_small(int L, const float* dy, const void* x1, const void* x2, int it, int64_t n, float* dx1,
                            float* dx2, hipStream_t s, bool* supported) {
  *supported = true;
  switch (L) {
    case 1: return launch_bwd_one<1>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 2: return launch_bwd_one<2>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 3: return launch_bwd_one<3>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 4: return launch_bwd_one<4>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 5: return launch_bwd_one<5>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 6: return launch_bwd_one<6>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    case 7: return launch_bwd_one<7>(dy, x1, x2, it, n, dx1, dx2, s, supported);
    default: break;  // L = 8: the forward's registers are already all in use; two launches
  }
  *supported = false;
  return hipSuccess;
}

hipError_t launch_full_small_padded(int L, const void* x1, int it1, int k1, const void* x2, int it2, int k2,
                                    int64_t n, float* y, int ko, hipStream_t s, bool* supported) {
  *supported = true;
  switch (L) {
    case 1: return launch_pad_one<1>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 2: return launch_pad_one<2>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 3: return launch_pad_one<3>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 4: return launch_pad_one<4>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 5: return launch_pad_one<5>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 6: return launch_pad_one<6>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 7: return launch_pad_one<7>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    case 8: return launch_pad_one<8>(x1, it1, x2, it2, n, y, k1, k2, ko, s, supported);
    default: break;
  }
  *supported = false;
  return hipSuccess;
}

hipError_t launch_pairs_small(const DevTables& t, const void* x1, int it1, const void* x2, int it2, int64_t n,
                              float* y, const PairIdx& pi, hipStream_t s, bool* supported) {
  *supported = true;
  if (t.L1 == t.L2 && t.L2 == t.Lout) {
    switch (t.L1) {
      case 1: return launch_pairs_one<1>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 2: return launch_pairs_one<2>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 3: return launch_pairs_one<3>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 4: return launch_pairs_one<4>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 5: return launch_pairs_one<5>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 6: return launch_pairs_one<6>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 7: return launch_pairs_one<7>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      case 8: return launch_pairs_one<8>(t, x1, it1, x2, it2, n, y, pi, s, supported);
      default: break;
    }
  }
  *supported = false;
  return hipSuccess;
}

int mix_fused_nct(int Co) {
  const int n = (Co + 15) / 16;
  if (n <= 1) return 1;
  if (n <= 2) return 2;
  if (n <= 4) return 4;
  if (n <= 8) return 8;
  return 0;
}

hipError_t launch_mix_fused(const DevTables& t, const void* x1, const void* x2, int it, const float* WB, float* y,
                            int64_t B, int64_t C1, int64_t C2, int Co, hipStream_t s, bool* supported) {
  *supported = false;
  const int nct = mix_fused_nct(Co);
  if (nct == 0 || t.L1 != t.L2 || t.L2 != t.Lout || B <= 0 || B > 0x7fffffff || C1 <= 0 || C2 <= 0 ||
      C1 * C2 > 0x7fffffff - kMixThreads)
    return hipSuccess;
  if (it != IN_F32 && it != IN_BF16) return hipSuccess;
  *supported = true;
  switch (t.L1) {
    case 1: return launch_mix_fused_one<1>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 2: return launch_mix_fused_one<2>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 3: return launch_mix_fused_one<3>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 4: return launch_mix_fused_one<4>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 5: return launch_mix_fused_one<5>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 6: return launch_mix_fused_one<6>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 7: return launch_mix_fused_one<7>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    case 8: return launch_mix_fused_one<8>(t, x1, x2, it, WB, y, B, C1, C2, Co, nct, s);
    default: break;
  }
  *supported = false;
  return hipSuccess;
}

hipError_t launch_self_stepwise_small(const DevTables& t1, const DevTables& t2, int nu, const void* x, int in_type,
                                      int64_t n, float* y, hipStream_t s, bool* supported) {
  *supported = true;
#define GTP_CASE(a, c) \
  if (t1.L1 == a && t1.L2 == a && t1.Lout == c && (nu == 2 || (t2.L1 == c && t2.L2 == a && t2.Lout == c))) \
    return launch_chain<a, c>(t1, t2, nu, x, in_type, n, y, s);
  GTP_SMALL_CHAINS(GTP_CASE)
#undef GTP_CASE
  *supported = false;
  return hipSuccess;
}

}  // namespace gtp
