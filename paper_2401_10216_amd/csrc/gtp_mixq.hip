// Channel mixing in the sample domain (the channel-mixing rule of the appendix,
// Implementation Details), equal degrees L = 1..8:
//   y[b, co] = sum_{c1, c2} W[co, c1, c2] GTP(x1[b, c1], x2[b, c2])
//            = P_L( sum_{c2} F2[c2] ( sum_{c1} W[co, c1, c2] F1[c1] ) )
// with F1, F2 the functions of the channels, taken at the Q points of a
// quadrature exact to degree 3 L.  Each channel's function is sampled once
// per batch entry, where forming the pair products transforms both inputs for
// each of the C1 C2 pairs; the inner sum over c1 is a matrix contraction at
// every point (rows co, contraction index c1, columns the points), and the sum
// over c2 one multiply-add per point on its result.
//
// All contractions run on v_mfma_f32_16x16x32_bf16 with operands in three bf16
// parts (gtp_split.hpp), which hold fp32 values exactly and, unlike fp16 parts,
// whatever the sizes of the values beside them: a channel, weight or output far
// below its neighbours keeps its bits.  Six products of parts stand for one (b2
// x b3 and b3 x b3, 2^-24 of a term at worst, are left out; three products
// where the inputs are bf16); the accumulators, F2 and the sum over c2 are fp32.
// One power of two per batch entry and input, and per output channel's
// weights, keeps products of large and small factors within fp32's exponents:
// inputs below 2^kX1 and 2^kX2, weights below 2^kW.  That leaves a channel its
// bits down to 2^-148 (3e-45) of the largest value of its entry, a weight down
// to 2^-110 (8e-34) of its output channel's largest.  The accumulator layout of the sampling (rows = channels) is the operand layout of
// the contraction over c1, so F1 stays in registers; F2 goes through the wave's
// own LDS columns, and the sampled sums through LDS to the analysis.
//
// Bound: issue of the matrix instructions (L = 6, C1 = C2 = Co = 32, per wave
// and batch entry: 2304 over c1, 288 for the sampling, 192 for the analysis, 16
// cycles each, 68 % of the SIMDs' cycles by counters) and of the vector
// instructions beside them (25 %), mostly the multiply-adds over c2 and the
// splits; the two do not overlap on a SIMD.
// Waves of their own columns rather than of their own channels: F1, F2 and the
// sums then never leave the wave until the analysis.  Loads go out together
// (staged rows, tiles of the quadrature's values, weights channels ahead).
// Measured, L = 6, 8192 entries of 32 x 32 -> 32: 521 us, against 1029 us of the
// pair products (k_mix_fused), error against 64-bit results 1.1e-7 (7.5e-8 to
// 1.9e-7 over degrees 1..8, 128 to 4096 pairs; pair products 1.4e-7 to 1.8e-7).  With operands in two fp16 parts, three products and scales shared by
// the channels of a turn, by a row of weights and by an output row, 352 us, but a
// weight 1e-6 of its row's largest kept 17 bits and one 1e-12 of it none.
#include "gtp_ct.hpp"
#include "gtp_device.hpp"
#include "gtp_mixq.hpp"
#include "gtp_mixq_tables.hpp"
#include "gtp_split.hpp"

namespace gtp {
namespace {

#include "gtp_mixq_consts.inc"

__device__ __forceinline__ float mq_ld(const float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float mq_ld(const uint16_t* p, int64_t i) { return __uint_as_float(uint32_t(p[i]) << 16); }

// The compiler knows nothing of the value past this point (it can neither be
// loaded again nor later).
template <typename T>
__device__ __forceinline__ void hold(T& v) {
  asm volatile("" : "+v"(v));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int d = 1; d < 64; d *= 2) v = fmaxf(v, __shfl_xor(v, d));
  return v;
}
// Exponents of the scaled inputs and weights.  A sample is below 2^5 of its
// channel's largest coefficient (degrees <= 8), the analysis adds 2^5: outputs
// stay below 2^(kX1 + kW + kX2 + 15) C1 C2 < 2^127 (C1 C2 < 2^36: the weights
// fit the memory).
constexpr int kX1 = 38, kW = 0, kX2 = 38;

// e with v < 2^e (0 for v = 0; of no consequence for Inf, whose channel and
// outputs are NaN)
__device__ __forceinline__ int exponent_of(float v) { return __builtin_amdgcn_frexp_expf(v); }

// The wave's LDS writes before, its reads after (or the other way round): one
// lane reads what another wrote.  The hardware keeps a wave's LDS accesses in
// order; this keeps the compiler from moving them.
__device__ __forceinline__ void lds_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// f(part of one operand, part of the other) for the six products of parts that
// count, the smallest first.
template <typename F>
__device__ __forceinline__ void each_pair(F&& f) {
  using P1 = std::integral_constant<int, 0>;
  using P2 = std::integral_constant<int, 1>;
  using P3 = std::integral_constant<int, 2>;
  f(P3{}, P1{});
  f(P2{}, P2{});
  f(P1{}, P3{});
  f(P2{}, P1{});
  f(P1{}, P2{});
  f(P1{}, P1{});
}

// The weights' operand images: for every 16-row tile of co, chunk of CK c1's
// and c2, lane 16 g + i holds row co = 16 tile + i, three operands: CK = 32:
// parts 1, 2, 3 of c1 = 16 (j / 4) + 4 g + j % 4 of the chunk, j < 8; CK = 16:
// of c1 = 4 g + j, j < 4, parts (1, 1), (2, 2), (1, 3); W times 2^(kW - ew[co]),
// ew[co] the exponent of that output channel's weights.  s1, s2: strides of c1
// and c2 in W.  One workgroup per tile (y) and share of the c2's (x); each takes
// its tile's exponents from the rows themselves.
template <int CK>
__global__ __launch_bounds__(1024) void k_mixq_weights(const float* __restrict__ W, u4* __restrict__ img,
                                                       int* __restrict__ ew, int64_t Co, int64_t C1, int64_t C2,
                                                       int64_t s1, int64_t s2) {
  __shared__ float red[16];
  lds_poison(red, 16);
  const int64_t per = C1 * C2, ct = blockIdx.y;
  {
    // a wave to a row, eight loads in flight
    const int64_t co = 16 * ct + threadIdx.x / 64;
    const float* const row = W + (co < Co ? co : Co - 1) * per;
    float mx = 0.0f;
    for (int64_t e0 = threadIdx.x & 63; e0 < per; e0 += 8 * 64) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = row[e0 + 64 * j < per ? e0 + 64 * j : e0];
#pragma unroll
      for (int j = 0; j < 8; ++j) mx = fmaxf(mx, fabsf(v[j]));
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = co < Co ? mx : 0.0f;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  const int ex = exponent_of(red[i]);
  const int64_t co = 16 * ct + i, nck = (C1 + CK - 1) / CK;
  if (blockIdx.x == 0 && threadIdx.x < 16) ew[co] = ex;
  for (int64_t f = int64_t(blockIdx.x) * 16 + threadIdx.x / 64; f < nck * C2; f += int64_t(gridDim.x) * 16) {
    const int64_t ck = f / C2, c2 = f - ck * C2;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t c1 = CK * ck + (CK == 32 ? 16 * (j >> 2) : 0) + 4 * g + (j & 3);
      v[j] = co < Co && c1 < C1 ? ldexpf(W[co * per + c1 * s1 + c2 * s2], kW - ex) : 0.0f;
    }
    u4 p[3];
    split3x8(v, p);
    u4* const o = img + ((ct * nck + ck) * C2 + c2) * 192 + lane;
    if constexpr (CK == 32) {
      o[0] = p[0];
      o[64] = p[1];
      o[128] = p[2];
    } else {
      o[0] = p[0];  // (j and j + 4 are the same channel)
      o[64] = p[1];
      o[128] = u4{p[0][0], p[0][1], p[2][0], p[2][1]};
    }
  }
}

template <int L, typename TX, int CK, int NCOT>
__global__ __launch_bounds__(64 * MixqGeo<L>::NWQ) __attribute__((amdgpu_waves_per_eu(2))) void k_mixq(
    const TX* __restrict__ x1, const TX* __restrict__ x2, const u4* __restrict__ img, const int* __restrict__ ew,
    float* __restrict__ y, int64_t B, int64_t C1, int64_t C2, int64_t Co) {
  using G = MixqGeo<L>;
  const u4* const yimg = reinterpret_cast<const u4*>(MixqImages<L>::get());
  constexpr int K = G::K, S = K | 1, T = G::T, NB = G::NB, U = NB * T, KS = G::KS, NWQ = G::NWQ;
  constexpr int XP = sizeof(TX) == 2 ? 1 : 3;  // parts of an input value
  // a wave's own LDS: 32 staged rows and, in their place (after them where
  // several batch entries are staged in turn), F2's columns; then its sampled sums
  constexpr int F2 = NB > 1 ? 32 * S : 0, STG = 32 * S > F2 + 32 * 16 * U ? 32 * S : F2 + 32 * 16 * U;
  constexpr int REG = ((STG > 3072 ? STG : 3072) + 3) / 4 * 4;  // three parts of the sums of a 16-row tile: 3072
  static_assert(T <= 8, "one operand holds the wave's tiles");
  __shared__ __align__(16) float lds[NWQ * REG];
  lds_poison(lds, NWQ * REG);
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const st = lds + wave * REG;
  const int64_t b0 = int64_t(blockIdx.x) * NB;
  const int64_t nc1 = (C1 + CK - 1) / CK;

  // the exponents of each batch entry's two inputs, where its channels are
  // more than one stage takes (else that stage finds them)
  const bool one1 = C1 <= CK, one2 = C2 <= 32;
  int e1[NB], e2[NB];
  cfor<0, NB>([&](auto BB) {
    constexpr int b = decltype(BB)::value;
    const int64_t bb = b0 + b < B ? b0 + b : B - 1;  // past the last entry: the last one again
    auto largest = [&](const TX* r, int64_t n) {
      float m = 0.0f;
      for (int64_t e0 = lane; e0 - lane < n; e0 += 8 * 64) {  // eight loads in flight
        float v[8];
        cfor<0, 8>([&](auto J) {
          const int64_t e = e0 + 64 * decltype(J)::value;
          v[decltype(J)::value] = mq_ld(r, e < n ? e : n - 1);
        });
        cfor<0, 8>([&](auto J) { m = fmaxf(m, fabsf(v[decltype(J)::value])); });
      }
      return __builtin_amdgcn_readfirstlane(exponent_of(wave_max(m)));
    };
    e1[b] = one1 ? 0 : largest(x1 + bb * C1 * K, C1 * K);
    e2[b] = one2 ? 0 : largest(x2 + bb * C2 * K, C2 * K);
  });

  // samples of the channels c0 .. c0 + 16 RT - 1 of batch entry b at this
  // wave's points, times 2^(top - e): out(tile, row tile, values), rows =
  // channels (register r of lane group g: channel c0 + 16 rt + 4 g + r), columns
  // = points.  own: these are all C channels, e is found here.
  auto sample = [&](auto RTC, const TX* x, int64_t C, int64_t c0, int b, int top, int& e, bool own, auto&& out) {
    constexpr int RT = decltype(RTC)::value, NR = 16 * RT;
    int lane = threadIdx.x & 63;
    hold(lane);  // or the addresses of all stages are made ahead and spilled
    const int g = lane >> 4, i = lane & 15;
    const int64_t bb = b0 + b < B ? b0 + b : B - 1;
    const int rows = int(C - c0 < NR ? C - c0 : NR);
    const TX* const xr = x + (bb * C + c0) * K;
    lds_exchange();
    {
      constexpr int NL = (NR * K + 63) / 64;
      float v[NL];
      const int last = rows * K - 1;
      cfor<0, NL>([&](auto J) {
        const int q = lane + 64 * decltype(J)::value;
        v[decltype(J)::value] = mq_ld(xr, q < last ? q : last);
      });
      if (own) {
        float m = 0.0f;
        cfor<0, NL>([&](auto J) { m = fmaxf(m, fabsf(v[decltype(J)::value])); });
        e = __builtin_amdgcn_readfirstlane(exponent_of(wave_max(m)));
      }
      cfor<0, NL>([&](auto J) {
        const int q = lane + 64 * decltype(J)::value;
        float w = q <= last ? ldexpf(v[decltype(J)::value], top - e) : 0.0f;
        hold(w);
        if (q < NR * K) st[S == K ? q : q / K * S + q % K] = w;
      });
    }
    lds_exchange();
    u4 a[RT][KS][XP];
    cfor<0, RT>([&](auto RR) {
      cfor<0, KS>([&](auto SS) {
        constexpr int rt = decltype(RR)::value, s = decltype(SS)::value;
        float v[8];
        cfor<0, 8>([&](auto J) {
          constexpr int j = decltype(J)::value;
          const int k = 32 * s + 8 * g + j;
          float w = st[(16 * rt + i) * S + (k < K ? k : 0)];
          hold(w);  // read by every lane, then selected: no branch
          v[j] = k < K ? w : 0.0f;
        });
        u4 p[3];
        split3x8(v, p);
        cfor<0, XP>([&](auto PP) { a[rt][s][decltype(PP)::value] = p[decltype(PP)::value]; });
      });
    });
    lds_exchange();
    // the points' values, a tile ahead where the registers allow
    constexpr bool AHEAD = KS < 3;
    const u4* const yt = yimg + G::YS / 8 + wave * T * KS * 192 + lane;
    u4 yn[AHEAD ? KS : 1][3];
    if constexpr (AHEAD)
      cfor<0, 3 * KS>([&](auto Q) { yn[decltype(Q)::value / 3][decltype(Q)::value % 3] = yt[decltype(Q)::value * 64]; });
    cfor<0, T>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      u4 yv[KS][3];
      cfor<0, 3 * KS>([&](auto Q) {
        constexpr int s = decltype(Q)::value / 3, p = decltype(Q)::value % 3;
        if constexpr (AHEAD) {
          yv[s][p] = yn[s][p];
          if constexpr (t + 1 < T) yn[s][p] = yt[((t + 1) * KS * 3 + decltype(Q)::value) * 64];
        } else {
          yv[s][p] = yt[(t * KS * 3 + decltype(Q)::value) * 64];
        }
      });
      __builtin_amdgcn_sched_barrier(0);
      f4 d[RT];
      cfor<0, RT>([&](auto RR) { d[decltype(RR)::value] = f4{0.0f, 0.0f, 0.0f, 0.0f}; });
      // the small terms of all steps first, then the large ones: one rounding
      // of the sum per instruction
      auto add = [&](auto PX, auto PY) {
        if constexpr (decltype(PX)::value < XP)
          cfor<0, KS>([&](auto SS) {
            cfor<0, RT>([&](auto RR) {
              constexpr int rt = decltype(RR)::value, s = decltype(SS)::value;
              d[rt] = mfma_bf(a[rt][s][decltype(PX)::value < XP ? decltype(PX)::value : 0], yv[s][decltype(PY)::value], d[rt]);
            });
          });
      };
      each_pair(add);
      cfor<0, RT>([&](auto RR) { out(TT, RR, d[decltype(RR)::value]); });
    });
  };

  const int64_t ct0 = int64_t(blockIdx.y) * NCOT;  // this workgroup's output channels: 16 NCOT from 16 ct0
  f4 acc[U][NCOT];
  cfor<0, U>([&](auto UU) {
    cfor<0, NCOT>([&](auto CC) { acc[decltype(UU)::value][decltype(CC)::value] = f4{0.0f, 0.0f, 0.0f, 0.0f}; });
  });
  constexpr int FP = CK == 32 ? 3 : 2;
  for (int64_t ck = 0; ck < nc1; ++ck) {
    // F1 as operands: CK = 32: the three parts of eight channels; CK = 16: parts
    // (1, 2) and (3, 1) of four
    u4 f1[U][FP];
    cfor<0, NB>([&](auto BB) {
      constexpr int b = decltype(BB)::value;
      f4 lo;
      sample(std::integral_constant<int, CK / 16>{}, x1, C1, ck * CK, b, kX1, e1[b], one1, [&](auto TT, auto RR, f4 d) {
        constexpr int u = b * T + decltype(TT)::value;
        if constexpr (CK == 16) {
          uint32_t p[2], q[2], r[2];
          split3(d[0], d[1], p[0], q[0], r[0]);
          split3(d[2], d[3], p[1], q[1], r[1]);
          f1[u][0] = u4{p[0], p[1], q[0], q[1]};
          f1[u][1] = u4{r[0], r[1], p[0], p[1]};
        } else if constexpr (decltype(RR)::value == 0) {
          lo = d;
        } else {
          split3x8({lo[0], lo[1], lo[2], lo[3], d[0], d[1], d[2], d[3]}, f1[u]);
        }
      });
    });
    for (int64_t c20 = 0; c20 < C2; c20 += 32) {
      const int n2 = int(C2 - c20 < 32 ? C2 - c20 : 32);
      // F2 of the next 32 channels to LDS [channel][tile, point]
      cfor<0, NB>([&](auto BB) {
        constexpr int b = decltype(BB)::value;
        sample(std::integral_constant<int, 2>{}, x2, C2, c20, b, kX2, e2[b], one2, [&](auto TT, auto RR, f4 d) {
          cfor<0, 4>([&](auto R) {
            constexpr int rt = decltype(RR)::value, r = decltype(R)::value, u = b * T + decltype(TT)::value;
            st[F2 + (16 * rt + 4 * g + r) * (16 * U) + 16 * u + i] = d[r];
          });
        });
      });
      lds_exchange();
      const u4* wp[NCOT];
      cfor<0, NCOT>([&](auto CC) {
        constexpr int cc = decltype(CC)::value;
        const int64_t ct = ct0 + cc < (Co + 15) / 16 ? ct0 + cc : ct0;
        wp[cc] = img + ((ct * nc1 + ck) * C2 + c20) * 192 + lane;
      });
      // the weights PD channels ahead, as the registers allow
      constexpr int PD = U * NCOT <= 4 ? 4 : U * NCOT <= 8 ? 2 : 1;
      u4 wr[PD][NCOT][3];
      cfor<0, PD>([&](auto PP) {
        constexpr int j = decltype(PP)::value;
        const int cn = j < n2 ? j : n2 - 1;
        cfor<0, 3 * NCOT>([&](auto Q) {
          constexpr int cc = decltype(Q)::value / 3, p = decltype(Q)::value % 3;
          wr[j][cc][p] = wp[cc][cn * 192 + 64 * p];
        });
      });
      for (int cb = 0; cb < n2; cb += PD) {
        cfor<0, PD>([&](auto JJ) {
          constexpr int ring = decltype(JJ)::value;
          const int c = cb + ring;
          if (PD > 1 && c >= n2) return;
          u4 w[NCOT][3];
          const int cn = c + PD < n2 ? c + PD : n2 - 1;
          cfor<0, 3 * NCOT>([&](auto Q) {
            constexpr int cc = decltype(Q)::value / 3, p = decltype(Q)::value % 3;
            w[cc][p] = wr[ring][cc][p];
            wr[ring][cc][p] = wp[cc][cn * 192 + 64 * p];
          });
          float f[U];
          cfor<0, U>([&](auto UU) { f[decltype(UU)::value] = st[F2 + c * (16 * U) + 16 * decltype(UU)::value + i]; });
          // GU tiles at a time, so that no instruction waits for the one before
          constexpr int GU = NCOT == 1 ? 4 : 2;
          cfor<0, (U + GU - 1) / GU>([&](auto PP) {
            constexpr int u0 = GU * decltype(PP)::value, nu = U - u0 < GU ? U - u0 : GU;
            f4 d[nu][NCOT];
            cfor<0, nu * NCOT>([&](auto Q) {
              d[decltype(Q)::value / NCOT][decltype(Q)::value % NCOT] = f4{0.0f, 0.0f, 0.0f, 0.0f};
            });
            auto add = [&](auto PW, auto PF) {
              cfor<0, nu * NCOT>([&](auto Q) {
                constexpr int u = decltype(Q)::value / NCOT, cc = decltype(Q)::value % NCOT;
                d[u][cc] = mfma_bf(w[cc][decltype(PW)::value], f1[u0 + u][decltype(PF)::value], d[u][cc]);
              });
            };
            if constexpr (CK == 32) {
              each_pair(add);
            } else {
              add(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});  // 1 x 3, 3 x 1
              add(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{});  // 2 x 1, 2 x 2
              add(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});  // 1 x 1, 1 x 2
            }
            cfor<0, nu * NCOT>([&](auto Q) {
              constexpr int u = decltype(Q)::value / NCOT, cc = decltype(Q)::value % NCOT;
              acc[u0 + u][cc] += f[u0 + u] * d[u][cc];
            });
            __builtin_amdgcn_sched_barrier(0);
          });
          __builtin_amdgcn_sched_barrier(0);
        });
        asm volatile("" ::: "memory");  // or the loads move down to their use
      }
    }
  }
  // ---- analysis, one batch entry and 16 output channels at a time
  cfor<0, NB>([&](auto BB) {
    cfor<0, NCOT>([&](auto CC) {
      constexpr int b = decltype(BB)::value, cc = decltype(CC)::value;
      const int64_t co0 = 16 * (ct0 + cc);
      // the three parts: [part][row][point of the tile][tile]
      lds_exchange();
      u4* const gs = reinterpret_cast<u4*>(st);
      cfor<0, 4>([&](auto R) {
        constexpr int r = decltype(R)::value;
        float v[8];
        cfor<0, 8>([&](auto TT) {
          constexpr int t = decltype(TT)::value;
          v[t] = t < T ? acc[b * T + (t < T ? t : 0)][cc][r] : 0.0f;
        });
        u4 p[3];
        split3x8(v, p);
        cfor<0, 3>([&](auto PP) { gs[256 * decltype(PP)::value + (4 * g + r) * 16 + i] = p[decltype(PP)::value]; });
      });
      __syncthreads();
      for (int kt = wave; kt < G::KT; kt += NWQ) {
        // the large terms in two sums per wave's points, the small ones apart
        f4 d = {0.0f, 0.0f, 0.0f, 0.0f}, hi[NWQ][2];
        cfor<0, NWQ>([&](auto WW) {
          constexpr int w = decltype(WW)::value;
          u4 ya[4][3];  // a wave's points at a time, all loads first
          cfor<0, 12>([&](auto Q) {
            ya[decltype(Q)::value / 3][decltype(Q)::value % 3] =
                yimg[G::YA / 8 + ((kt * NWQ + w) * 12 + decltype(Q)::value) * 64 + lane];
          });
          cfor<0, 4>([&](auto SS) {
            constexpr int s = decltype(SS)::value;
            const u4* const ga = reinterpret_cast<const u4*>(lds + w * REG) + i * 16 + 4 * s + g;
            const u4 a[3] = {ga[0], ga[256], ga[512]};
            each_pair([&](auto PA, auto PY) {
              constexpr int pa = decltype(PA)::value, py = decltype(PY)::value;
              if constexpr (pa + py > 0) d = mfma_bf(a[pa], ya[s][py], d);
            });
            hi[w][s / 2] = mfma_bf(a[0], ya[s][0], s % 2 ? hi[w][s / 2] : f4{0.0f, 0.0f, 0.0f, 0.0f});
          });
          hi[w][0] += hi[w][1];
          if constexpr (w > 0) hi[0][0] += hi[w][0];
          __builtin_amdgcn_sched_barrier(0);  // one wave's points in registers at a time
        });
        d += hi[0][0];
        const int k = 16 * kt + i, ex = e1[b] + e2[b] - kX1 - kW - kX2;
        cfor<0, 4>([&](auto R) {
          constexpr int r = decltype(R)::value;
          const int64_t co = co0 + 4 * g + r;
          if (b0 + b < B && co < Co && k < K) y[((b0 + b) * Co + co) * K + k] = ldexpf(d[r], ex + ew[co]);
        });
      }
      __syncthreads();  // the regions are read: the next rows may land there
    });
  });
}

int64_t image_bytes(int64_t Co, int64_t C1, int64_t C2) {
  return (Co + 15) / 16 * (C1 <= 16 ? 1 : (C1 + 31) / 32) * C2 * 3072;
}

template <int L, typename TX, int CK, int NCOT>
hipError_t launch_typed(const MixqArgs& a, hipStream_t s) {
  using G = MixqGeo<L>;
  u4* const img = static_cast<u4*>(a.work);
  int* const ew = reinterpret_cast<int*>(static_cast<char*>(a.work) + image_bytes(a.Co, a.C1, a.C2));
  const int64_t nck = (a.C1 + CK - 1) / CK, share = (nck * a.C2 + 15) / 16;
  hipLaunchKernelGGL((k_mixq_weights<CK>), dim3(unsigned(share < 32 ? share : 32), unsigned((a.Co + 15) / 16)),
                     dim3(1024), 0, s, a.W, img, ew, a.Co, a.C1, a.C2, a.s1, a.s2);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(unsigned((a.B + G::NB - 1) / G::NB), unsigned((a.Co + 16 * NCOT - 1) / (16 * NCOT)));
  const dim3 block(64 * G::NWQ);
  hipLaunchKernelGGL((k_mixq<L, TX, CK, NCOT>), grid, block, 0, s, static_cast<const TX*>(a.x1),
                     static_cast<const TX*>(a.x2), img, ew, a.y, a.B, a.C1, a.C2, a.Co);
  return hipGetLastError();
}

template <int L, typename TX>
hipError_t launch_sized(const MixqArgs& a, hipStream_t s) {
  if (a.C1 <= 16) return a.Co <= 16 ? launch_typed<L, TX, 16, 1>(a, s) : launch_typed<L, TX, 16, 2>(a, s);
  return a.Co <= 16 ? launch_typed<L, TX, 32, 1>(a, s) : launch_typed<L, TX, 32, 2>(a, s);
}

template <int L>
hipError_t launch_degree(const MixqArgs& a, hipStream_t s) {
  return a.in_type == IN_BF16 ? launch_sized<L, uint16_t>(a, s) : launch_sized<L, float>(a, s);
}

}  // namespace

int64_t mixq_work_bytes(int64_t Co, int64_t C1, int64_t C2) {
  return image_bytes(Co, C1, C2) + (Co + 15) / 16 * 64;
}

hipError_t launch_mixq(int L, const MixqArgs& a, hipStream_t s, bool* supported) {
  *supported = true;
  switch (L) {
    case 1: return launch_degree<1>(a, s);
    case 2: return launch_degree<2>(a, s);
    case 3: return launch_degree<3>(a, s);
    case 4: return launch_degree<4>(a, s);
    case 5: return launch_degree<5>(a, s);
    case 6: return launch_degree<6>(a, s);
    case 7: return launch_degree<7>(a, s);
    case 8: return launch_degree<8>(a, s);
    default: break;
  }
  *supported = false;
  return hipSuccess;
}

}  // namespace gtp
