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
// All contractions run on v_mfma_f32_16x16x32_f16 with split operands (the
// part-2 x part-2 products, 2^-22 of a term, left out); the accumulators, F2
// and the sum over c2 are fp32.  Powers of two bring every input channel, every
// output channel's weights and its sampled sums into the half type's range.  In the sum over
// c1 the channels' own scales must stand: channels whose scales lie within
// 2^kClass of the largest enter together, at that one's scale; smaller ones,
// if a batch entry has such, in further turns at theirs (one output channel
// may weigh only them).  The accumulator layout of the sampling (rows =
// channels) is the operand layout of the contraction over c1, so F1 stays in
// registers; F2 goes through the wave's own LDS columns, and the sampled sums
// through LDS to the analysis.
//
// Bound: issue of the matrix instructions (L = 6, C1 = C2 = Co = 32, per wave
// and batch entry: 1152 over c1, 144 for the sampling, 96 for the analysis, 16
// cycles each) and of the vector instructions beside them, mostly the
// multiply-adds over c2 and the splits; the two do not overlap on a SIMD.
// Waves of their own columns rather than of their own channels: F1, F2 and the
// sums then never leave the wave until the analysis.  Loads go out together
// (staged rows, tiles of the quadrature's values, weights channels ahead):
// with one load per wait the kernel took 652 us instead of 386 (B = 8192).
// There 1.05 ms -> 0.40 ms against the pair products (k_mix_fused), error
// against 64-bit results 5.8e-7 -> 1.7e-7; L = 8, 600 entries of 64 x 64 -> 64
// channels 1.94 -> 0.42 ms; L = 1, 500 of those 151 -> 93 us; C1 C2 = 128 at
// L <= 4 the same as before.
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
constexpr int kXs = 6;      // input channels below 2^kXs
constexpr int kWs = 12;     // weights below 2^kWs
constexpr int kGs = 13;     // sampled sums below 2^kGs
constexpr int kClass = 10;  // scales of one turn: samples below 2^14, the smallest channels' near 1
constexpr int kNone = -140; // the exponent of zeros
constexpr int kBad = 1 << 20;     // of a channel with a NaN or Inf: in every turn
constexpr int kDone = -(1 << 20); // the turn of an entry that has had all its channels

__device__ __forceinline__ float finite_abs(float v) {
  const float a = fabsf(v);
  return a < __builtin_inff() ? a : 0.0f;  // NaN and Inf set no scale
}
// e with v < 2^e, at least kNone (so for v = 0)
__device__ __forceinline__ int exponent_of(float v) {
  const int e = v > 0.0f ? __builtin_amdgcn_frexp_expf(v) : kNone;
  return e < kNone ? kNone : e;
}

// The weights' operand images: for every 16-row tile of co, chunk of CK c1's
// and c2, lane 16 g + i holds row co = 16 tile + i, contraction indices c1 = 16
// (j / 4) + 4 g + j % 4 of the chunk (CK = 32) or 4 g + j % 4 twice (CK = 16),
// part 1 then part 2, W times 2^(kWs - ew[co]), ew[co] the exponent of that
// output channel's weights.  s1, s2: strides of c1 and c2 in W.  One
// workgroup per tile (y) and share of the c2's (x); each takes its tile's
// exponents from the rows themselves.
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
      for (int j = 0; j < 8; ++j) mx = fmaxf(mx, finite_abs(v[j]));
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
      v[j] = co < Co && c1 < C1 ? ldexpf(W[co * per + c1 * s1 + c2 * s2], kWs - ex) : 0.0f;
    }
    const u4 a = split4(v[0], v[1], v[2], v[3]), b = split4(v[4], v[5], v[6], v[7]);
    u4* const o = img + ((ct * nck + ck) * C2 + c2) * 128 + lane;
    o[0] = u4{a[0], a[1], b[0], b[1]};
    o[64] = u4{a[2], a[3], b[2], b[3]};
  }
}

template <int L, typename TX, int CK, int NCOT>
__global__ __launch_bounds__(64 * MixqGeo<L>::NWQ) __attribute__((amdgpu_waves_per_eu(2))) void k_mixq(
    const TX* __restrict__ x1, const TX* __restrict__ x2, const u4* __restrict__ img, const int* __restrict__ ew,
    float* __restrict__ y, int64_t B, int64_t C1, int64_t C2, int64_t Co) {
  using G = MixqGeo<L>;
  constexpr int ka = MixqImages<L>::ka;
  const u4* const yimg = reinterpret_cast<const u4*>(MixqImages<L>::get());
  constexpr int K = G::K, S = K | 1, T = G::T, NB = G::NB, U = NB * T, KS = G::KS, NWQ = G::NWQ;
  // a wave's own LDS: 32 staged rows, then F2's columns, then its sampled sums
  constexpr int REG = (32 * S > 32 * 16 * U ? 32 * S : 32 * 16 * U);
  static_assert(REG * 4 >= 8192 && T <= 8, "the sampled sums of a 16-row tile in the wave's region");
  __shared__ __align__(16) float lds[NWQ * REG + NWQ * 16];
  lds_poison(lds, NWQ * REG + NWQ * 16);
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const st = lds + wave * REG;
  float* const mxb = lds + NWQ * REG;  // the output rows' maxima per wave
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
        cfor<0, 8>([&](auto J) { m = fmaxf(m, finite_abs(v[decltype(J)::value])); });
      }
      return __builtin_amdgcn_readfirstlane(exponent_of(wave_max(m)));
    };
    e1[b] = one1 ? kNone : largest(x1 + bb * C1 * K, C1 * K);
    e2[b] = one2 ? kNone : largest(x2 + bb * C2 * K, C2 * K);
  });

  // samples of the channels c0 .. c0 + 16 RT - 1 of batch entry b at this
  // wave's points, each channel times 2^(kXs + kYs) over its own power of two:
  // out(tile, row tile, values, exponents), rows = channels (register r of lane
  // group g: channel c0 + 16 rt + 4 g + r), columns = points; before them
  // all(e), the largest of the exponents, where these are all C channels
  auto sample = [&](auto RTC, const TX* x, int64_t C, int64_t c0, int b, auto&& all, auto&& out) {
    constexpr int RT = decltype(RTC)::value, NR = 16 * RT;
    int lane = threadIdx.x & 63;
    hold(lane);  // or the addresses of all stages are made ahead and spilled
    const int g = lane >> 4, i = lane & 15;
    const int64_t bb = b0 + b < B ? b0 + b : B - 1;
    const int rows = int(C - c0 < NR ? C - c0 : NR);
    const TX* const xr = x + (bb * C + c0) * K;
    {
      constexpr int NL = (NR * K + 63) / 64;
      float v[NL];
      const int last = rows * K - 1;
      cfor<0, NL>([&](auto J) {
        const int q = lane + 64 * decltype(J)::value;
        v[decltype(J)::value] = mq_ld(xr, q < last ? q : last);
      });
      cfor<0, NL>([&](auto J) {
        const int q = lane + 64 * decltype(J)::value;
        float w = q <= last ? v[decltype(J)::value] : 0.0f;
        hold(w);
        if (q < NR * K) st[S == K ? q : q / K * S + q % K] = w;
      });
    }
    // the rows' exponents: 64 / NR lanes to a row
    float mx = 0.0f;
    int bad = 0;
    cfor<0, (K + 64 / NR - 1) / (64 / NR)>([&](auto J) {
      const int k = lane / NR + 64 / NR * decltype(J)::value;
      const float w = st[(lane % NR) * S + (k < K ? k : 0)];
      mx = fmaxf(mx, finite_abs(w));
      bad |= !(fabsf(w) < __builtin_inff());
    });
#pragma unroll
    for (int d = NR; d < 64; d *= 2) {
      mx = fmaxf(mx, __shfl_xor(mx, d));
      bad |= __shfl_xor(bad, d);
    }
    const int er = bad ? kBad : exponent_of(mx);
    if (C <= NR) {
      int em = bad ? kNone : er;
#pragma unroll
      for (int d = 1; d < NR; d *= 2) {
        const int o = __shfl_xor(em, d);
        em = o > em ? o : em;
      }
      all(__builtin_amdgcn_readfirstlane(em));
    }
    int ed[RT][4];  // of the result rows
    cfor<0, RT>([&](auto RR) {
      cfor<0, 4>([&](auto R) {
        ed[decltype(RR)::value][decltype(R)::value] =
            __shfl(er, 16 * decltype(RR)::value + 4 * g + decltype(R)::value);
      });
    });
    u4 a[RT][KS][2];
    cfor<0, RT>([&](auto RR) {
      const int es = __shfl(er, 16 * decltype(RR)::value + i), ea = kXs - (es == kBad ? 0 : es);
      cfor<0, KS>([&](auto SS) {
        constexpr int rt = decltype(RR)::value, s = decltype(SS)::value;
        float v[8];
        cfor<0, 8>([&](auto J) {
          constexpr int j = decltype(J)::value;
          const int k = 32 * s + 8 * g + j;
          float w = st[(16 * rt + i) * S + (k < K ? k : 0)];
          hold(w);  // read by every lane, then selected: no branch
          v[j] = k < K ? ldexpf(w, ea) : 0.0f;
        });
        const u4 p = split4(v[0], v[1], v[2], v[3]), q = split4(v[4], v[5], v[6], v[7]);
        a[rt][s][0] = u4{p[0], p[1], q[0], q[1]};
        a[rt][s][1] = u4{p[2], p[3], q[2], q[3]};
      });
    });
    // the points' values a tile ahead
    const u4* const yt = yimg + G::YS / 8 + wave * T * KS * 128 + lane;
    u4 yn[KS][2];
    cfor<0, KS>([&](auto SS) {
      yn[decltype(SS)::value][0] = yt[decltype(SS)::value * 128];
      yn[decltype(SS)::value][1] = yt[decltype(SS)::value * 128 + 64];
    });
    cfor<0, T>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      u4 yv[KS][2];
      cfor<0, KS>([&](auto SS) {
        constexpr int s = decltype(SS)::value;
        yv[s][0] = yn[s][0];
        yv[s][1] = yn[s][1];
        if constexpr (t + 1 < T) {
          yn[s][0] = yt[((t + 1) * KS + s) * 128];
          yn[s][1] = yt[((t + 1) * KS + s) * 128 + 64];
        }
      });
      __builtin_amdgcn_sched_barrier(0);
      f4 d[RT];
      cfor<0, RT>([&](auto RR) { d[decltype(RR)::value] = f4{0.0f, 0.0f, 0.0f, 0.0f}; });
      cfor<0, KS>([&](auto SS) {
        constexpr int s = decltype(SS)::value;
        cfor<0, RT>([&](auto RR) {
          constexpr int rt = decltype(RR)::value;
          d[rt] = mfma(a[rt][s][0], yv[s][1], d[rt]);
        });
        cfor<0, RT>([&](auto RR) {
          constexpr int rt = decltype(RR)::value;
          d[rt] = mfma(a[rt][s][1], yv[s][0], d[rt]);
        });
      });
      // the large terms last: one rounding of the sum per instruction
      cfor<0, KS>([&](auto SS) {
        constexpr int s = decltype(SS)::value;
        cfor<0, RT>([&](auto RR) {
          constexpr int rt = decltype(RR)::value;
          d[rt] = mfma(a[rt][s][0], yv[s][0], d[rt]);
        });
      });
      cfor<0, RT>([&](auto RR) { out(TT, RR, d[decltype(RR)::value], ed[decltype(RR)::value]); });
    });
  };

  const int64_t ct0 = int64_t(blockIdx.y) * NCOT;  // this workgroup's output channels: 16 NCOT from 16 ct0
  f4 acc[U][NCOT];
  cfor<0, U>([&](auto UU) {
    cfor<0, NCOT>([&](auto CC) { acc[decltype(UU)::value][decltype(CC)::value] = f4{0.0f, 0.0f, 0.0f, 0.0f}; });
  });
  // turns: the channels of x1 whose exponents lie in (ec - kClass, ec], from
  // the largest down; done when no channel is left below
  int ec[NB];
  cfor<0, NB>([&](auto BB) { ec[decltype(BB)::value] = e1[decltype(BB)::value]; });
  for (bool first = true, more = true; more; first = false) {
    int below[NB];  // the largest exponent under this turn's
    cfor<0, NB>([&](auto BB) { below[decltype(BB)::value] = kNone; });
    for (int64_t ck = 0; ck < nc1; ++ck) {
      u4 f1[U][2];  // F1 as operands: parts 1 and 2 of eight channels (CK = 32), or both of four
      cfor<0, NB>([&](auto BB) {
        constexpr int b = decltype(BB)::value;
        f4 lo[T];
        int under = kNone;
        auto all = [&](int e) {
          e1[b] = e;
          if (first) ec[b] = e;
        };
        sample(std::integral_constant<int, CK / 16>{}, x1, C1, ck * CK, b, all,
               [&](auto TT, auto RR, f4 d, const int (&e)[4]) {
          constexpr int t = decltype(TT)::value, u = b * T + t;
          cfor<0, 4>([&](auto R) {
            constexpr int r = decltype(R)::value;
            const int rel = e[r] - ec[b];
            // (a NaN or Inf reaches every sample of its channel, and stands)
            if (e[r] != kBad) d[r] = rel <= 0 && rel > -kClass ? ldexpf(d[r], rel) : 0.0f;
            if constexpr (t == 0) {
              if (rel <= -kClass) under = e[r] > under ? e[r] : under;
            }
          });
          if constexpr (CK == 16) {
            f1[u][0] = split4(d[0], d[1], d[2], d[3]);
          } else if constexpr (decltype(RR)::value == 0) {
            lo[t] = d;
          } else {
            const u4 p = split4(lo[t][0], lo[t][1], lo[t][2], lo[t][3]), q = split4(d[0], d[1], d[2], d[3]);
            f1[u][0] = u4{p[0], p[1], q[0], q[1]};
            f1[u][1] = u4{p[2], p[3], q[2], q[3]};
          }
        });
  #pragma unroll
        for (int d = 16; d < 64; d *= 2) {
          const int o = __shfl_xor(under, d);
          under = o > under ? o : under;
        }
        under = __builtin_amdgcn_readfirstlane(under);
        below[b] = under > below[b] ? under : below[b];
      });
      for (int64_t c20 = 0; c20 < C2; c20 += 32) {
        const int n2 = int(C2 - c20 < 32 ? C2 - c20 : 32);
        // F2 of the next 32 channels over its input's power of two, and the
        // contraction's scales taken back, to LDS [channel][tile, point]
        f4 f2[U][2];
        cfor<0, NB>([&](auto BB) {
          constexpr int b = decltype(BB)::value;
          int back = 0;
          auto all = [&](int e) { e2[b] = e; };
          sample(std::integral_constant<int, 2>{}, x2, C2, c20, b, all, [&](auto TT, auto RR, f4 d, const int (&e)[4]) {
            if constexpr (decltype(TT)::value == 0 && decltype(RR)::value == 0)
              back = ec[b] - e1[b] - e2[b] - 2 * (kXs + kYs) - kWs;
            cfor<0, 4>([&](auto R) {
              constexpr int r = decltype(R)::value;
              d[r] = ldexpf(d[r], e[r] + back);
            });
            f2[b * T + decltype(TT)::value][decltype(RR)::value] = d;
          });
        });
        cfor<0, 2>([&](auto RR) {
          cfor<0, 4>([&](auto R) {
            constexpr int rt = decltype(RR)::value, r = decltype(R)::value;
            cfor<0, U>([&](auto UU) {
              constexpr int u = decltype(UU)::value;
              st[(16 * rt + 4 * g + r) * (16 * U) + 16 * u + i] = f2[u][rt][r];
            });
          });
        });
        const u4* wp[NCOT];
        cfor<0, NCOT>([&](auto CC) {
          constexpr int cc = decltype(CC)::value;
          const int64_t ct = ct0 + cc < (Co + 15) / 16 ? ct0 + cc : ct0;
          wp[cc] = img + ((ct * nc1 + ck) * C2 + c20) * 128 + lane;
        });
        // the weights PD channels ahead, as the registers allow
        constexpr int PD = U * NCOT <= 4 ? 4 : U * NCOT <= 8 ? 2 : 1;
        u4 wr[PD][NCOT][2];
        cfor<0, PD>([&](auto PP) {
          constexpr int j = decltype(PP)::value;
          const int cn = j < n2 ? j : n2 - 1;
          cfor<0, NCOT>([&](auto CC) {
            constexpr int cc = decltype(CC)::value;
            wr[j][cc][0] = wp[cc][cn * 128];
            wr[j][cc][1] = wp[cc][cn * 128 + 64];
          });
        });
        for (int cb = 0; cb < n2; cb += PD) {
          cfor<0, PD>([&](auto JJ) {
            constexpr int ring = decltype(JJ)::value;
            const int c = cb + ring;
            if (PD > 1 && c >= n2) return;
            u4 w[NCOT][2];
            const int cn = c + PD < n2 ? c + PD : n2 - 1;
            cfor<0, NCOT>([&](auto CC) {
              constexpr int cc = decltype(CC)::value;
              w[cc][0] = wr[ring][cc][0];
              w[cc][1] = wr[ring][cc][1];
              wr[ring][cc][0] = wp[cc][cn * 128];
              wr[ring][cc][1] = wp[cc][cn * 128 + 64];
            });
            float f[U];
            cfor<0, U>([&](auto UU) { f[decltype(UU)::value] = st[c * (16 * U) + 16 * decltype(UU)::value + i]; });
            // GU tiles at a time, so that no instruction waits for the one before
            constexpr int GU = NCOT == 1 ? 4 : 2;
            cfor<0, (U + GU - 1) / GU>([&](auto PP) {
              constexpr int u0 = GU * decltype(PP)::value, nu = U - u0 < GU ? U - u0 : GU;
              f4 d[nu][NCOT];
              cfor<0, nu>([&](auto UU) {
                cfor<0, NCOT>([&](auto CC) {
                  d[decltype(UU)::value][decltype(CC)::value] =
                      mfma(w[decltype(CC)::value][1], f1[u0 + decltype(UU)::value][0], f4{0.0f, 0.0f, 0.0f, 0.0f});
                });
              });
              if constexpr (CK == 32)
                cfor<0, nu>([&](auto UU) {
                  cfor<0, NCOT>([&](auto CC) {
                    f4& r = d[decltype(UU)::value][decltype(CC)::value];
                    r = mfma(w[decltype(CC)::value][0], f1[u0 + decltype(UU)::value][1], r);
                  });
                });
              cfor<0, nu>([&](auto UU) {
                cfor<0, NCOT>([&](auto CC) {
                  f4& r = d[decltype(UU)::value][decltype(CC)::value];
                  r = mfma(w[decltype(CC)::value][0], f1[u0 + decltype(UU)::value][0], r);
                });
              });
              cfor<0, nu>([&](auto UU) {
                cfor<0, NCOT>([&](auto CC) {
                  constexpr int u = u0 + decltype(UU)::value;
                  acc[u][decltype(CC)::value] += f[u] * d[decltype(UU)::value][decltype(CC)::value];
                });
              });
              __builtin_amdgcn_sched_barrier(0);
            });
            __builtin_amdgcn_sched_barrier(0);
          });
          asm volatile("" ::: "memory");  // or the loads move down to their use
        }
      }
    }
    more = false;
    cfor<0, NB>([&](auto BB) {
      constexpr int b = decltype(BB)::value;
      more = more || below[b] > kNone;
      ec[b] = below[b] > kNone ? below[b] : kDone;
    });
  }
  // ---- analysis, one batch entry and 16 output channels at a time
  cfor<0, NB>([&](auto BB) {
    cfor<0, NCOT>([&](auto CC) {
      constexpr int b = decltype(BB)::value, cc = decltype(CC)::value;
      const int64_t co0 = 16 * (ct0 + cc);
      // an exponent for each output row: one output channel's sums may lie any
      // way below another's
      int eg[4];
      cfor<0, 4>([&](auto R) {
        constexpr int r = decltype(R)::value;
        float mx = 0.0f;
        cfor<0, T>([&](auto TT) { mx = fmaxf(mx, finite_abs(acc[b * T + decltype(TT)::value][cc][r])); });
#pragma unroll
        for (int d = 1; d < 16; d *= 2) mx = fmaxf(mx, __shfl_xor(mx, d));
        if constexpr (NWQ > 1) {
          if (i == 0) mxb[wave * 16 + 4 * g + r] = mx;
        } else {
          eg[r] = exponent_of(mx);
        }
      });
      if constexpr (NWQ > 1) {
        __syncthreads();
        cfor<0, 4>([&](auto R) {
          constexpr int r = decltype(R)::value;
          float mx = 0.0f;
          cfor<0, NWQ>([&](auto W) { mx = fmaxf(mx, mxb[decltype(W)::value * 16 + 4 * g + r]); });
          eg[r] = exponent_of(mx);
        });
      }
      // parts 1, then 2: [row][point of the tile][tile]
      u4* const gs = reinterpret_cast<u4*>(st);
      cfor<0, 4>([&](auto R) {
        constexpr int r = decltype(R)::value;
        float v[8];
        cfor<0, 8>([&](auto TT) {
          constexpr int t = decltype(TT)::value;
          v[t] = t < T ? ldexpf(acc[b * T + (t < T ? t : 0)][cc][r], kGs - eg[r]) : 0.0f;
        });
        const u4 p = split4(v[0], v[1], v[2], v[3]), q = split4(v[4], v[5], v[6], v[7]);
        gs[(4 * g + r) * 16 + i] = u4{p[0], p[1], q[0], q[1]};
        gs[256 + (4 * g + r) * 16 + i] = u4{p[2], p[3], q[2], q[3]};
      });
      __syncthreads();
      for (int kt = wave; kt < G::KT; kt += NWQ) {
        // the large terms in two sums per wave's points, the small ones apart
        f4 d = {0.0f, 0.0f, 0.0f, 0.0f}, hi[NWQ][2];
        cfor<0, NWQ>([&](auto WW) {
          constexpr int w = decltype(WW)::value;
          u4 ya[4][2];  // a wave's points at a time, all loads first
          cfor<0, 4>([&](auto SS) {
            constexpr int s = decltype(SS)::value;
            ya[s][0] = yimg[G::YA / 8 + (kt * NWQ * 4 + 4 * w + s) * 128 + lane];
            ya[s][1] = yimg[G::YA / 8 + (kt * NWQ * 4 + 4 * w + s) * 128 + 64 + lane];
          });
          cfor<0, 4>([&](auto SS) {
            constexpr int s = decltype(SS)::value;
            const u4* const ga = reinterpret_cast<const u4*>(lds + w * REG) + i * 16 + 4 * s + g;
            const u4 a1 = ga[0], a2 = ga[256];
            d = mfma(a1, ya[s][1], d);
            d = mfma(a2, ya[s][0], d);
            hi[w][s / 2] = mfma(a1, ya[s][0], s % 2 ? hi[w][s / 2] : f4{0.0f, 0.0f, 0.0f, 0.0f});
          });
          hi[w][0] += hi[w][1];
          if constexpr (w > 0) hi[0][0] += hi[w][0];
        });
        d += hi[0][0];
        const int k = 16 * kt + i, ex = e1[b] + e2[b] - kGs - ka;
        cfor<0, 4>([&](auto R) {
          constexpr int r = decltype(R)::value;
          const int64_t co = co0 + 4 * g + r;
          if (b0 + b < B && co < Co && k < K) y[((b0 + b) * Co + co) * K + k] = ldexpf(d[r], ex + eg[r] + ew[co]);
        });
      }
      __syncthreads();  // the regions are read: the next rows, or stage, may land there
    });
  });
}

int64_t image_bytes(int64_t Co, int64_t C1, int64_t C2) {
  return (Co + 15) / 16 * (C1 <= 16 ? 1 : (C1 + 31) / 32) * C2 * 2048;
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

int64_t mixq_steps(int64_t C) { return C <= 16 ? 2 : 3 * ((C + 31) / 32); }

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
