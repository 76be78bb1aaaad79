// Backward pass of the weighted Gaunt tensor product (Sec. 3.1, eq.
// tp-eq-mul-weight) at equal degrees L = 1..8 in one kernel: with
//   z  = GTP(w1 x1, w2 x2),   u1 = GTP(wout dy, w2 x2),   u2 = GTP(wout dy, w1 x1)
// it writes dx1 = w1 u1 and dx2 = w2 u2 and sums the weights' gradients
//   dwout[r, l] = sum <dy, z>_l,  dw1[r, l] = sum <x1, u1>_l,  dw2[r, l] = sum <x2, u2>_l
// over the products of each weight row.
//
// One lane owns one product at a time (the thread-per-product core).  Lane v
// of the V in the grid takes the products v, v + V, ..; V is a multiple of the
// channel count, so a lane's products share their weight row and its sums
// over them stay with it (in registers, from degree 5 in LDS) until the end;
// a second kernel adds the lanes of a row in a fixed order.  The three
// products of a lane run as a loop that is not unrolled (one copy of the
// core).  Each needs all three rows: two as operands (registers, LDS tile),
// the third for the dot products; rows already on chip are kept, the others
// read again while they are still in the caches, and neither u1, u2 nor z goes
// to memory.
//
// Bound: vector issue (73 % of the SIMDs' cycles at degree 4 by counters) and HBM
// (three products per five rows moved).  Before, the three products went through
// memory to separate reductions, 17 rows in all: forward and backward of 1M
// products of degree 4 with per-channel weights 0.66 -> 0.28 ms; bf16 inputs,
// which had no weighted fp32 x bf16 kernel and took the workgroup kernel, 65536
// products of degree 8 3.01 -> 0.12 ms.
#include "gtp_small_core.hpp"
#include "gtp_wbwd.hpp"

namespace gtp {
namespace {

constexpr int kRedThreads = 1024;

// The sums over a lane's products: registers where the core leaves room,
// else LDS columns of its own.
template <int L>
constexpr bool sums_in_regs() {
  return L <= 4;
}

template <int L, typename TX>
__global__ __launch_bounds__(kTile) __attribute__((amdgpu_waves_per_eu(sums_in_regs<L>() ? 3 : 2))) void k_wbwd_small(
    const TX* __restrict__ x1, const TX* __restrict__ x2, const float* __restrict__ dy, const float* __restrict__ w1,
    const float* __restrict__ w2, const float* __restrict__ wo, float* __restrict__ dx1, float* __restrict__ dx2,
    float* __restrict__ partial, int64_t n, int64_t V, int64_t C, int per_channel, int need) {
  constexpr int K = csh(L), S = lds_stride(K), NS = 3 * (L + 1);
  constexpr bool REGS = sums_in_regs<L>();
  __shared__ __align__(16) float lds[kTile * S + (REGS ? 0 : NS * kTile)];
  lds_poison(lds, kTile * S + (REGS ? 0 : NS * kTile));
  float* const tile = lds;
  float* const col = lds + kTile * S;  // [sum][lane]
  float sum[REGS ? NS : 1];
  cfor<0, NS>([&](auto J) {
    if constexpr (REGS) {
      sum[decltype(J)::value] = 0.0f;
    } else {
      col[decltype(J)::value * kTile + threadIdx.x] = 0.0f;
    }
  });
  const int64_t v0 = int64_t(blockIdx.x) * kTile;
  const int64_t wrow = per_channel ? (v0 + threadIdx.x) % C * (L + 1) : 0;
  for (int64_t p0 = v0; p0 < n; p0 += V) {
    const int cnt = int((n - p0) < kTile ? (n - p0) : kTile);
    float xa[K], acc[K];
    // product 0: z from (w1 x1, w2 x2), with dy; 1: u1 from (wout dy, w2 x2),
    // with x1; 2: u2 from (wout dy, w1 x1), with x2
#pragma unroll 1
    for (int g = 0; g < 3; ++g) {
      if (!(need >> g & 1)) continue;
      // indices from an opaque copy of the lane id: rebuilt, not held across the core
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      const int64_t row = (p0 + (tid < cnt ? tid : cnt - 1)) * K;  // lanes past the end repeat the last product
      auto load_a = [&](auto src, const float* w) {
        cfor<0, K>([&](auto I) { xa[decltype(I)::value] = ld_in(src + row, decltype(I)::value); });
        if (w) scale_by_degree<L, K>(w + wrow, [&](auto I) -> float& { return xa[decltype(I)::value]; });
      };
      if (g == 0) {
        load_a(x1, w1);
      } else if (g == 1 || !(need & 2)) {
        load_a(dy, wo);  // kept for product 2
      }
#pragma unroll
      for (int i = 0; i < K; ++i) asm volatile("" : "+v"(xa[i]));  // (no synthesis hoisted across the products)
      // the tile: x2 for the first of products 0 and 1, x1 for product 2
      if (g == 2 || g == 0 || !(need & 1)) {
        const TX* const x = g == 2 ? x1 : x2;
        const float* const w = g == 2 ? w1 : w2;
        cfor<0, K>([&](auto I) { tile[tid * S + decltype(I)::value] = ld_in(x + row, decltype(I)::value); });
        if (w)
          scale_by_degree<L, K>(w + wrow, [&](auto I) -> float& { return tile[tid * S + decltype(I)::value]; });
      }
      gtp_core_lit<L>(RegX<K>{xa}, LdsX{tile, tid * S}, acc);
      int td = threadIdx.x;
      asm volatile("" : "+v"(td));
      const int64_t rw = (p0 + (td < cnt ? td : cnt - 1)) * K;
      // per-degree dot products with the third row
      auto dots = [&](auto src, auto G) {
        constexpr int gg = decltype(G)::value;
        cfor<0, L + 1>([&](auto LL) {
          constexpr int l = decltype(LL)::value;
          float d = 0.0f;
          cfor<l * l, (l + 1) * (l + 1)>([&](auto I) {
            constexpr int i = decltype(I)::value;
            d = fmaf(ld_in(src + rw, i), acc[i], d);
          });
          d = td < cnt ? d : 0.0f;
          if constexpr (REGS) {
            sum[gg * (L + 1) + l] += d;
          } else {
            col[(gg * (L + 1) + l) * kTile + td] += d;
          }
        });
      };
      float* out = nullptr;
      const float* w = nullptr;
      if (g == 0) {
        dots(dy, std::integral_constant<int, 0>{});
      } else if (g == 1) {
        if (need & 16) dots(x1, std::integral_constant<int, 1>{});
        out = dx1;
        w = w1;
      } else {
        if (need & 32) dots(x2, std::integral_constant<int, 2>{});
        out = dx2;
        w = w2;
      }
      if (out) {
        if (w) scale_by_degree<L, K>(w + wrow, [&](auto I) -> float& { return acc[decltype(I)::value]; });
        __syncthreads();
        store_rows<K, K>(out, p0, cnt, tile, acc, td);
      }
      __syncthreads();  // the tile's reads are done before the next rows land there
    }
  }
  // this lane's sums: [sum][lane of the grid]; with one weight row, the
  // wave's sums [sum][wave]
  if (!partial) return;
  cfor<0, NS>([&](auto J) {
    constexpr int j = decltype(J)::value;
    float s;
    if constexpr (REGS) {
      s = sum[j];
    } else {
      s = col[j * kTile + threadIdx.x];
    }
    if (per_channel) {
      partial[j * V + v0 + threadIdx.x] = s;
    } else {
#pragma unroll
      for (int d = 1; d < 64; d *= 2) s += __shfl_xor(s, d);
      if (threadIdx.x == 0) partial[j * gridDim.x + blockIdx.x] = s;
    }
  });
}

// dw[r, l] = sum over the entries e = r, r + R, .. < N of partial[j][e], j the
// sum's number: 64 (or R) rows per workgroup, the entries of a row dealt to
// slices of threads, the slices added pairwise.
__global__ __launch_bounds__(kRedThreads) void k_wbwd_sum(const float* __restrict__ partial, int64_t N, int64_t R,
                                                          int L, float* __restrict__ dwo, float* __restrict__ dw1,
                                                          float* __restrict__ dw2) {
  __shared__ float red[kRedThreads];
  lds_poison(red, kRedThreads);
  const int cw = R < 64 ? int(R) : 64, slices = kRedThreads / cw;
  const int c = threadIdx.x % cw, s = threadIdx.x / cw;
  const int64_t r = int64_t(blockIdx.x) * cw + c;
  const int j = blockIdx.y, g = j / (L + 1), l = j - g * (L + 1);
  float* const dw = g == 0 ? dwo : g == 1 ? dw1 : dw2;
  if (!dw) return;  // whole-workgroup exit
  float a = 0.0f;
  if (r < R && s < slices) {
    const float* const p = partial + j * N;
#pragma unroll 4
    for (int64_t e = r + s * R; e < N; e += slices * R) a += p[e];
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int h = 512; h > 0; h /= 2) {
    if (s < h && s + h < slices) red[s * cw + c] += red[(s + h) * cw + c];
    __syncthreads();
  }
  if (s == 0 && r < R) dw[r * (L + 1) + l] = red[c];
}

int64_t gcd64(int64_t a, int64_t b) {
  while (b) {
    const int64_t t = a % b;
    a = b;
    b = t;
  }
  return a;
}

template <int L, typename TX>
hipError_t launch_typed(const WbwdArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.waves)), block(kTile);
  hipLaunchKernelGGL((k_wbwd_small<L, TX>), grid, block, 0, s, static_cast<const TX*>(a.x1),
                     static_cast<const TX*>(a.x2), a.dy, a.w1, a.w2, a.wo, a.dx1, a.dx2, a.partial, a.n,
                     a.waves * kTile, a.C, a.per_channel, a.need);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.partial) return e;
  const int64_t R = a.per_channel ? a.C : 1, N = a.per_channel ? a.waves * kTile : a.waves;
  const int64_t cw = R < 64 ? R : 64;
  hipLaunchKernelGGL(k_wbwd_sum, dim3(unsigned((R + cw - 1) / cw), unsigned(3 * (L + 1))), dim3(kRedThreads), 0, s,
                     a.partial, N, R, L, a.dwo, a.dw1, a.dw2);
  return hipGetLastError();
}

template <int L>
hipError_t launch_degree(const WbwdArgs& a, hipStream_t s) {
  return a.in_type == IN_BF16 ? launch_typed<L, uint16_t>(a, s) : launch_typed<L, float>(a, s);
}

}  // namespace

int64_t wbwd_waves(int64_t n, int64_t C, int per_channel) {
  // one product per lane (any count: lane = product), or about eight waves
  // per CU (more lanes would only make the last sums longer) in whole
  // weight-row cycles
  const int64_t all = (n + kTile - 1) / kTile, unit = per_channel ? C / gcd64(C, kTile) : 1;
  const int64_t w = (2048 + unit - 1) / unit * unit;
  return all < w ? all : w;
}

int64_t wbwd_partial_floats(int L, int64_t waves, int per_channel) {
  return 3 * (L + 1) * waves * (per_channel ? kTile : 1);
}

hipError_t launch_wbwd_small(int L, const WbwdArgs& a, hipStream_t s, bool* supported) {
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
