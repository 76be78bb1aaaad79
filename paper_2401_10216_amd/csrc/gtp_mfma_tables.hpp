// Operand images of the split-operand matrix-core product kernel
// (gtp_mfma.hip), made on the host.
//
// With L = L1 = L2 = Lout in {16, 32}: pairs j = 1..L of theta nodes (j,
// 2L + 1 - j) in NPT = L / 16 tiles of 16; m-parts 1..L in L / 4 quads of four
// orders of one parity, m = (L / 4) mi + 2 jq + 1 (odd, quads q < L / 8) or + 2
// (even), mi = 0..3, jq = q mod (L / 8), so that every quad has the same work;
// phi samples k = 0..Q in NMB blocks of 16.  par = 0, 1 picks the degrees l =
// m + par + 2 u.
//
// The theta synthesis runs on v_mfma_f32_16x16x4_f32 (lane 16 g + i: row or
// column i, contraction index g), STEPS(mi) steps of four degrees per order and
// parity; its images are fp32:
//   SA[tile][q][v][lane][4]  step f = 4 v + j of the quad's NSTEP, orders mi
//        ascending, par 0 before par 1, steps s ascending: S(l, m, pair
//        16 tile + i + 1) at u = 4 s + g
//   S0[task][v][lane][4]     the m = 0 tasks, step s = 4 v + j: S(2 (4 s + g) +
//        par, 0, pair 16 tile + i + 1) for task 2 tile + par, and the pole
//        (pair 0, column 0 only) for task 2 NPT + par
// Every other contraction runs on v_mfma_f32_16x16x32_f16 (contraction indices
// 8 g .. 8 g + 7 as the eight halves of a 16-byte load) with split operands: a
// value v enters as h1 + h2 with h1 = fp16(v), h2 = fp16(v - h1), a table entry
// the same way ("parts" 1 and 2), products accumulating in fp32.  Images:
//   TP[type][mb][lane][8]    phi synthesis, row i = sample 16 mb + i, types cos
//        even, cos odd, sin even, sin odd: L = 32: parts 1 of the four orders
//        of quad g of the class, then parts 2; L = 16: lane groups 0, 1 hold
//        part 1 of quad g twice, groups 2, 3 part 2 of quad g - 2 twice
//   TA[type][part][lane][8]  phi analysis, row 4 a + b = order 2 (4 b + a) + 2
//        (even) or + 1 (odd; L = 16: b < 2), w_k trig(m phi_k) with w_k = 1/2
//        at k = 0, Q: L = 32: samples 16 (j / 4) + 4 g + j % 4; L = 16: no part
//        index, parts 1 of samples 4 g + j, j < 4, then parts 2; row 2 of type
//        0 is order 0
//   WC[q][mi][par][part][lane][8]  theta analysis, column i = u: pairs 8 g + j
//        + 1 (L = 32); L = 16: no part index, lane groups 0, 1 part 1 of pairs
//        8 g + j + 1, groups 2, 3 part 2 of pairs 8 (g - 2) + j + 1
//   W0[x][part][lane][8]     the same for m = 0: x < NE0 even degrees l = 2 (16
//        x + i), the others odd ones
// The phi tables TP and TA are stored times PHI, the m = 0 values that meet TP's
// sums (S0, not the poles) too, and W over PHI^3 (two syntheses, one analysis):
// two fp16 parts leave up to 2^-23 of an entry, twice fp32's rounding, but the
// 52 samples of L = 16 have only 13 different magnitudes, and there is a scale at
// which all of them have short expansions (5.4e-9 rms and 1.0e-8 at most are
// left, 2.9e-8 and 6.0e-8 at scale 1, 1.4e-8 rms in fp32).
// W is stored times 2^kw (largest entry in [2^10, 2^11)), so that the second
// parts of its typical entries stay normal halves.
//
// The index images give, per thread, where its operands and results lie in
// the workgroup's LDS images (byte offsets, rows of k1, k2 inputs and of kk
// outputs; entries past a row's degrees point at a slot of zeros, results
// past it at a spare slot):
//   gather[wave][lane][GATHER]  input coefficient of step f, then of the wave's
//        m = 0 task's steps, as 4 times the element's index in the stage (x1's
//        rows of k1 from 0, x2's rows of k2 from 4 K, zeros at 8 K)
//   scatter[wave][lane][12]     output image offsets of (c = 2 mi + par, column
//        i): cos in the low half, sin in the high one; entry 8 the wave's m = 0
//        one
#pragma once

#include <cstdint>
#include <vector>

#include "gtp_tables.hpp"

namespace gtp {

// Sizes and offsets of the images of degree L.
template <int L>
struct MfmaGeo {
  static_assert(L == 16 || L == 32, "matrix-core product kernel degrees");
  static constexpr int NPT = L / 16, NQ = L / 4, NSL = L / 8;
  static constexpr int NP = (3 * L + 1 + 3) / 4 * 4, Q = NP / 4, NMB = (Q + 1 + 15) / 16;
  static constexpr int NE0 = (L / 2 + 1 + 15) / 16, NPART = NE0 + (L / 2 + 15) / 16;
  static constexpr int steps(int mi) { return L == 16 ? (mi < 2 ? 2 : 1) : 4 - mi; }
  // first step of (mi, par)
  static constexpr int step0(int mi, int par) {
    int f = 0;
    for (int k = 0; k < mi; ++k) f += 2 * steps(k);
    return f + par * steps(mi);
  }
  static constexpr int order(int q, int mi) {
    return (L / 4) * mi + 2 * (q % NSL) + (q / NSL ? 2 : 1);
  }
  static constexpr int NSTEP = L == 16 ? 12 : 20, NS0 = (L / 2 + 1 + 3) / 4, NT0 = 2 * NPT + 2;
  static constexpr int SAV = NSTEP / 4, S0V = (NS0 + 3) / 4;  // 16-byte loads per lane
  // fp32 images (floats)
  static constexpr int SA = 0, S0 = SA + NPT * NQ * SAV * 256, FLOATS = S0 + NT0 * S0V * 256;
  // fp16 images (halves)
  static constexpr int TAI = L == 16 ? 1 : 2;     // stored images per phi-analysis operand
  static constexpr int WPARTS = L == 16 ? 1 : 2;  // and per theta-analysis operand
  static constexpr int FR = 64 * 8;               // halves of one image
  static constexpr double PHI = L == 16 ? 14910466.0 / 16777216.0 : 1.0;
  static constexpr int TP = 0, TA = TP + 4 * NMB * FR, WC = TA + 4 * TAI * FR, W0 = WC + NQ * 8 * WPARTS * FR,
                       HALVES = W0 + NPART * WPARTS * FR;
  // index images: halves of the gather, words of the scatter, per thread
  static constexpr int GATHER = (NSTEP + NS0 + 7) / 8 * 8, SCATTER = 12, NTH = 64 * NQ;
};

// fp16 bits of a double (round to nearest even, subnormals kept) and back.
uint16_t half_bits(double v);
double half_value(uint16_t h);

// The images of a plan's tables; empty unless L1 = L2 = Lout in {16, 32}.
struct MfmaImages {
  std::vector<double> f;    // fp32 images
  std::vector<uint16_t> h;  // fp16 images
  int kw = 0;               // exponent of the theta-analysis scale
};
MfmaImages build_mfma_images(const Tables& t);

// The index images (gather, then scatter) of the degree-L kernel for rows of
// k1, k2 inputs and min(ko, (L + 1)^2) outputs; L in {16, 32}.
std::vector<uint16_t> build_mfma_index(int L, int k1, int k2, int ko);

}  // namespace gtp
