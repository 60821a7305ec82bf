// HIP kernels of the Image Source Method for gfx950 (MI355X).
//
// Three kernels per call:
//   tables_kernel      per (RIR, axis, lattice index): square of the displacement
//                      of the image coordinate from the receiver in samples
//                      (FP64) and the axis factor of the reflection gain (Sec. 2.1, Eq. (1)
//                      and the gain rule below it); for directional receivers
//                      also the displacement's share of the projection onto the
//                      receiver's orientation. Also flags invalid pairs.
//   accumulate_kernel  per work item (RIR, output tile, slab of the image shell):
//                      enumerates exactly the lattice images whose window can
//                      reach the tile, computes each image's delay and amplitude
//                      (Eq. (2)-(4), times the receiver's polar pattern when
//                      directional) and adds its Hann-windowed sinc (Eq. (5),
//                      (6)): FP32 calls sum the moments of the images' delay
//                      fractions per integer delay and convolve these with the
//                      taps' polynomials once per item, table taps (Eq. (9))
//                      do so with pulses per table phase; FP16 taps, and the others
//                      in calls of few images per tile, are added image by image into
//                      wave-private FP32 LDS tiles.
//   reduce_kernel      sums, in a fixed order, the partial tiles of tiles that
//                      were split over several work items.
//
// Squared distances and delays are FP64 (gfx950 issues FP64 additions,
// multiplications, fused multiply-adds, roundings and conversions at the FP32
// rate: 4.5 to 5.4 clocks per wave instruction measured against 4.35), so the
// fractional delay keeps ~1e-8 sample accuracy at 1e5-sample distances; gains,
// taps and accumulation are FP32.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <type_traits>

#include "ism.h"
#include "ism_internal.h"
#include "ism_math.h"

namespace ism {

// Bits of a staged record that carry the tile-local base of an image (its
// integer delay minus the tile start), and the mask that extracts them.
constexpr int kBaseBits = (TILE <= 256) ? 8 : 9;
constexpr uint32_t kBaseMask = (1u << kBaseBits) - 1u;
static_assert(TILE <= (1 << kBaseBits), "tile-local bases must fit the record");
// b^e for e >= 0 by binary powering (0^0 = 1), in FP64: the gain of an image many
// reflections deep is accurate to its FP32 rounding.
__device__ double int_pow(double b, int e) {
  double r = 1.0;
  while (e > 0) {
    if (e & 1) r *= b;
    e >>= 1;
    b *= b;
  }
  return r;
}

// ---------------------------------------------------------------------------
// Compile-time constants of the tap loop (evaluated in double by the compiler).
// ---------------------------------------------------------------------------
constexpr double kPi = 3.14159265358979323846;

constexpr double cx_sin(double x) {  // |x| <= pi: Taylor series to double accuracy
  double term = x, sum = x;
  for (int k = 1; k < 30; ++k) {
    term *= -x * x / ((2.0 * k) * (2.0 * k + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double cx_cos(double x) {
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 30; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}

// FP16 taps. For one image with fractional delay f, tap j (Eq. (6) at
// v = j - f) is A s_j(t) with t = f - 1/2 in [-1/2, 1/2) and
//   s_j(t) = sinc(j - f) (1 + cos(2 pi (j - f) / W)) / 2,
// an entire function of t. Each s_j is replaced by its interpolant of degree
// SPD at the Chebyshev nodes of [-1/2, 1/2] (interpolation error < 6e-5),
// written as c0 + t q(t), q = c1 + c2 t + ... + c5 t^4. A tap then adds
// A c0 in FP32 and q(t) (A t), with q evaluated in packed FP16 (two taps per
// register) and the product and sum in FP32. FP16 rounding of q and t bounds
// the tap error by ~6e-4 A at the central taps and ~2.5e-4 A elsewhere.
constexpr int SPD = 5;
template <int WT>
struct SincPoly {
  float c[SPD + 1][WT];  // c[k][jj] multiplies t^k for tap j = jj + 1 - W/2
};
constexpr double s_tap(int j, double t, int wt) {
  const double f = t + 0.5;  // in (0, 1) at the nodes, so j - f != 0
  const double v = j - f;
  const double sg = (j % 2 == 0) ? -1.0 : 1.0;  // sin(pi v) = sg sin(pi f)
  return sg * cx_sin(kPi * f) / (kPi * v) * 0.5 * (1.0 + cx_cos(2.0 * kPi * v / wt));
}
template <int WT>
constexpr SincPoly<WT> make_sinc_poly() {
  constexpr int NP = SPD + 1;
  SincPoly<WT> P{};
  for (int jj = 0; jj < WT; ++jj) {
    const int j = jj + 1 - WT / 2;
    double x[NP] = {}, y[NP] = {};
    for (int k = 0; k < NP; ++k) {
      x[k] = 0.5 * cx_cos((2.0 * k + 1.0) * kPi / (2.0 * NP));
      y[k] = s_tap(j, x[k], WT);
    }
    // Newton divided differences, then expansion to monomials
    double d[NP] = {};
    for (int k = 0; k < NP; ++k) d[k] = y[k];
    for (int lvl = 1; lvl < NP; ++lvl)
      for (int k = NP - 1; k >= lvl; --k) d[k] = (d[k] - d[k - 1]) / (x[k] - x[k - lvl]);
    double m[NP] = {};  // coefficients of the running polynomial, highest first
    m[0] = d[NP - 1];
    int deg = 0;
    for (int k = NP - 2; k >= 0; --k) {  // m(t) = m(t) * (t - x[k]) + d[k]
      double nm[NP] = {};
      for (int q = 0; q <= deg; ++q) {
        nm[q] += m[q];
        nm[q + 1] -= m[q] * x[k];
      }
      ++deg;
      nm[deg] += d[k];
      for (int q = 0; q < NP; ++q) m[q] = nm[q];
    }
    for (int q = 0; q < NP; ++q) P.c[SPD - q][jj] = (float)m[q];
  }
  return P;
}

// Monomial coefficients of the degree-SPD interpolant at the Chebyshev nodes
// of [-1/2, 1/2]: c = V^-1 y for the node values y, V the Vandermonde matrix
// of the nodes (inverted in double by the compiler, Gauss-Jordan with partial
// pivoting). Used for general-mode FP16 windows, whose interpolants are
// computed per call.
struct ChebFit {
  float node[SPD + 1];
  float vinv[SPD + 1][SPD + 1];  // vinv[k][i]: coefficient of t^k per unit value at node i
  float sin_pi_f[SPD + 1];       // sin(pi f_i) / pi at f_i = node_i + 1/2
};
constexpr ChebFit make_cheb_fit() {
  constexpr int NP = SPD + 1;
  ChebFit F{};
  double x[NP] = {}, a[NP][2 * NP] = {};
  for (int i = 0; i < NP; ++i) x[i] = 0.5 * cx_cos((2.0 * i + 1.0) * kPi / (2.0 * NP));
  for (int i = 0; i < NP; ++i) {  // [V | I], V[i][k] = x_i^k
    double pw = 1.0;
    for (int k = 0; k < NP; ++k) {
      a[i][k] = pw;
      pw *= x[i];
    }
    a[i][NP + i] = 1.0;
  }
  for (int c = 0; c < NP; ++c) {
    int piv = c;
    for (int r = c + 1; r < NP; ++r)
      if ((a[r][c] < 0 ? -a[r][c] : a[r][c]) > (a[piv][c] < 0 ? -a[piv][c] : a[piv][c])) piv = r;
    for (int k = 0; k < 2 * NP; ++k) {
      const double t = a[c][k];
      a[c][k] = a[piv][k];
      a[piv][k] = t;
    }
    const double d = a[c][c];
    for (int k = 0; k < 2 * NP; ++k) a[c][k] /= d;
    for (int r = 0; r < NP; ++r)
      if (r != c) {
        const double m = a[r][c];
        for (int k = 0; k < 2 * NP; ++k) a[r][k] -= m * a[c][k];
      }
  }
  // V^-1 maps node values to coefficients: c_k = sum_i (V^-1)[k][i] y_i
  for (int k = 0; k < NP; ++k)
    for (int i = 0; i < NP; ++i) F.vinv[k][i] = (float)a[k][NP + i];
  for (int i = 0; i < NP; ++i) {
    F.node[i] = (float)x[i];
    F.sin_pi_f[i] = (float)(cx_sin(kPi * (x[i] + 0.5)) / kPi);  // pi (x + 1/2) in (0, pi)
  }
  return F;
}
__constant__ ChebFit kChebFit = make_cheb_fit();

// FP32 taps by moments. As for FP16, tap j of an image is A s_j(t), t = f - 1/2,
// and s_j is replaced by its interpolant of degree MOM - 1 at the Chebyshev
// nodes, c_j0 + c_j1 t + ... (error < 3e-9 for every tap, so it is exact to FP32
// rounding: a windowed sinc is band-limited, and its Chebyshev coefficients
// over one sample fall faster than (pi/4)^p / p!). The images of one integer
// delay k0 then enter the RIR through the MOM sums M_p[k0] = sum A t^p alone,
//   h[k] = sum_j sum_p c_jp M_p[k - j],
// which costs an image MOM sums instead of W taps, and a convolution of MOM
// W per output sample whatever the number of images.
// The window is even, so s_{1-j}(t) = s_j(-t) and c_{1-j,p} = (-1)^p c_jp.
constexpr int MOM = 10;
template <int NP>
struct ChebFitD {
  double node[NP];
  double vinv[NP][NP];  // vinv[k][i]: coefficient of t^k per unit value at node i
};
template <int NP>
constexpr ChebFitD<NP> make_cheb_fit_d() {
  ChebFitD<NP> F{};
  for (int i = 0; i < NP; ++i) F.node[i] = 0.5 * cx_cos((2.0 * i + 1.0) * kPi / (2.0 * NP));
  // column i of the inverse Vandermonde matrix: the Lagrange polynomial of node i
  for (int i = 0; i < NP; ++i) {
    double m[NP] = {};  // coefficients of the running product, lowest first
    m[0] = 1.0;
    int deg = 0;
    double den = 1.0;
    for (int k = 0; k < NP; ++k) {
      if (k == i) continue;
      for (int q = ++deg; q > 0; --q) m[q] = m[q - 1] - F.node[k] * m[q];
      m[0] *= -F.node[k];
      den *= F.node[i] - F.node[k];
    }
    for (int k = 0; k < NP; ++k) F.vinv[k][i] = m[k] / den;
  }
  return F;
}
__constant__ ChebFitD<MOM> kMomFit = make_cheb_fit_d<MOM>();
// c[p][e]: coefficient of tap j = WT/2 + 15 - e, zero outside the window (the
// order and padding in which the convolution reads them).
template <int WT>
struct MomCoef {
  float c[MOM][WT + 32];
};
template <int WT>
constexpr MomCoef<WT> make_mom_coef() {
  constexpr ChebFitD<MOM> F = make_cheb_fit_d<MOM>();
  MomCoef<WT> t{};
  for (int j = 1; j <= WT / 2; ++j) {
    double y[MOM] = {};
    for (int i = 0; i < MOM; ++i) y[i] = s_tap(j, F.node[i], WT);
    for (int p = 0; p < MOM; ++p) {
      double v = 0.0;
      for (int i = 0; i < MOM; ++i) v += F.vinv[p][i] * y[i];
      t.c[p][WT / 2 + 15 - j] = (float)v;
      t.c[p][WT / 2 + 15 - (1 - j)] = (float)(p % 2 ? -v : v);
    }
  }
  return t;
}

// General-mode windows. W is any real number; with h = W/2, the taps j = 1 ..
// floor(h) (and their mirrors 1 - j) lie inside the window for every f, while tap
// j2 = floor(h) + 1 (mirror 1 - j2) is inside only for f > f1 = j2 - h (mirror:
// f < 1 - f1) and meets the window's end with a jump in its second derivative of
// about 20 / W^3, which a polynomial over the whole sample cannot follow. Under
// caps up to kEdgeCap its values are therefore summed image by image, A e(u) with
// u the distance inside the end and e the polynomial
//   e(u) = u^2 (e_0 + e_1 (u - 1/2) + ... + e_9 (u - 1/2)^9)
// of the windowed sinc there (off by at most 1.9e-9, just below W = 6; with two
// coefficients fewer 2.5e-7 there and 9.5e-8 just below W = 8); above, the
// jump moves the fit by at most 3.3e-8 (just below W = 65) and the tap takes the
// moments too. The moments of the other taps are off by at most 7.6e-8 at W = 4,
// 2.0e-8 from W = 6 and 8.4e-9 from W = 8, where the Hann window still bends
// within a sample. Windows shorter than kDirectWin vary too fast for the moments:
// their at most four taps are evaluated and summed image by image.
constexpr int kEdgeCap = 64;
constexpr int kEdgeCoef = 10;
constexpr float kDirectWin = 4.0f;
__constant__ ChebFitD<kEdgeCoef> kEdgeFit = make_cheb_fit_d<kEdgeCoef>();
// Layout of the FP32 constants of a general window of cap WT: c_jp at [p][j - 1]
// for j = 1 .. WT/2, then e_0 .. e_9, f1, j2 (0: no tap is cut).
constexpr int wc_edge(int WT) { return MOM * (WT / 2); }
static_assert(wc_edge(32) + kEdgeCoef + 2 <= 32 * WC_STRIDE, "window constants");

// Taylor coefficients (-1)^k / (2k)! and (-1)^k / (2k + 1)!, k <= 9.
struct TrigSeries {
  double c[10], s[10];
};
constexpr TrigSeries make_trig_series() {
  TrigSeries t{};
  double f = 1.0;
  for (int k = 0; k < 10; ++k) {
    const double sg = k % 2 ? -1.0 : 1.0;
    if (k > 0) f *= 2.0 * k;
    t.c[k] = sg / f;
    f *= 2.0 * k + 1.0;
    t.s[k] = sg / f;
  }
  return t;
}
// sin(pi x) and cos(pi x) in double for moderate |x| (reduction to |r| <= 1/4,
// Taylor series with terms below 1e-18 left out).
__device__ __forceinline__ void sincospi_d(double x, double &s, double &c) {
  constexpr TrigSeries T = make_trig_series();
  const double n = __builtin_rint(2.0 * x);
  const double y = (x - 0.5 * n) * kPi, y2 = y * y;
  double a = T.s[9], b = T.c[9];
#pragma unroll
  for (int k = 8; k >= 0; --k) {
    a = __builtin_fma(a, y2, T.s[k]);
    b = __builtin_fma(b, y2, T.c[k]);
  }
  a *= y;
  const int q = ((int)n) & 3;
  s = q == 0 ? a : q == 1 ? b : q == 2 ? -a : -b;
  c = q == 0 ? b : q == 1 ? -a : q == 2 ? -b : a;
}
// The windowed sinc of Eq. (6) at v != 0, without its cut at |v| = W/2.
__device__ double windowed_sinc_d(double v, double W) {
  double sn, cs, wn, wc;
  sincospi_d(v, sn, cs);
  sincospi_d(2.0 * v / W, wn, wc);
  return sn / (kPi * v) * 0.5 * (1.0 + wc);
}
// FP32 constants of a general window, by one block: the node values of every
// tap j >= 1 (and of the edge polynomial), then each coefficient.
__device__ void moment_consts(double W, int WT, float *__restrict__ wc) {
  static_assert(kEdgeCoef <= MOM, "one row of node values holds either fit");
  __shared__ double y[MAX_WINDOW / 2 + 1][MOM];
  const int half = WT / 2, nt = (int)blockDim.x;
  const int j2 = (int)__builtin_floor(0.5 * W) + 1;
  const bool edge = WT <= kEdgeCap && (double)j2 - 0.5 * W < 1.0 && j2 <= half;
  for (int e = threadIdx.x; e < (half + 1) * MOM; e += nt) {
    const int j = e / MOM + 1, i = e % MOM;
    double v = 0.0;
    if (j <= half) {
      const double x = (double)j - (kMomFit.node[i] + 0.5);
      if (!(edge && j == j2) && __builtin_fabs(x) < 0.5 * W) v = windowed_sinc_d(x, W);
    } else if (edge && i < kEdgeCoef) {
      const double u = kEdgeFit.node[i] + 0.5;
      v = windowed_sinc_d(0.5 * W - u, W) / (u * u);
    }
    y[j - 1][i] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < (half + 1) * MOM; e += nt) {
    const int p = e / (half + 1), jj = e % (half + 1);
    double v = 0.0;
    if (jj < half) {
      for (int i = 0; i < MOM; ++i) v += kMomFit.vinv[p][i] * y[jj][i];
      wc[p * half + jj] = (float)v;
    } else if (p < kEdgeCoef) {
      for (int i = 0; i < kEdgeCoef; ++i) v += kEdgeFit.vinv[p][i] * y[half][i];
      wc[wc_edge(WT) + p] = (float)v;
    }
  }
  if (threadIdx.x == 0) {
    wc[wc_edge(WT) + kEdgeCoef] = (float)((double)j2 - 0.5 * W);
    wc[wc_edge(WT) + kEdgeCoef + 1] = edge ? (float)j2 : 0.0f;
  }
}

// FP16 constants of tap jj (j = jj + 1 - WT/2) of a general-mode window of W
// samples under cap WT into e[0 .. WC_STRIDE): the interpolant of s_j(t) = tap
// value at f = t + 1/2 (Eq. (6), 0 where |j - f| >= W/2) at the Chebyshev nodes.
__device__ void window_const_entry(float W, int WT, int jj, float *e) {
  const int j = jj + 1 - WT / 2;
  const float sg = (j & 1) ? 1.0f : -1.0f;  // sin(pi (j - f)) = sg sin(pi f)
  for (int k = 0; k < WC_STRIDE; ++k) e[k] = 0.0f;
  float y[SPD + 1];
  for (int i = 0; i <= SPD; ++i) {
    const float f = kChebFit.node[i] + 0.5f;
    const float v = (float)j - f;
    float sn, cs;
    sincospi_acc(2.0f * v / W, sn, cs);
    y[i] = (__builtin_fabsf(v) < 0.5f * W) ? sg * kChebFit.sin_pi_f[i] / v * 0.5f * (1.0f + cs) : 0.0f;
  }
  for (int k = 0; k <= SPD; ++k) {
    float ck = 0.0f;
    for (int i = 0; i <= SPD; ++i) ck = __builtin_fmaf(kChebFit.vinv[k][i], y[i], ck);
    e[k] = ck;
  }
}

// Lookup-table taps (Eq. (9)): the windowed sinc of Eq. (6) tabulated at Q
// points per sample, L[n] = (1 + cos(2 pi n / (Q W))) / 2 sinc(n / Q) for
// n = -QW/2 .. QW/2, and each tap interpolated linearly between the two
// entries around its delay. For tap j of an image with fraction f = (fl + fr)/Q
// (fl an integer in [0, Q), fr in [0, 1)), v = j - f lies between entries
// Q j - fl - 1 and Q j - fl, with weight 1 - fr on the upper one: the image is a
// pulse of weight A (1 - fr) at phase fl of its sample and one of A fr at phase
// fl + 1, each filtered with the table. The pulses of all images of one integer
// delay are added up per phase (0 .. Q), and
//   h[k] = sum_j sum_phase L[Q j - phase] pulse[k - j][phase],
// the convolution of the moments with other coefficients.
constexpr int kLutQ = 16;
constexpr double lut_entry(int i, int wt) {  // L[i - QW/2]
  const int n = i - kLutQ * wt / 2;
  const double hann = 0.5 * (1.0 + cx_cos(2.0 * kPi * n / (kLutQ * wt)));  // angle in [-pi, pi]
  if (n == 0) return hann;
  // sin(pi n / Q) with n = Q m + r, 0 <= r < Q: (-1)^m sin(pi r / Q), keeping
  // the series argument in [0, pi)
  const int r = ((n % kLutQ) + kLutQ) % kLutQ;
  const int m = (n - r) / kLutQ;
  const double s = ((m & 1) ? -1.0 : 1.0) * cx_sin(kPi * r / kLutQ);
  const double v = (double)n / kLutQ;
  return hann * s / (kPi * v);
}
// c[phase][e]: L[Q j - phase] of tap j = WT/2 + 15 - e, zero outside the window.
template <int WT>
struct LutCoef {
  float c[kLutQ + 1][WT + 32];
};
template <int WT>
constexpr LutCoef<WT> make_lut_coef() {
  LutCoef<WT> t{};
  for (int j = 1 - WT / 2; j <= WT / 2; ++j)
    for (int ph = 0; ph <= kLutQ; ++ph) {
      const int i = kLutQ * j - ph + kLutQ * WT / 2;
      // the window's ends (1 + cos(pi) = 0) and what lies past them
      t.c[ph][WT / 2 + 15 - j] = i <= 0 || i >= kLutQ * WT ? 0.0f : (float)lut_entry(i, WT);
    }
  return t;
}

// ---------------------------------------------------------------------------
// Kernel 1: per-RIR axis tables.
// ---------------------------------------------------------------------------
// Table entry e (axis a, lattice index n) of the RIR with source s, receiver r.
__device__ __forceinline__ AxisEntry table_entry(const RoomArgs &ra, const float *__restrict__ s3,
                                                 const float *__restrict__ r3, int e,
                                                 const float *__restrict__ o3 = nullptr) {
  const int a = e < ra.off[1] ? 0 : (e < ra.off[2] ? 1 : 2);
  const int n = ra.lo[a] + (e - ra.off[a]);
  const float s = s3[ra.perm[a]], r = r3[ra.perm[a]];
  // Eq. (1): even n -> n L + s, odd n -> (n + 1) L - s.
  const bool odd = (n & 1) != 0;
  const double L = (double)ra.L_hi[a] + (double)ra.L_lo[a], q = (double)ra.q_hi + (double)ra.q_lo;
  // displacement in samples
  const double v = ((double)(odd ? n + 1 : n) * L + ((odd ? -(double)s : (double)s) - (double)r)) * q;
  // Gain factor: the path from image n crosses |floor(n/2)| copies of the wall
  // at 0 and |ceil(n/2)| copies of the wall at L along this axis.
  const int e0 = abs(n >> 1), e1 = abs((n + 1) >> 1);
  const double g = int_pow((double)ra.beta[2 * a] + (double)ra.beta_lo[2 * a], e0) *
                   int_pow((double)ra.beta[2 * a + 1] + (double)ra.beta_lo[2 * a + 1], e1);
  // receiver orientation (polar calls): the displacement's share of the
  // projection onto the unit orientation, whose three shares add up to
  // |d| cos(theta) in samples
  float proj = 0.0f;
  if (o3) {
    const float inv = __builtin_amdgcn_rsqf(o3[0] * o3[0] + o3[1] * o3[1] + o3[2] * o3[2]);
    proj = (float)v * (o3[ra.perm[a]] * inv);
  }
  // the enumeration only needs the square of the displacement
  return AxisEntry{v * v, (float)g, proj};
}

// Validity of a pair (both points strictly inside, distinct) and the family
// offsets of its axes.
__device__ __forceinline__ int rir_header(const RoomArgs &ra, const float *__restrict__ s3,
                                          const float *__restrict__ r3, AxisOrigin &o) {
  bool ok = true, same = true;
  for (int b = 0; b < 3; ++b) {
    const float sb = s3[ra.perm[b]], rb = r3[ra.perm[b]];
    ok = ok && sb > 0.0f && (sb - ra.L_hi[b]) < ra.L_lo[b] && rb > 0.0f && (rb - ra.L_hi[b]) < ra.L_lo[b];
    same = same && (sb == rb);
    o.e_even[b] = (sb - rb) * ra.q_hi;
    o.e_odd[b] = (-sb - rb) * ra.q_hi;
  }
  return (ok && !same) ? 1 : 0;
}

// Constants of a general-mode window, by one block.
__device__ __forceinline__ void window_consts(float W, int WT, int half, float *__restrict__ wc) {
  if (!half) moment_consts((double)W, WT, wc);
  else
    for (int jj = threadIdx.x; jj < WT; jj += blockDim.x) window_const_entry(W, WT, jj, wc + WC_STRIDE * jj);
}

// Blocks 0 .. n_blk - 1 write the tables; a general-mode call (wc set) adds one block
// that writes its window's constants.
__global__ __launch_bounds__(256) void tables_kernel(RoomArgs ra, const float *__restrict__ src,
                                                     const float *__restrict__ rcv,
                                                     const float *__restrict__ orient, AxisEntry *__restrict__ tab,
                                                     AxisOrigin *__restrict__ origin, int *__restrict__ valid,
                                                     int n_rir, int n_blk, float W, int half,
                                                     float *__restrict__ wc) {
  if ((int)blockIdx.x >= n_blk) {
    window_consts(W, (int)(2.0f * ra.half_w), half, wc);
    return;
  }
  const int64_t total = (int64_t)n_rir * ra.n_tab;
  for (int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; gid < total;
       gid += (int64_t)n_blk * blockDim.x) {
    const int rir = (int)(gid / ra.n_tab);
    const int e = (int)(gid % ra.n_tab);
    const float *s3 = src + 3 * (rir / ra.n_rcv);
    const float *r3 = rcv + 3 * (rir % ra.n_rcv);
    tab[gid] = table_entry(ra, s3, r3, e, orient ? orient + 3 * (rir % ra.n_rcv) : nullptr);
    if (e == 0) {
      AxisOrigin o;
      valid[rir] = rir_header(ra, s3, r3, o);
      origin[rir] = o;
    }
  }
}

// Batch mode: one block per batch-wide RIR, then (with general-mode windows) one
// per job, for its window's constants.
__global__ __launch_bounds__(256) void tables_batch_kernel(const JobDev *__restrict__ jobs,
                                                           const BatchRir *__restrict__ rirs,
                                                           AxisEntry *__restrict__ tab,
                                                           AxisOrigin *__restrict__ origin,
                                                           int *__restrict__ valid, uint32_t n_rir, int half) {
  if (blockIdx.x >= n_rir) {
    const JobDev &jb = jobs[blockIdx.x - n_rir];
    if (jb.wc) window_consts(2.0f * jb.ra.win_hw, (int)(2.0f * jb.ra.half_w), half, jb.wc);
    return;
  }
  const BatchRir br = rirs[blockIdx.x];
  const JobDev &jb = jobs[br.job];
  const RoomArgs &ra = jb.ra;
  const float *s3 = jb.src + 3 * (br.rir / ra.n_rcv);
  const float *r3 = jb.rcv + 3 * (br.rir % ra.n_rcv);
  AxisEntry *t = tab + jb.tab_base + (size_t)br.rir * ra.n_tab;
  const float *o3 = jb.orient ? jb.orient + 3 * (br.rir % ra.n_rcv) : nullptr;
  for (int e = threadIdx.x; e < ra.n_tab; e += blockDim.x) t[e] = table_entry(ra, s3, r3, e, o3);
  if (threadIdx.x == 0) {
    AxisOrigin o;
    valid[blockIdx.x] = rir_header(ra, s3, r3, o);
    origin[blockIdx.x] = o;
  }
}

// ---------------------------------------------------------------------------
// Wave-level helpers.
// ---------------------------------------------------------------------------
// Inclusive prefix sum over the 64 lanes with DPP lane shifts (no LDS):
// Hillis-Steele within each row of 16 lanes, then the row totals are carried
// into the later rows by the row broadcasts of lanes 15 and 31.
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return v;
}
// Inclusive running maximum over the 64 lanes of unsigned values, same lane
// pattern as wave_incl_scan.
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
  return v;
}
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Image displacements along one axis are strictly increasing in the lattice
// index n: even n = 2m at m P + e_even, odd n = 2m - 1 at m P + e_odd (P = 2 L q).
// The table index (n - lo) of the first n with displacement >= b is therefore
// the number of images below b, which first_ge counts family by family:
// family f holds M_f images m = m0_f .. m0_f + M_f - 1, of which
// clamp(ceil((b - e_f) / P) - m0_f, 0, M_f) lie below b. Float rounding can
// move the count by one only for images within ~1e-2 samples of b; callers
// widen their bounds by a sample so such images lie outside the band that
// matters. first_ge is monotone in b and a pure function of it, so equal
// bounds split a range exactly.
struct AxisRange {
  float inv_p;            // 1 / P
  float c_even, c_odd;    // -(e_f / P + m0_f)
  float n_even, n_odd;    // M_f
};
__device__ __forceinline__ AxisRange axis_range(int lo, int N, float inv_p, float e_even, float e_odd) {
  const int hi = lo + N;  // exclusive
  const int me0 = (lo + 1) >> 1, me1 = (hi - 1) >> 1;  // even n = 2m in [lo, hi)
  const int mo0 = (lo + 2) >> 1, mo1 = hi >> 1;        // odd n = 2m - 1 in [lo, hi)
  AxisRange a;
  a.inv_p = inv_p;
  a.c_even = -__builtin_fmaf(e_even, inv_p, (float)me0);
  a.c_odd = -__builtin_fmaf(e_odd, inv_p, (float)mo0);
  a.n_even = (float)max(me1 - me0 + 1, 0);
  a.n_odd = (float)max(mo1 - mo0 + 1, 0);
  return a;
}
__device__ __forceinline__ float first_ge_f(const AxisRange &a, float b) {
  const float ce = __builtin_amdgcn_fmed3f(ceilf(__builtin_fmaf(b, a.inv_p, a.c_even)), 0.0f, a.n_even);
  const float co = __builtin_amdgcn_fmed3f(ceilf(__builtin_fmaf(b, a.inv_p, a.c_odd)), 0.0f, a.n_odd);
  return ce + co;
}
__device__ __forceinline__ int first_ge(const AxisRange &a, float b) { return (int)first_ge_f(a, b); }

// Entry i of a table (uniform base, 32-bit offset).
__device__ __forceinline__ AxisEntry entry_at(const AxisEntry *__restrict__ t, int i) {
  return *reinterpret_cast<const AxisEntry *>(reinterpret_cast<const char *>(t) + (uint32_t)(i << 4));
}

// ---------------------------------------------------------------------------
// Kernel 2: enumeration of the image shell of one tile + windowed-sinc taps.
//
// Work item = (RIR, output tile, slab of the image shell along x). The wave
// walks the columns (nx, ny) that cross the shell, numbers their z candidates
// and hands them to a consumer that turns candidates into image
// parameters (delay, amplitude; lanes = images) and adds their taps.
//
// FP32 and table-tap consumer (moment_item): images are collected per integer
// delay and enter through their moments (pulses). One-wave consumer (tap_item, lanes =
// taps; FP16, and the others in calls of few images per tile): the candidates' parameters
// are staged in LDS; each half-wave (FP32 windows above 96 samples: the wave) then
// takes one staged image per step and its lanes add its taps into the
// group's own FP32 tile. All addresses of one step are distinct and
// consecutive, so there are no bank conflicts and no lost updates; steps of a
// group reach LDS in program order.
//
// Items end with a fixed-order sum, so results are bitwise reproducible.
// ---------------------------------------------------------------------------
typedef int int4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));

// Per-wave LDS of the shell enumeration. The candidates of a batch of 64
// columns are numbered 0 .. total-1, column by column; column lane c holds
// positions [excl_c, excl_c + n1_c + n2_c), its first run of z indices
// (z1_c ..) then its second (z2_c ..). M16 (directional receivers on four waves): 16-bit
// marks (up to 64), so that four workgroups fit a compute unit beside the columns' projections (256 rooms with
// cardioid receivers in one batch 1.59 ms, three workgroups with 32-bit marks 1.82; 64
// rooms with a window of 244.5 samples, whose kernel held two, 0.76 and 0.92).
template <bool M16>
struct EnumLds {
  typedef typename std::conditional<M16, uint16_t, uint32_t>::type Mark;
  Mark mark[64];       // per chunk of 64 positions: column lane + 1 where a column starts
  int4v col_run[64];   // (excl + n1, z1 - excl, z2 - n1 - excl, gain bits): position p
                       // of the column has z index p + (p < excl + n1 ? z1 - excl : z2 - n1 - excl)
  double col_s[64];    // column part of the squared distance
  // per x lane of the row batch: (first column << 11) | first y table index
  // (column counts stay below 64 * 2048 = 2^17, table indices below 2^11)
  uint32_t nx_col[64];
};
static_assert(ISM_MAX_N_IMG <= 2048, "nx_col packs y table indices in 11 bits");

// Wave-uniform geometry of one work item.
struct ItemGeom {
  int T0;                        // first sample of the tile
  int K1;                        // owned integer delays: k0 in [T0, K1)
  float R0, R1;                  // shell radii in samples, widened by 2
  double r1, r0;                 // their squares (r0 = 0 where R0 < 0)
  int nx_a, nx_b;                // x table indices of the slab
};

__device__ __forceinline__ ItemGeom item_geom(const RoomArgs &ra, const AxisRange &ax, int TL, int tile_id, int C,
                                              int c) {
  ItemGeom g;
  g.T0 = tile_id * TL;
  g.K1 = min(g.T0 + TL, ra.k_end);
  // The owned images have delay x in [T0, K1); the enumeration bounds are
  // widened by two samples on each side and every candidate is then filtered
  // exactly on its integer delay.
  g.R1 = (float)g.K1 + 2.0f;
  g.R0 = (float)g.T0 - 2.0f;
  g.r1 = (double)g.R1 * (double)g.R1;
  g.r0 = g.R0 > 0.0f ? (double)g.R0 * (double)g.R0 : 0.0;
  // Slab of the shell along the x displacement owned by chunk c of C.
  float dlo = -INFINITY, dhi = INFINITY;
  if (c > 0) dlo = -g.R1 + (2.0f * g.R1) * ((float)c / (float)C);
  if (c < C - 1) dhi = -g.R1 + (2.0f * g.R1) * ((float)(c + 1) / (float)C);
  g.nx_a = max(first_ge(ax, dlo), first_ge(ax, -g.R1));
  g.nx_b = min(first_ge(ax, dhi), first_ge(ax, g.R1));
  return g;
}

// Walks the shell of the item, shared by the NW waves of a workgroup: the columns
// of each block of 64 x indices are cut into equal batches of at most 64, the
// same number for every wave (each wave has its own EnumLds and repeats the x
// step). next() goes to the wave's next
// batch with candidates: it fills es.col_run and es.col_s and sets total, the
// candidates in the batch, and on column lane c its first position excl and its
// count cnt; false when there is none left. The column gain in col_run is the
// product of the x and y gain factors times gscale.
// DUMP (enumeration check): col_xy receives each column's x and y table
// indices, (x << 16) | y.
template <bool POLAR, bool DUMP, int NW>
struct ShellWalk {
  const ItemGeom &g;
  const AxisEntry *__restrict__ tx;
  const AxisEntry *__restrict__ ty;
  const AxisRange &ay, &az;
  float gscale;
  typedef EnumLds<POLAR && (NW > 1)> Lds;
  Lds &es;
  float *__restrict__ col_p;
  uint32_t *__restrict__ col_xy;
  int wv;
  int nx_next, nx0 = 0, ncols = 0;     // x block and its columns
  int gc0 = 0, bs = 0;                 // first column of the wave's next batch, columns per batch
  int col0 = 0, ny_cnt = 0;                           // this x lane's first column and its columns
  int total = 0, excl = 0, cnt = 0;

  __device__ __forceinline__ ShellWalk(const ItemGeom &g_, const AxisEntry *tx_, const AxisEntry *ty_,
                                       const AxisRange &ay_, const AxisRange &az_, float gscale_, Lds &es_,
                                       float *col_p_, uint32_t *col_xy_, int wv_)
      : g(g_), tx(tx_), ty(ty_), ay(ay_), az(az_), gscale(gscale_), es(es_), col_p(col_p_), col_xy(col_xy_), wv(wv_),
        nx_next(g_.nx_a) {}

  __device__ __forceinline__ bool next() {
    const int lane = threadIdx.x & 63;
    for (;;) {
      while (gc0 >= ncols) {
        if (nx_next >= g.nx_b) return false;
        nx0 = nx_next;
        nx_next += 64;
        // lanes = x indices: y range of the columns that reach the outer sphere
        const int nxi = nx0 + lane;
        int ny_lo = 0;
        ny_cnt = 0;
        if (nxi < g.nx_b) {
          const float rh = (float)(g.r1 - entry_at(tx, nxi).sq);
          if (rh > 0.0f) {
            const float R = __builtin_amdgcn_sqrtf(rh) + 1.0f;
            ny_lo = first_ge(ay, -R);
            ny_cnt = first_ge(ay, R) - ny_lo;
          }
        }
        const int incl_y = wave_incl_scan(ny_cnt);
        ncols = __builtin_amdgcn_readlane(incl_y, 63);
        col0 = incl_y - ny_cnt;
        wave_sync();
        es.nx_col[lane] = ((uint32_t)col0 << 11) | (uint32_t)ny_lo;
        // (a block without columns gets batches of one, none of which exists)
        const int rounds = max((ncols + 64 * NW - 1) / (64 * NW), 1);
        bs = NW > 1 ? max((ncols + NW * rounds - 1) / (NW * rounds), 1) : 64;
        gc0 = wv * bs;
      }
      // lanes = columns (nx, ny): z ranges of the shell
      const int gcol = gc0 + lane;
      // x lane of the column: the last x lane with columns starting at or
      // before it (each marks its first column in the batch; a running
      // maximum carries the marks forward, as for the candidates, from the
      // x lane of the batch's first column)
      es.mark[lane] = 0;
      wave_sync();
      if (ny_cnt > 0 && (uint32_t)(col0 - gc0) < 64u) es.mark[col0 - gc0] = (typename Lds::Mark)(lane + 1);
      wave_sync();
      const uint64_t before = __ballot(ny_cnt > 0 && col0 <= gc0);
      const uint32_t xm = max(wave_incl_max(es.mark[lane]), 64u - (uint32_t)__builtin_clzll(before | 1u));
      // (columns past the last repeat it and take no candidates)
      const int i = (int)xm - 1;
      const uint32_t xc = es.nx_col[i];
      const int iy = (int)(xc & 0x7ffu) + (min(gcol, ncols - 1) - (int)(xc >> 11));
      const AxisEntry ex = entry_at(tx, nx0 + i), ey = entry_at(ty, iy);
      if constexpr (DUMP) col_xy[lane] = ((uint32_t)(nx0 + i) << 16) | (uint32_t)iy;
      const double S = ex.sq + ey.sq;
      es.col_s[lane] = S;
      if constexpr (POLAR) col_p[lane] = ex.proj + ey.proj;  // column part of |d| cos(theta)
      const float cg = (ex.gain * ey.gain) * gscale;
      const float rh = (float)(g.r1 - S), hh = (float)(g.r0 - S);
      const float zmax = __builtin_amdgcn_sqrtf(fmaxf(rh, 0.0f)) + 1.0f;
      const float zmin = fmaxf(__builtin_amdgcn_sqrtf(fmaxf(hh, 0.0f)) - 1.0f, 0.0f);
      // displacements in [-zmax, -zmin) and [zmin, zmax): two runs of the
      // table (contiguous when zmin = 0)
      const float f1 = first_ge_f(az, -zmax), f2 = first_ge_f(az, zmin);
      const bool some = gcol < ncols && lane < bs && rh > 0.0f;
      const float m1 = first_ge_f(az, -zmin) - f1;
      const int z1 = (int)f1, z2 = (int)f2;
      const int n1 = some ? (int)m1 : 0;
      cnt = some ? (int)(m1 + (first_ge_f(az, zmax) - f2)) : 0;
      gc0 += NW * bs;
      const int incl = wave_incl_scan(cnt);
      total = __builtin_amdgcn_readlane(incl, 63);
      excl = incl - cnt;
      es.col_run[lane] = int4v{excl + n1, z1 - excl, z2 - n1 - excl, __float_as_int(cg)};
      wave_sync();
      if (total > 0) return true;
    }
  }
};

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// Parameters of one image candidate (column part cs of the squared distance,
// column gain cgain = fs / (4 pi c) times the x and y gains, z table row ez). ok
// is false when the tile does not own the image. base = k0 - T0, fr the delay
// fraction in [0, 1] (1 by rounding), A the amplitude of Eq. (4) (times the receiver's
// polar pattern when directional).
struct ImageParams {
  bool ok;
  int base;
  float fr, A;
};
template <bool POLAR>
__device__ __forceinline__ ImageParams image_params(const RoomArgs &ra, const ItemGeom &g, const double cs,
                                                    const float cgain, const AxisEntry ez, const float cp) {
  ImageParams p;
  // x = sqrt(S) in samples (Eq. (2)-(3)): FP32 estimate, one Newton step in FP64
  const double S = cs + ez.sq;
  const float sf = (float)S;
  const float rx = __builtin_amdgcn_rsqf(sf);
  const double xh = (double)(sf * rx);
  const double x = __builtin_fma(__builtin_fma(-xh, xh, S), (double)(0.5f * rx), xh);
  const double k = __builtin_floor(x);
  p.fr = (float)(x - k);
  p.base = (int)k - g.T0;
  p.ok = sf < 1.0e18f && (uint32_t)p.base < (uint32_t)(g.K1 - g.T0);
  // Eq. (4) amplitude (times the constant factor carried by the column gain)
  p.A = (cgain * ez.gain) * rx;
  // receiver polar pattern a + b cos(theta), cos(theta) = (d . o) / |d|
  if constexpr (POLAR) p.A *= __builtin_fmaf(ra.dir_b, (cp + ez.proj) * rx, ra.dir_a);
  return p;
}

// Staged record of the FP16 taps: (t, A') with t = f - 1/2 in FP32 and A' the
// amplitude with the base in its 8 low mantissa bits (relative change < 2^-15).
__device__ __forceinline__ float2v stage_record(const ImageParams &p) {
  const uint32_t Ab = (__float_as_uint(p.A) & ~kBaseMask) | ((uint32_t)p.base & kBaseMask);
  return float2v{p.fr - 0.5f, __uint_as_float(Ab)};
}

// Walks the candidates of a wave's batches in chunks of 64 positions (lane i of
// chunk q has position q + i). The column of a position is the last one starting
// at or before it: each column marks its first position in the chunk, a running
// maximum over the lanes carries the marks forward, and the last lane's column
// carries into the next chunk (columns start in increasing order). The next
// chunk's column and z table row are found ahead of its use.
template <bool POLAR, bool DUMP, int NW>
struct ChunkWalk {
  ShellWalk<POLAR, DUMP, NW> &sw;
  const AxisEntry *__restrict__ tz;
  int q = 0, total = 0;
  uint32_t carry = 0;
  int cl = 0, nz = 0;  // of the chunk at q: column lane, z table index and row, column gain
  float cg = 0.0f;
  AxisEntry ez{};

  __device__ __forceinline__ ChunkWalk(ShellWalk<POLAR, DUMP, NW> &sw_, const AxisEntry *tz_) : sw(sw_), tz(tz_) {}
  __device__ __forceinline__ void locate(int q0) {
    const int lane = threadIdx.x & 63;
    typedef typename ShellWalk<POLAR, DUMP, NW>::Lds Lds;
    Lds &es = sw.es;
    es.mark[lane] = 0;
    wave_sync();
    const int r = sw.excl - q0;
    if (sw.cnt > 0 && (uint32_t)r < 64u) es.mark[r] = (typename Lds::Mark)(lane + 1);
    wave_sync();
    const uint32_t m = max(wave_incl_max(es.mark[lane]), carry);
    carry = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
    cl = (int)m - 1;
    const int4v cr = es.col_run[cl];
    // positions past the last repeat it
    const int pos = min(q0 + lane, total - 1);
    nz = pos + (pos < cr.x ? cr.y : cr.z);
    cg = __int_as_float(cr.w);
    ez = entry_at(tz, nz);
  }
  // Goes to the wave's next chunk; false when there is none left.
  __device__ __forceinline__ bool advance() {
    if (q >= total) {
      if (!sw.next()) return false;
      total = sw.total;
      q = 0;
      carry = 0;
      locate(0);
    }
    return true;
  }
  // chunk(live, cl, nz, cg, ez) on the current chunk, whose successor is located first.
  template <class Chunk>
  __device__ __forceinline__ void visit(Chunk &&chunk) {
    const int lane = threadIdx.x & 63;
    const int cl_c = cl, nz_c = nz;
    const float cg_c = cg;
    const AxisEntry ez_c = ez;
    const bool live = q + lane < total;
    q += 64;
    if (q < total) locate(q);
    chunk(live, cl_c, nz_c, cg_c, ez_c);
  }
};

// Per-tap constants, indexed by jj = j - (1 - W/2).
__constant__ SincPoly<32> kPoly32 = make_sinc_poly<32>();
__constant__ SincPoly<64> kPoly64 = make_sinc_poly<64>();
__constant__ SincPoly<96> kPoly96 = make_sinc_poly<96>();
__constant__ SincPoly<128> kPoly128 = make_sinc_poly<128>();
template <int WT> __device__ __forceinline__ const SincPoly<WT> &poly_table();
template <> __device__ __forceinline__ const SincPoly<32> &poly_table<32>() { return kPoly32; }
template <> __device__ __forceinline__ const SincPoly<64> &poly_table<64>() { return kPoly64; }
template <> __device__ __forceinline__ const SincPoly<96> &poly_table<96>() { return kPoly96; }
template <> __device__ __forceinline__ const SincPoly<128> &poly_table<128>() { return kPoly128; }
// Compile-time checks of the tables: entries within [-0.25, 1], 1 at v = 0,
// and 0 (to FP32 rounding) at the other integers, where the sinc vanishes.
template <int WT>
constexpr bool lut_sane(const LutCoef<WT> &t) {
  for (int ph = 0; ph <= kLutQ; ++ph)
    for (int j = 1 - WT / 2; j <= WT / 2; ++j) {
      const double e = t.c[ph][WT / 2 + 15 - j];
      if (!(e >= -0.25 && e <= 1.0)) return false;
      const int n = kLutQ * j - ph;
      if (n == 0 && e != 1.0) return false;
      if (n != 0 && n % kLutQ == 0 && (e > 1e-7 || e < -1e-7)) return false;
    }
  return true;
}
static_assert(lut_sane(make_lut_coef<32>()) && lut_sane(make_lut_coef<64>()), "table of Eq. (9)");
static_assert(lut_sane(make_lut_coef<96>()) && lut_sane(make_lut_coef<128>()), "table of Eq. (9)");
__constant__ LutCoef<32> kLut32 = make_lut_coef<32>();
__constant__ LutCoef<64> kLut64 = make_lut_coef<64>();
__constant__ LutCoef<96> kLut96 = make_lut_coef<96>();
__constant__ LutCoef<128> kLut128 = make_lut_coef<128>();
__constant__ MomCoef<32> kMom32 = make_mom_coef<32>();
__constant__ MomCoef<64> kMom64 = make_mom_coef<64>();
__constant__ MomCoef<96> kMom96 = make_mom_coef<96>();
__constant__ MomCoef<128> kMom128 = make_mom_coef<128>();
template <int WT> __device__ __forceinline__ const MomCoef<WT> &mom_table();
template <> __device__ __forceinline__ const MomCoef<32> &mom_table<32>() { return kMom32; }
template <> __device__ __forceinline__ const MomCoef<64> &mom_table<64>() { return kMom64; }
template <> __device__ __forceinline__ const MomCoef<96> &mom_table<96>() { return kMom96; }
template <> __device__ __forceinline__ const MomCoef<128> &mom_table<128>() { return kMom128; }
template <int WT> __device__ __forceinline__ const LutCoef<WT> &lut_table();
template <> __device__ __forceinline__ const LutCoef<32> &lut_table<32>() { return kLut32; }
template <> __device__ __forceinline__ const LutCoef<64> &lut_table<64>() { return kLut64; }
template <> __device__ __forceinline__ const LutCoef<96> &lut_table<96>() { return kLut96; }
template <> __device__ __forceinline__ const LutCoef<128> &lut_table<128>() { return kLut128; }


// Output of a work item whose taps are in LDS tiles t0 (+ t1): the tile's own
// samples go to dst, the W/2 - 1 samples before and the W/2 after to marg
// (layout: left margin, then right margin; W - 1 values).
template <int WT, int NT>
__device__ __forceinline__ void write_item(float (*tile)[TILE + WT - 1], int n_own, float *__restrict__ dst,
                                           float *__restrict__ marg, int tid, int nthreads) {
  constexpr int LM = WT / 2 - 1;
  for (int k = tid; k < n_own; k += nthreads) {
    float v = tile[0][LM + k];
#pragma unroll
    for (int w = 1; w < NT; ++w) v += tile[w][LM + k];
    dst[k] = v;
  }
  for (int i = tid; i < WT - 1; i += nthreads) {
    const int ti = i < LM ? i : TILE + i;
    float v = tile[0][ti];
#pragma unroll
    for (int w = 1; w < NT; ++w) v += tile[w][ti];
    marg[i] = v;
  }
}
template <int WT>
__device__ __forceinline__ void write_invalid(int n_own, float *__restrict__ dst, float *__restrict__ marg, int tid,
                                              int nthreads) {
  for (int k = tid; k < n_own; k += nthreads) dst[k] = __builtin_nanf("");
  for (int i = tid; i < WT - 1; i += nthreads) marg[i] = __builtin_nanf("");
}

// The taps of a general window that its end cuts: e(u) at the left and the right end of
// the window of an image (t = f - 1/2).
template <bool EDGE>
struct EdgeTaps {
  float ec[EDGE ? kEdgeCoef : 1], f1;
  __device__ __forceinline__ void load(const float *__restrict__ e) {
#pragma unroll
    for (int i = 0; i < kEdgeCoef; ++i) ec[i] = e[i];
    f1 = e[kEdgeCoef];
  }
  __device__ __forceinline__ void taps(float t, float &el, float &er) const {
    // left end: inside for f < 1 - f1; right end: inside for f > f1
    const float ul = fmaxf((0.5f - f1) - t, 0.0f), ur = fmaxf(t + (0.5f - f1), 0.0f);
    const float xl = ul - 0.5f, xr = ur - 0.5f;
    float pl = ec[kEdgeCoef - 1], pr = ec[kEdgeCoef - 1];
#pragma unroll
    for (int i = kEdgeCoef - 2; i >= 0; --i) {
      pl = __builtin_fmaf(pl, xl, ec[i]);
      pr = __builtin_fmaf(pr, xr, ec[i]);
    }
    el = ul * (ul * pl);
    er = ur * (ur * pr);
  }
};
// A times the taps j = -1 .. 2 of a window shorter than kDirectWin, at v = j - f (|v| < 2).
__device__ __forceinline__ void direct_taps(const RoomArgs &ra, float t, float A, float (&w)[4]) {
  const float f = fminf(fmaxf(t + 0.5f, 0x1p-24f), 0x1.fffffep-1f);
  const float C2 = A * __builtin_amdgcn_sinf(0.5f * fminf(f, 1.0f - f)) * (float)(0.5 / kPi);
#pragma unroll
  for (int j = -1; j <= 2; ++j) {
    const float v = (float)j - f;
    const float x = __builtin_fabsf(v) < ra.win_hw
                        ? __builtin_fmaf(C2, __builtin_amdgcn_cosf(v * ra.inv_win), C2) * __builtin_amdgcn_rcpf(v)
                        : 0.0f;
    w[j + 1] = (j & 1) ? x : -x;
  }
}

// ---------------------------------------------------------------------------
// Taps of the one-wave items (lanes = taps): groups of LPG lanes, NQ = 64 / LPG images per
// step. init() loads the lane's constants (l: lane within its group), record() forms the
// staged record of an image (lanes = images), and step() adds the taps of the record's image
// to the group's LDS tile (sample k0 + j at base + j - 1 + W/2).
// ---------------------------------------------------------------------------
// FP16 taps: lane l adds the taps j = 1 - W/2 + l + LPG m (m < TPL).
template <int WT, bool GEN>
struct HalfTaps {
  static constexpr int LPG = 32, NQ = 64 / LPG;
  static constexpr int TPL = WT / LPG;          // taps per lane per step
  static constexpr int NPAIR = (TPL + 1) / 2;   // packed FP16 tap pairs per lane
  static_assert(WT % LPG == 0, "window must be a multiple of the lanes per image");
  typedef float2v Rec;
  float pc0[TPL];          // c0 of each tap
  half2_t pq[NPAIR][SPD];  // and c1..c5 of tap pairs (2p, 2p + 1)
  // GEN: general-mode window (WT is the cap, W = 2 ra.win_hw): the constants come from wc
  // ([WT][WC_STRIDE], written for this window by tables_kernel)
  __device__ __forceinline__ void init(const RoomArgs &, const float *__restrict__ wc, int l) {
    auto coef = [&](int k, int jj) {
      if constexpr (GEN) return wc[WC_STRIDE * jj + k];
      else return poly_table<WT>().c[k][jj];
    };
#pragma unroll
    for (int m = 0; m < TPL; ++m) pc0[m] = coef(0, l + LPG * m);
#pragma unroll
    for (int pr = 0; pr < NPAIR; ++pr)
#pragma unroll
      for (int k = 0; k < SPD; ++k) {
        const int m0 = 2 * pr, m1 = 2 * pr + 1;
        const float a = coef(k + 1, l + LPG * m0);
        const float b = m1 < TPL ? coef(k + 1, l + LPG * m1) : 0.0f;
        pq[pr][k] = half2_t{(_Float16)a, (_Float16)b};
      }
  }
  __device__ __forceinline__ Rec record(const RoomArgs &, const ImageParams &p) const { return stage_record(p); }
  // The empty asm consumes the record as one value where the step starts,
  // which keeps its LDS read a single 8-byte read issued ahead.
  __device__ __forceinline__ void step(const Rec P, float *tile, int l) const {
    __asm__ volatile("" ::"v"(P));
    const int b = (int)(__float_as_uint(P.y) & kBaseMask);
    float *t = tile + l + b;
    // tap = A (c0 + t q(t)), q in packed FP16 two taps at a time, the
    // rest in FP32 (t q(t) + c0 as one mixed-precision FMA)
    const float tf = P.x, A = P.y;
    const half2_t tt = {(_Float16)tf, (_Float16)tf};
#pragma unroll
    for (int pr = 0; pr < NPAIR; ++pr) {
      half2_t q = pq[pr][SPD - 1];
#pragma unroll
      for (int k = SPD - 2; k >= 0; --k) q = __builtin_elementwise_fma(q, tt, pq[pr][k]);
      const int m0 = 2 * pr, m1 = 2 * pr + 1;
      t[LPG * m0] = __builtin_fmaf(A, __builtin_fmaf(tf, (float)q.x, pc0[m0]), t[LPG * m0]);
      if (m1 < TPL) t[LPG * m1] = __builtin_fmaf(A, __builtin_fmaf(tf, (float)q.y, pc0[m1]), t[LPG * m1]);
    }
  }
};

// FP32 taps: with the moments' polynomials s_j(t) = E(t^2) + t O(t^2) and s_{1-j}(t) =
// E - t O, so lane l adds the pairs of taps j and 1 - j, j = 1 + l + LPG m, for 13
// instructions a pair (W = 32: 32 lanes per image, one tap each, t negated for 1 - j).
// General windows: the taps that the window's end cuts, or all of a window shorter than
// kDirectWin, are formed with the record (lanes = images).
template <int WT, bool GEN>
struct PairTaps {
  static constexpr int LPG = WT <= 96 ? 32 : 64, NQ = 64 / LPG;
  static constexpr bool ONE = WT == 32;  // one tap per lane
  static constexpr int PPL = ONE ? 1 : (WT / 2 + LPG - 1) / LPG;  // pairs per lane
  static constexpr bool EDGE = GEN && WT <= kEdgeCap, DIRECT = GEN && WT == 32;
  struct Plain { float t, A; int base; };
  // x1, x0: A times the cut taps j2 and 1 - j2; windows shorter than kDirectWin: taps 1
  // and 0, t and A then hold taps 2 and -1
  struct Cut { float t, A; int base; float x1, x0; };
  typedef typename std::conditional<EDGE, Cut, Plain>::type Rec;
  float c[PPL][MOM];
  float sign;  // ONE: of t
  int at[2];   // offsets of the lane's first pair (ONE: its tap) from the base
  int cut;     // 1: this lane's pair is cut; 2: it is taps 2 and -1 of a short window
  const float *edge;
  __device__ __forceinline__ void init(const RoomArgs &ra, const float *__restrict__ wc, int l) {
    const bool direct = DIRECT && 2.0f * ra.win_hw < kDirectWin;
    const int first = ONE ? l & 15 : l;  // pair: j = 1 + first
    sign = ONE && l >= 16 ? -1.0f : 1.0f;
    at[0] = WT / 2 + first;
    at[1] = WT / 2 - 1 - first;
    if (ONE && l >= 16) at[0] = at[1];
#pragma unroll
    for (int m = 0; m < PPL; ++m) {
      const int q = min(first + LPG * m, WT / 2 - 1);
#pragma unroll
      for (int p = 0; p < MOM; ++p) {
        if constexpr (GEN) c[m][p] = direct ? 0.0f : wc[p * (WT / 2) + q];
        else c[m][p] = mom_table<WT>().c[p][(uint32_t)(WT / 2 + 14 - q)];
      }
    }
    cut = 0;
    if constexpr (EDGE) {
      edge = wc + wc_edge(WT);
      if (DIRECT && direct) cut = first < 2 ? first + 1 : 0;
      else if (first + 1 == (int)edge[kEdgeCoef + 1]) cut = 1;
    }
  }
  __device__ __forceinline__ Rec record(const RoomArgs &ra, const ImageParams &p) const {
    const float t = p.fr - 0.5f;
    if constexpr (EDGE) {
      if (DIRECT && 2.0f * ra.win_hw < kDirectWin) {
        float w[4];
        direct_taps(ra, t, p.A, w);
        return Rec{w[3], w[0], p.base, w[2], w[1]};
      }
      EdgeTaps<true> et;
      et.load(edge);
      float el, er;
      et.taps(t, el, er);
      return Rec{t, p.A, p.base, p.A * er, p.A * el};
    } else {
      return Rec{t, p.A, p.base};
    }
  }
  __device__ __forceinline__ void step(const Rec &P, float *tile, int l) const {
    const float t = P.t, A = P.A, u = t * t;
#pragma unroll
    for (int m = 0; m < PPL; ++m) {
      float e = c[m][8], d = c[m][9];
#pragma unroll
      for (int p = 6; p >= 0; p -= 2) {
        e = __builtin_fmaf(e, u, c[m][p]);
        d = __builtin_fmaf(d, u, c[m][p + 1]);
      }
      float x1 = 0.0f, x0 = 0.0f;
      if constexpr (EDGE) {
        x1 = cut == 1 ? P.x1 : cut == 2 ? t : 0.0f;
        x0 = cut == 1 ? P.x0 : cut == 2 ? A : 0.0f;
      }
      float *const o1 = tile + (P.base + at[0] + LPG * m);
      if constexpr (ONE) {
        const float v = __builtin_fmaf(A, __builtin_fmaf(sign * t, d, e), *o1);
        *o1 = EDGE ? v + (sign > 0.0f ? x1 : x0) : v;
      } else if (PPL * LPG == WT / 2 || l + LPG * m < WT / 2) {
        float *const o0 = tile + (P.base + at[1] - LPG * m);
        d *= t;
        const float v1 = __builtin_fmaf(A, e + d, *o1), v0 = __builtin_fmaf(A, e - d, *o0);
        *o1 = EDGE ? v1 + x1 : v1;
        *o0 = EDGE ? v0 + x0 : v0;
      }
    }
  }
};

// Table taps (Eq. (9)): the image's two pulses, A (1 - fr) at phase fl and A fr at
// fl + 1, times the table's points; lane l adds the taps of HalfTaps.
template <int WT>
struct TableTaps {
  static constexpr int LPG = 32, NQ = 64 / LPG, TPL = WT / LPG;
  typedef struct { f4v a; } Rec;  // pulses, base, phase
  int first;  // the lane's first tap in a row of the table
  __device__ __forceinline__ void init(const RoomArgs &, const float *__restrict__, int l) { first = WT + 14 - l; }
  __device__ __forceinline__ Rec record(const RoomArgs &, const ImageParams &p) const {
    const float x = p.fr * (float)kLutQ, fl = fminf(floorf(x), (float)(kLutQ - 1));
    const float hi = p.A * (x - fl);
    return Rec{f4v{p.A - hi, hi, __int_as_float(p.base), __int_as_float((int)fl)}};
  }
  __device__ __forceinline__ void step(const Rec &P, float *tile, int l) const {
    const float *const row = &lut_table<WT>().c[0][0] + (uint32_t)(__float_as_int(P.a.w) * (WT + 32) + first);
    float *const t = tile + l + __float_as_int(P.a.z);
    float c0[TPL], c1[TPL];
#pragma unroll
    for (int m = 0; m < TPL; ++m) {
      c0[m] = row[-LPG * m];
      c1[m] = row[WT + 32 - LPG * m];
    }
#pragma unroll
    for (int m = 0; m < TPL; ++m)
      t[LPG * m] = __builtin_fmaf(P.a.x, c0[m], __builtin_fmaf(P.a.y, c1[m], t[LPG * m]));
  }
};

// One work item on one wave: FP16 taps, and the other taps in calls of few images per tile
// (few_images in ism_host.cpp). Bound by the taps' VALU and LDS updates where there are
// images and by the item's chain of table reads where there are none; 24 items share a
// compute unit (FP16 28), so a call of many small items has six times as many in flight as
// with moments: 1024 RIRs of 4800 samples, direct path alone 36 us (moments 149), lattice of
// 15 per axis 122 (172); table taps 36 (312) and 126 (342). dst receives the own samples of the tile (or a
// partial tile when C > 1), marg the margins. Accumulation is FP32.
template <int WT, class Taps, bool POLAR>
__device__ __forceinline__ void tap_item(const RoomArgs &ra, const int tile_id, const int C, const int c,
                                         const AxisEntry *__restrict__ tab, const AxisOrigin &org, const bool valid,
                                         float *__restrict__ dst, float *__restrict__ marg,
                                         const float *__restrict__ wc) {
  constexpr int LSPAN = TILE + WT - 1;
  constexpr int NQ = Taps::NQ, LPG = Taps::LPG;  // images per step, lanes per image
  // staged images: up to 64 new + NQ - 1 carried, + the read-ahead of a step
  constexpr int SCAP = 64 + 3 * NQ;

  __shared__ float tile[NQ][LSPAN];
  typedef typename Taps::Rec Rec;
  __shared__ Rec stp[SCAP];  // staged records
  __shared__ EnumLds<false> es;
  __shared__ float col_p[POLAR ? 64 : 1];  // polar calls: column part of |d| cos(theta)

  const int lane = threadIdx.x & 63;
  const int h = lane / LPG, l = lane % LPG;  // image group, lane within it
  const int n_own = min(TILE, ra.n_samples - tile_id * TILE);  // may be <= 0 past nS
  if (!valid) {
    write_invalid<WT>(n_own, dst, marg, lane, 64);
    return;
  }
  const AxisEntry *__restrict__ tx = tab + ra.off[0];
  const AxisEntry *__restrict__ ty = tab + ra.off[1];
  const AxisEntry *__restrict__ tz = tab + ra.off[2];
  const AxisRange ax = axis_range(ra.lo[0], ra.N[0], ra.inv_period[0], org.e_even[0], org.e_odd[0]);
  const AxisRange ay = axis_range(ra.lo[1], ra.N[1], ra.inv_period[1], org.e_even[1], org.e_odd[1]);
  const AxisRange az = axis_range(ra.lo[2], ra.N[2], ra.inv_period[2], org.e_even[2], org.e_odd[2]);
  const ItemGeom g = item_geom(ra, ax, TILE, tile_id, C, c);

  Taps taps;
  taps.init(ra, wc, l);
  for (int i = lane; i < NQ * LSPAN; i += 64) (&tile[0][0])[i] = 0.0f;
  float *const th = tile[h];
  auto step = [&](const Rec &P) { taps.step(P, th, l); };
  // staged record k
  auto rec = [&](int k) { return stp[k]; };

  int ns = 0;  // staged images (wave-uniform)
  ShellWalk<POLAR, false, 1> sw(g, tx, ty, ay, az, ra.kappa, es, col_p, nullptr, 0);
  ChunkWalk<POLAR, false, 1> cw(sw, tz);
  while (cw.advance()) {
    cw.visit([&](bool live, int cl, int, float cg, const AxisEntry ez) {
      // lanes = candidates: parameters, then compaction into the stage
      ImageParams p;
      p = image_params<POLAR>(ra, g, es.col_s[cl], cg, ez, POLAR ? col_p[cl] : 0.0f);
      p.ok = p.ok && live;
      const uint64_t okm = __ballot(p.ok);
      const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(okm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)okm, 0u));
      if (p.ok) stp[ns + rank] = taps.record(ra, p);
      ns += __builtin_popcountll(okm);
      wave_sync();
      // lanes = taps: NQ staged images per step, one per lane group; the next
      // step's record is read ahead of this step's tile update (reads ahead
      // stay inside the stage: indices < NQ (np + 1) + h <= SCAP)
      const int np = ns / NQ;
      Rec PA = rec(h);
      for (int s = 0; s < np; s += 2) {
        const Rec PB = rec(NQ * (s + 1) + h);
        __builtin_amdgcn_sched_barrier(0);  // keep the read-ahead in front of the step
        step(PA);
        if (s + 1 < np) {
          PA = rec(NQ * (s + 2) + h);
          __builtin_amdgcn_sched_barrier(0);
          step(PB);
        }
      }
      // carry the remaining images to the front of the stage (the ranges do
      // not overlap when np > 0)
      const int rem = ns - NQ * np;
      if (np > 0 && rem > 0) {
        if constexpr (std::is_class<Rec>::value) {  // (word by word: a struct would go through memory)
          typedef uint32_t __attribute__((may_alias)) Word;
          const Word *const from = reinterpret_cast<const Word *>(&stp[NQ * np + lane]);
          uint32_t w[sizeof(Rec) / 4] = {};
          if (lane < rem) {
#pragma unroll
            for (int i = 0; i < (int)(sizeof(Rec) / 4); ++i) w[i] = from[i];
          }
          wave_sync();
          if (lane < rem) {
#pragma unroll
            for (int i = 0; i < (int)(sizeof(Rec) / 4); ++i) reinterpret_cast<Word *>(&stp[lane])[i] = w[i];
          }
        } else {
          Rec P{};
          if (lane < rem) P = stp[NQ * np + lane];
          wave_sync();
          if (lane < rem) stp[lane] = P;
        }
      }
      ns = rem;
      wave_sync();
    });
  }
  if (h < ns) step(stp[h]);  // last images, fewer than NQ

  wave_sync();
  write_item<WT, NQ>(tile, n_own, dst, marg, lane, 64);
}

// ---------------------------------------------------------------------------
// One work item on a workgroup of four waves with FP32 taps, by moments (MOM
// above), or with table taps (LUT), by pulses per phase (kLutQ above).
//
// Collection (lanes = images): each wave enumerates its share of the columns; an
// image's record (t, A) goes to the next slot of the wave's part of an LDS pool
// and is linked into the wave's list of its integer delay with one exchange on
// the list's head, so images of one delay in one chunk need no ordering and
// nothing is lost. When the waves have filled their parts, each thread takes
// its delays of the tile: the four waves' lists of a delay are linked into one,
// and each lane walks its list and adds every record's moments into its registers
// (lanes = delays). A list holds its wave's images in program order, those that one
// exchange instruction links to the same head in the order in which LDS serves its
// lanes (undocumented, the same from call to call: repeated calls agree bit for bit),
// and the lists are joined in wave order, so a call always adds in the same order.
// Four waves share a pool because the walk takes as many steps as the longest of
// 64 lists: with Poisson lengths of mean 10 that is 1.9 steps per image and
// lane, with a wave's own pool (256 delays, mean 2.5) 2.9.
// Table taps add a record's two pulses to the lane's own column of an LDS array
// [phase][delay] instead, which no other lane touches.
// Convolution: at the end of the item the moments go to LDS planes and
// matrix instructions form the item's T + W - 1 output samples: output
// o = 16 a + r of row r, column a is the sum over planes and k' of
// coefficient[k' - r] and plane[16 a + k'], an FP32 16 x 16 x 4 product per
// four k', whose left operand is the same for all columns; wave w takes a
// quarter of the k'. Planes are kept at x + x / 16 so that the 16 columns read
// different banks.
// ---------------------------------------------------------------------------
constexpr int MOM_WAVES = 4;
// Pool slots per wave: 10 chunks of 64 positions. With these a workgroup takes 40 KB
// of LDS and four fit a compute unit: 1024-room batch 6.43 ms, 64 microphones at
// 48 kHz 2.37 ms, against 7.39 and 2.76 with 15 chunks (three workgroups) and 6.90
// and 2.48 with 7 (five), all before long tiles (now 5.97 and 2.18). Long tiles: 7 chunks beside their 12 KB of list ends.
// Table taps: 6 chunks, three workgroups with the 17 KB of pulses (32 receivers 201 us;
// 220 with 4 chunks, 253 with 10 and two workgroups; image by image in LDS tiles 703).
constexpr int mom_slots(int TL, bool lut) { return lut ? 384 : TL == TILE ? 640 : 448; }
// end of a list (slots are linked by byte offset in rec)
constexpr int mom_end(int TL, bool lut) { return 8 * MOM_WAVES * mom_slots(TL, lut); }
static_assert(mom_end(TILE, false) < 65536, "16-bit links");
static_assert(item_threads(ITEM_MOMENTS) == 64 * MOM_WAVES && item_threads(ITEM_FP16) == 64, "threads per item");
template <int TL, bool LUT>
struct MomPool {
  float2v rec[MOM_WAVES * mom_slots(TL, LUT) + 1];  // (t, A), table taps (f, A); the last slot ends every list: (0, 0)
  uint32_t head[MOM_WAVES][TL];
  uint16_t next[MOM_WAVES * mom_slots(TL, LUT) + 4];
  uint16_t tail[MOM_WAVES][TL];
  float pulse[LUT ? kLutQ + 1 : 1][LUT ? TL : 1];
};
template <int WT, int TL, bool EDGE, bool LUT, bool GEN>
struct MomShape {
  static constexpr int NB = TL / (64 * MOM_WAVES);                  // delays per thread
  static constexpr int P = LUT ? kLutQ + 1 : MOM + (EDGE ? 2 : 0);  // planes
  static constexpr int KS = (WT + 16) / 4;                // matrix steps per plane
  static constexpr int NBLK = (TL + WT - 1 + 15) / 16;    // output blocks of 16
  static constexpr int NCT = (NBLK + 15) / 16;            // column tiles of 16 blocks
  static constexpr int XN = 16 * NBLK + WT;               // plane entries
  static constexpr int PL = XN + XN / 16;                 // plane length with the bank skew
  static constexpr int CL = WT + 32;                      // coefficients per plane, zeros around
  // planes in LDS at a time
  static constexpr int CG = GEN ? CL : 0;
  static constexpr int PB = P * (PL + CG) * sizeof(float) <= sizeof(MomPool<TL, LUT>) ? P : (P + 1) / 2;
  static_assert(TL % (64 * MOM_WAVES) == 0 && XN % 16 == 0 && KS % MOM_WAVES == 0, "convolution shape");
};

template <int WT, int TL, bool LUT, bool POLAR, bool GEN>
__device__ __forceinline__ void moment_item(const RoomArgs &ra, const int tile_id, const int C, const int c,
                                            const AxisEntry *__restrict__ tab, const AxisOrigin &org,
                                            const bool valid, float *__restrict__ dst, float *__restrict__ marg,
                                            const float *__restrict__ wc) {
  constexpr bool EDGE = GEN && WT <= kEdgeCap;
  constexpr bool DIRECT = GEN && WT == 32;  // may hold windows shorter than kDirectWin
  static_assert(!(GEN && LUT), "table taps are built for the exact windows");
  typedef MomShape<WT, TL, EDGE, LUT, GEN> Sh;
  constexpr int P = Sh::P, NT = 64 * MOM_WAVES, SLOTS = mom_slots(TL, LUT), NB = Sh::NB;
  constexpr int LM = WT / 2 - 1;
  constexpr uint32_t END = mom_end(TL, LUT);
  union alignas(16) Lds {
    MomPool<TL, LUT> pool;
    float conv[Sh::PB * (Sh::PL + Sh::CG)];
    float part[MOM_WAVES][256 * Sh::NCT];
  };
  __shared__ Lds u;
  __shared__ EnumLds<POLAR> es_all[MOM_WAVES];
  __shared__ float col_p_all[POLAR ? MOM_WAVES : 1][POLAR ? 64 : 1];  // column part of |d| cos(theta)
  __shared__ alignas(16) int more_all[MOM_WAVES];
  // the planner and the batch grid count on waves_per_simd workgroups per compute unit (16
  // bytes for the next item of a batch); the compiler allots registers by what the LDS allows
  static_assert(sizeof(Lds) + sizeof(es_all) + (POLAR ? sizeof(col_p_all) : 0) + sizeof(more_all) + 16 <=
                    160 * 1024 / waves_per_simd(ITEM_MOMENTS, LUT), "workgroups per compute unit");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_own = min(TL, ra.n_samples - tile_id * TL);  // may be <= 0 past nS
  if (!valid) {
    write_invalid<WT>(n_own, dst, marg, tid, NT);
    return;
  }
  const AxisEntry *__restrict__ tx = tab + ra.off[0];
  const AxisEntry *__restrict__ ty = tab + ra.off[1];
  const AxisEntry *__restrict__ tz = tab + ra.off[2];
  const AxisRange ax = axis_range(ra.lo[0], ra.N[0], ra.inv_period[0], org.e_even[0], org.e_odd[0]);
  const AxisRange ay = axis_range(ra.lo[1], ra.N[1], ra.inv_period[1], org.e_even[1], org.e_odd[1]);
  const AxisRange az = axis_range(ra.lo[2], ra.N[2], ra.inv_period[2], org.e_even[2], org.e_odd[2]);
  const ItemGeom g = item_geom(ra, ax, TL, tile_id, C, c);

  // this thread's delays tid, tid + NT, ..: sums of A t^p (then the edge taps);
  // table taps: the pulses, at the end
  float m[NB][P];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      m[b][p] = 0.0f;
      if constexpr (LUT) u.pool.pulse[p][tid + NT * b] = 0.0f;
    }
#pragma unroll
    for (int v = 0; v < MOM_WAVES; ++v) u.pool.head[v][tid + NT * b] = END;
  }
  if (tid == 0) {
    u.pool.rec[END / 8] = float2v{0.0f, 0.0f};
    u.pool.next[END / 8] = (uint16_t)END;
  }
  const bool direct = DIRECT && 2.0f * ra.win_hw < kDirectWin;
  EdgeTaps<EDGE> et;
  if constexpr (EDGE) et.load(wc + wc_edge(WT));

  // one record into the sums of this thread's delay b
  auto add = [&](const int b, const float2v r, auto taps) {
    const float t = r.x, A = r.y;
    if constexpr (LUT) {
      const float x = t * (float)kLutQ, fl = fminf(floorf(x), (float)(kLutQ - 1));
      const float hi = A * (x - fl);
      float *const g = &u.pool.pulse[(int)fl][tid + NT * b];
      g[0] += A - hi;
      g[TL] += hi;
      return;
    }
    if constexpr (decltype(taps)::value) {
      // into sum j + 1
      float w[4];
      direct_taps(ra, t, A, w);
#pragma unroll
      for (int j = 0; j < 4; ++j) m[b][j] += w[j];
      return;
    }
    const float At = A * t, t2 = t * t, t4 = t2 * t2, t6 = t4 * t2, t8 = t4 * t4;
    m[b][0] += A;
    m[b][1] += At;
    m[b][2] = __builtin_fmaf(A, t2, m[b][2]);
    m[b][3] = __builtin_fmaf(At, t2, m[b][3]);
    m[b][4] = __builtin_fmaf(A, t4, m[b][4]);
    m[b][5] = __builtin_fmaf(At, t4, m[b][5]);
    m[b][6] = __builtin_fmaf(A, t6, m[b][6]);
    m[b][7] = __builtin_fmaf(At, t6, m[b][7]);
    m[b][8] = __builtin_fmaf(A, t8, m[b][8]);
    m[b][9] = __builtin_fmaf(At, t8, m[b][9]);
    if constexpr (EDGE) {
      float el, er;
      et.taps(t, el, er);
      m[b][MOM] = __builtin_fmaf(A, el, m[b][MOM]);
      m[b][MOM + 1] = __builtin_fmaf(A, er, m[b][MOM + 1]);
    }
  };
  char *const rec0 = reinterpret_cast<char *>(u.pool.rec), *const next0 = reinterpret_cast<char *>(u.pool.next);
  auto rec_at = [&](uint32_t o) { return *reinterpret_cast<const float2v *>(rec0 + o); };
  auto next_at = [&](uint32_t o) -> uint16_t & { return *reinterpret_cast<uint16_t *>(next0 + (o >> 2)); };
  // the list's end links to itself and its record adds zero: a lane whose list
  // is shorter than the longest goes on adding it
  auto walk = [&](uint32_t (&i0)[NB], auto taps) {
    if constexpr (NB == 1) {
      while (__any(i0[0] != END)) {
        const uint32_t i1 = next_at(i0[0]);
        const float2v r0 = rec_at(i0[0]);
        const float2v r1 = rec_at(i1);
        i0[0] = next_at(i1);
        add(0, r0, taps);
        add(0, r1, taps);
      }
    } else {
      // the lists of the thread's delays side by side, two at a time
#pragma unroll
      for (int b = 0; b < NB; b += 2)
        while (__any(i0[b] != END || i0[b + 1] != END)) {
          const float2v r0 = rec_at(i0[b]), r1 = rec_at(i0[b + 1]);
          i0[b] = next_at(i0[b]);
          i0[b + 1] = next_at(i0[b + 1]);
          add(b, r0, taps);
          add(b + 1, r1, taps);
        }
    }
  };

  ShellWalk<POLAR, false, MOM_WAVES> sw(g, tx, ty, ay, az, ra.kappa, es_all[wv], col_p_all[POLAR ? wv : 0], nullptr,
                                        wv);
  ChunkWalk<POLAR, false, MOM_WAVES> cw(sw, tz);
  const EnumLds<POLAR> &es = es_all[wv];
  const float *const col_p = col_p_all[POLAR ? wv : 0];
  __syncthreads();
  for (;;) {
    bool more = true;
    for (int slot = 0; slot < SLOTS; slot += 64) {
      more = cw.advance();
      if (!more) break;
      cw.visit([&](bool live, int cl, int, float cg, const AxisEntry ez) {
        const ImageParams p = image_params<POLAR>(ra, g, es.col_s[cl], cg, ez, POLAR ? col_p[cl] : 0.0f);
        if (live && p.ok) {
          const uint32_t i = (uint32_t)(8 * (wv * SLOTS + slot + lane));
          const uint32_t old = atomicExch(&u.pool.head[wv][p.base], i);
          u.pool.rec[i / 8] = float2v{LUT ? p.fr : p.fr - 0.5f, p.A};
          next_at(i) = (uint16_t)old;
          if (old == END) u.pool.tail[wv][p.base] = (uint16_t)i;
        }
      });
    }
    if (lane == 0) more_all[wv] = more ? 1 : 0;
    __syncthreads();
    const int4v more4 = *reinterpret_cast<const int4v *>(more_all);
    uint32_t i0[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int k = tid + NT * b;
      i0[b] = END;
#pragma unroll
      for (int v = MOM_WAVES - 1; v >= 0; --v) {
        const uint32_t hv = u.pool.head[v][k];
        u.pool.head[v][k] = END;
        if (hv != END) {
          next_at(u.pool.tail[v][k]) = (uint16_t)i0[b];
          i0[b] = hv;
        }
      }
    }
    if constexpr (DIRECT) {
      if (direct) walk(i0, std::true_type{});
      else walk(i0, std::false_type{});
    } else {
      walk(i0, std::false_type{});
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(more4.x | more4.y | more4.z | more4.w)) break;
  }

  if constexpr (LUT) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int p = 0; p < P; ++p) m[b][p] = u.pool.pulse[p][tid + NT * b];
    __syncthreads();
  }
  // convolution, planes of PB moments at a time (highest first)
  float *const planes = u.conv, *const coefs = u.conv + Sh::PB * Sh::PL;
  const int lc = lane & 15, lk = lane >> 4;  // matrix row (coefficients) / column (planes), k group
  int a[Sh::NCT];                            // this lane's output block of each column tile
#pragma unroll
  for (int t = 0; t < Sh::NCT; ++t) a[t] = min(lc + 16 * t, Sh::NBLK - 1);
  // sums of planes 0, 1 and of the others apart (then smallest first; table taps: of
  // every third phase): each rounds at its own, smaller size
  f4v d[3][Sh::NCT];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int t = 0; t < Sh::NCT; ++t) d[i][t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int KQ = Sh::KS / MOM_WAVES;  // steps of this wave: s0 .. s0 + KQ - 1
  const int s0 = wv * KQ;
#pragma unroll
  for (int pb = (P - 1) / Sh::PB * Sh::PB; pb >= 0; pb -= Sh::PB) {
    constexpr int PB = Sh::PB;
    if (pb + PB < P) __syncthreads();  // the planes above are used up
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int x = tid + NT * b + WT - 1;
#pragma unroll
      for (int q = 0; q < PB; ++q)
        if (pb + q < P) planes[q * Sh::PL + x + (x >> 4)] = m[b][pb + q < P ? pb + q : 0];
    }
    // zeros before and after the tile's delays
    constexpr int NZ = Sh::XN - TL;
    for (int e = tid; e < NZ; e += NT) {
      const int xz = e < WT - 1 ? e : e + TL;
#pragma unroll
      for (int q = 0; q < PB; ++q) planes[q * Sh::PL + xz + (xz >> 4)] = 0.0f;
    }
    if constexpr (GEN) {
      // coefficients in the order of MomCoef
      const int j2 = EDGE ? (int)wc[wc_edge(WT) + kEdgeCoef + 1] : 0;
      for (int e = tid; e < Sh::CL; e += NT) {
        const int j = WT / 2 + 15 - e;
        const bool in = j > -WT / 2 && j <= WT / 2;
        const int jj = in ? (j >= 1 ? j - 1 : -j) : 0;
#pragma unroll
        for (int q = 0; q < PB; ++q) {
          const int p = pb + q;
          float v = 0.0f;
          if (DIRECT && direct) {
            v = (p < 4 && j == p - 1) ? 1.0f : 0.0f;
          } else if (p >= MOM) {
            v = (j2 > 0 && j == (p == MOM ? 1 - j2 : j2)) ? 1.0f : 0.0f;
          } else {
            v = wc[p * (WT / 2) + jj];
            if (!in) v = 0.0f;
            if (j < 1 && (p & 1)) v = -v;
          }
          coefs[q * Sh::CL + e] = v;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = PB - 1; q >= 0; --q) {
      const int p = pb + q;
      if (p >= P) continue;
      const int i = LUT ? p % 3 : p < 2 ? p : 2;
      const float *const pl = planes + q * Sh::PL + lk;
#pragma unroll
      for (int k = 0; k < KQ; ++k) {
        const int s = s0 + k;
        float cv;
        if constexpr (GEN) cv = coefs[q * Sh::CL + 4 * s + (lk - lc + 15)];
        else if constexpr (LUT) cv = lut_table<WT>().c[p][(uint32_t)(4 * s + (lk - lc + 15))];
        else cv = mom_table<WT>().c[p][(uint32_t)(4 * s + (lk - lc + 15))];
#pragma unroll
        for (int t = 0; t < Sh::NCT; ++t)
          d[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(cv, pl[17 * a[t] + 4 * s + (s >> 2)], d[i][t], 0, 0, 0);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < Sh::NCT; ++t)
    *reinterpret_cast<f4v *>(&u.part[wv][256 * t + 16 * lc + 4 * lk]) = d[2][t] + (d[1][t] + d[0][t]);
  __syncthreads();
  // output o: sample o - LM of the tile; before and after it the margins
  for (int o = tid; o < TL + WT - 1; o += NT) {
    const float v = (u.part[0][o] + u.part[3][o]) + (u.part[1][o] + u.part[2][o]);
    if (o < LM) marg[o] = v;
    else if (o >= LM + TL) marg[o - TL] = v;
    else if (o - LM < n_own) dst[o - LM] = v;
  }
}

// The item function of a kernel's item kind.
template <int WT, int TL, int KIND, bool LUT, bool POLAR, bool GEN>
__device__ __forceinline__ void run_item(const RoomArgs &ra, const int tile_id, const int C, const int c,
                                         const AxisEntry *__restrict__ tab, const AxisOrigin &org, const bool valid,
                                         float *__restrict__ dst, float *__restrict__ marg,
                                         const float *__restrict__ wc) {
  if constexpr (KIND == ITEM_FP16)
    tap_item<WT, HalfTaps<WT, GEN>, POLAR>(ra, tile_id, C, c, tab, org, valid, dst, marg, wc);
  else if constexpr (KIND == ITEM_FEW && LUT)
    tap_item<WT, TableTaps<WT>, POLAR>(ra, tile_id, C, c, tab, org, valid, dst, marg, wc);
  else if constexpr (KIND == ITEM_FEW)
    tap_item<WT, PairTaps<WT, GEN>, POLAR>(ra, tile_id, C, c, tab, org, valid, dst, marg, wc);
  else
    moment_item<WT, TL, LUT, POLAR, GEN>(ra, tile_id, C, c, tab, org, valid, dst, marg, wc);
}

// The 16 dispatch positions of plan block blk on lanes 0 .. 15: chunks per RIR, and the
// items before the position within the block.
struct PlanLanes {
  int chunks;
  uint32_t before;
};
__device__ __forceinline__ PlanLanes plan_lanes(const PlanArgs &pa, int blk) {
  const int lane = (int)(threadIdx.x & 63), p = blk * PLAN_BLK + lane;
  PlanLanes l;
  l.chunks = lane < PLAN_BLK && p < pa.n_tiles ? (int)pa.chunks[pa.n_tiles - 1 - p] : 0;
  const int n = pa.n_rir * l.chunks;
  l.before = (uint32_t)(wave_incl_scan(n) - n);
  return l;
}
// First work item of dispatch position pos (see PlanArgs).
__device__ __forceinline__ uint32_t plan_first_item(const PlanArgs &pa, int pos) {
  const PlanLanes l = plan_lanes(pa, pos / PLAN_BLK);
  return pa.first_blk[pos / PLAN_BLK] + (uint32_t)__builtin_amdgcn_readlane((int)l.before, pos % PLAN_BLK);
}

// Work item of a single-room launch: the item index decodes through the
// per-tile chunk counts.
struct SingleItem {
  int pos, tile_id, C, rir, c;
  uint32_t first;  // first item of the dispatch position
};
__device__ __forceinline__ SingleItem decode_item(const PlanArgs &pa, uint32_t item) {
  // largest dispatch position pos whose first item is <= item: the block, then the
  // position within it, each by one load on all lanes (a search in scalar loads takes
  // up to 20 one after the other: a call of 4 receivers 67.2 -> 65.6 us)
  const int lane = (int)(threadIdx.x & 63);
  const int nblk = (pa.n_tiles + PLAN_BLK - 1) / PLAN_BLK;
  int blk = 0;
  uint32_t base = 0;
  for (int b0 = 0; b0 < nblk && nblk > 1; b0 += 64) {
    const uint32_t f = b0 + lane < nblk ? pa.first_blk[b0 + lane] : 0xffffffffu;
    const int n = __builtin_popcountll(__ballot(b0 + lane < nblk && f <= item));
    if (n == 0) break;
    blk = b0 + n - 1;
    base = (uint32_t)__builtin_amdgcn_readlane((int)f, n - 1);
    if (n < 64) break;
  }
  const PlanLanes l = plan_lanes(pa, blk);
  const int at = __builtin_popcountll(__ballot(lane < PLAN_BLK && blk * PLAN_BLK + lane < pa.n_tiles &&
                                               base + l.before <= item)) - 1;
  const uint32_t first = base + (uint32_t)__builtin_amdgcn_readlane((int)l.before, at);
  SingleItem si;
  si.pos = blk * PLAN_BLK + at;
  si.first = first;
  si.tile_id = pa.n_tiles - 1 - si.pos;
  si.C = __builtin_amdgcn_readlane(l.chunks, at);
  const uint32_t rel = item - first;
  si.rir = (int)(rel / (uint32_t)si.C);
  si.c = (int)(rel % (uint32_t)si.C);
  return si;
}

template <int WT, int TL, int KIND, bool LUT, bool POLAR, bool GEN>
__global__ __launch_bounds__(item_threads(KIND))
__attribute__((amdgpu_waves_per_eu(waves_per_simd(KIND, LUT)))) void
accumulate_kernel(RoomArgs ra, PlanArgs pa, const AxisEntry *__restrict__ tab_all,
                  const AxisOrigin *__restrict__ origin, const int *__restrict__ valid, float *__restrict__ out,
                  float *__restrict__ part, float *__restrict__ marg, const float *__restrict__ wc,
                  uint32_t first_item) {
  const uint32_t item = first_item + blockIdx.x;
  const SingleItem si = decode_item(pa, item);
  // (for a tile past nS, dst is never written: the tile has no own samples)
  float *dst = (si.C == 1) ? out + (size_t)si.rir * ra.n_samples + (size_t)si.tile_id * TL
                           : part + (size_t)item * TL;
  const AxisOrigin org = origin[si.rir];
  run_item<WT, TL, KIND, LUT, POLAR, GEN>(ra, si.tile_id, si.C, si.c, tab_all + (size_t)si.rir * ra.n_tab, org,
                                      valid[si.rir] != 0, dst, marg + (size_t)item * WT, wc);
}

// Enumeration check: the items of a single-room launch, images only, on the walk of the
// item kernels: shared by the four waves of a workgroup (FP32 and table taps) or on one
// wave (FP16). Every owned image is written to dump.rec.
template <int NW>
__global__ __launch_bounds__(64 * NW) void enumerate_dump_kernel(RoomArgs ra, PlanArgs pa,
                                                                 const AxisEntry *__restrict__ tab_all,
                                                                 const AxisOrigin *__restrict__ origin,
                                                                 const int *__restrict__ valid, DumpArgs dump,
                                                                 uint32_t first_item) {
  __shared__ EnumLds<false> es_all[NW];
  __shared__ uint32_t col_xy_all[NW][64];  // column table indices
  const SingleItem si = decode_item(pa, first_item + blockIdx.x);
  if (valid[si.rir] == 0) return;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const AxisEntry *__restrict__ tab = tab_all + (size_t)si.rir * ra.n_tab;
  const AxisOrigin org = origin[si.rir];
  const AxisRange ax = axis_range(ra.lo[0], ra.N[0], ra.inv_period[0], org.e_even[0], org.e_odd[0]);
  const AxisRange ay = axis_range(ra.lo[1], ra.N[1], ra.inv_period[1], org.e_even[1], org.e_odd[1]);
  const AxisRange az = axis_range(ra.lo[2], ra.N[2], ra.inv_period[2], org.e_even[2], org.e_odd[2]);
  const ItemGeom g = item_geom(ra, ax, ra.tile, si.tile_id, si.C, si.c);
  EnumLds<false> &es = es_all[wv];
  const uint32_t *const col_xy = col_xy_all[wv];
  ShellWalk<false, true, NW> sw(g, tab + ra.off[0], tab + ra.off[1], ay, az, ra.kappa, es, nullptr, col_xy_all[wv], wv);
  ChunkWalk<false, true, NW> cw(sw, tab + ra.off[2]);
  while (cw.advance()) {
    cw.visit([&](bool live, int cl, int nz, float cg, const AxisEntry ez) {
      const ImageParams p = image_params<false>(ra, g, es.col_s[cl], cg, ez, 0.0f);
      const bool ok = live && p.ok;
      const uint64_t okm = __ballot(ok);
      const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(okm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)okm, 0u));
      uint32_t first = 0;
      if (lane == 0 && okm != 0) first = atomicAdd(dump.count, (uint32_t)__builtin_popcountll(okm));
      first = (uint32_t)__builtin_amdgcn_readlane((int)first, 0);
      if (ok && first + (uint32_t)rank < dump.cap) {
        const uint32_t xy = col_xy[cl];
        // lattice index per table axis, then per room axis (table axis k is room axis perm[k])
        const int t0 = ra.lo[0] + (int)(xy >> 16), t1 = ra.lo[1] + (int)(xy & 0xffffu), t2 = ra.lo[2] + nz;
        DumpRec d;
        d.rir = si.rir;
        d.n[0] = ra.perm[0] == 0 ? t0 : (ra.perm[1] == 0 ? t1 : t2);
        d.n[1] = ra.perm[0] == 1 ? t0 : (ra.perm[1] == 1 ? t1 : t2);
        d.n[2] = ra.perm[0] == 2 ? t0 : (ra.perm[1] == 2 ? t1 : t2);
        d.k0 = g.T0 + p.base;
        d.fq = min((uint32_t)__builtin_rintf(p.fr * 0x1p24f), (1u << 24) - 1u);  // units of 2^-24
        d.A = p.A;
        d.pad = 0;
        dump.rec[first + (uint32_t)rank] = d;
      }
    });
  }
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Batch launch: persistent. The grid holds at most the resident workgroups; each
// takes item blockIdx.x first, then the next unclaimed
// item of the largest-first list from the class's queue counter (which the
// run sets to the grid size before the launch), until the list is exhausted.
// Without a queue (queue == null) a workgroup takes every gridDim.x-th item.
// Every item names its job; the job table carries the room.
template <int WT, int TL, int KIND, bool LUT, bool POLAR, bool GEN>
__global__ __launch_bounds__(item_threads(KIND))
__attribute__((amdgpu_waves_per_eu(waves_per_simd(KIND, LUT)))) void
accumulate_batch_kernel(
    const JobDev *__restrict__ jobs, const BatchItem *__restrict__ items, uint32_t n_items, uint32_t *queue,
    const AxisEntry *__restrict__ tab_all, const AxisOrigin *__restrict__ origin, const int *__restrict__ valid,
    float *__restrict__ part, float *__restrict__ marg) {
  constexpr bool MULTI = item_threads(KIND) > 64;
  const int lane = threadIdx.x & 63;
  __shared__ uint32_t next_item;
  uint32_t item = blockIdx.x;
  while (item < n_items) {
    // the next item's number arrives while this one is worked on
    uint32_t next = 0;
    if (MULTI && queue && threadIdx.x == 0) next = atomicAdd(queue, 1u);
    const BatchItem it = items[item];
    const JobDev &jb = jobs[it.job];
    const RoomArgs ra = jb.ra;
    const uint32_t grir = jb.rir_base + it.rir;
    float *dst = (it.slot == 0xffffffffu) ? jb.out + (size_t)it.rir * ra.n_samples + (size_t)it.tile * TL
                                          : part + (size_t)it.slot * TILE;
    const AxisOrigin org = origin[grir];
    run_item<WT, TL, KIND, LUT, POLAR, GEN>(ra, it.tile, it.chunks, it.chunk,
                                        tab_all + jb.tab_base + (size_t)it.rir * ra.n_tab, org, valid[grir] != 0, dst,
                                        marg + (size_t)it.mslot * MARG_UNIT, jb.wc);
    if (queue) {
      if constexpr (MULTI) {
        if (threadIdx.x == 0) next_item = next;
        __syncthreads();
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)next_item);
        __syncthreads();
      } else {
        if (lane == 0) next = atomicAdd(queue, 1u);
        item = (uint32_t)__builtin_amdgcn_readlane((int)next, 0);
      }
    } else {
      item += gridDim.x;
      if constexpr (MULTI) __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Kernel 3: ordered completion of the output tiles. Sample k of tile t is
//   (own sum) + (right margins of the items of tile t-1) + (left margins of
//   the items of tile t+1),
// where the own sum is the ordered sum of the tile's partials when it was
// split and the value already in the output otherwise. Every term is added in
// a fixed order, so results do not depend on scheduling.
// grid = (rir, dispatch position of the tile, segment of the tile)
// ---------------------------------------------------------------------------
// v + x[0] + x[stride] + ... + x[(n - 1) stride], added in that order; the
// loads of a group of 32 (then 8) are issued together, so a tile split into
// many items costs few memory round trips (the order of the additions, and
// so the result, does not depend on the grouping).
template <int B>
__device__ __forceinline__ float ordered_block(float v, const float *__restrict__ x, size_t stride) {
  float t[B];
#pragma unroll
  for (int u = 0; u < B; ++u) t[u] = x[(size_t)u * stride];
#pragma unroll
  for (int u = 0; u < B; ++u) v += t[u];
  return v;
}
__device__ __forceinline__ float ordered_sum(float v, const float *__restrict__ x, size_t stride, int n) {
  int cc = 0;
  for (; cc + 32 <= n; cc += 32) v = ordered_block<32>(v, x + (size_t)cc * stride, stride);
  for (; cc + 8 <= n; cc += 8) v = ordered_block<8>(v, x + (size_t)cc * stride, stride);
  if (cc < n) {  // the last (fewer than 8) terms, loaded together
    const int m = n - cc;
    float t[7];
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (u < m) t[u] = x[(size_t)(cc + u) * stride];
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (u < m) v += t[u];
  }
  return v;
}

// A run of n terms added to v in the fixed order of the reduce (the run
// length alone decides it): fewer than RED_SLICE_MIN terms one by one, longer
// runs as RED_SLICES consecutive slices, each summed in order from its first term,
// whose sums are then added to v in slice order. Launches with a long run
// take RED_SLICES threads per sample (a block covers RED_SAMPLES samples):
// each thread sums one slice and the sample's first thread adds the slice
// sums; the others take one thread per sample and add term by term (all
// their runs are short). n is uniform over the block (its barriers are);
// active: this thread's sample takes the run.
constexpr int RED_SAMPLES = 256 / RED_SLICES;
static_assert(TILE % 256 == 0 && LONG_TILE % 256 == 0 && 256 % RED_SAMPLES == 0, "reduce blocks tile the tile");
__device__ __forceinline__ float run_sum(float v, const float *__restrict__ x, size_t stride, int n, bool active,
                                         int slice, int ks, float (*red)[RED_SAMPLES]) {
  if (n < RED_SLICE_MIN) {
    if (active && slice == 0) v = ordered_sum(v, x, stride, n);
    return v;
  }
  const int m = (n + RED_SLICES - 1) / RED_SLICES;
  const int a = slice * m, len = min(m, n - a);
  red[slice][ks] = active ? ordered_sum(0.0f, x + (size_t)a * stride, stride, len) : 0.0f;
  __syncthreads();
  if (active && slice == 0) {
#pragma unroll
    for (int i = 0; i < RED_SLICES; ++i) v += red[i][ks];
  }
  __syncthreads();
  return v;
}

// One run of a sample's terms: n of them, stride apart.
struct Run {
  const float *x;
  size_t stride;
  int n;       // uniform over the block
  bool active;
};

// The reduce launches: plain (no tile was split), gather, sliced (a run of RED_SLICE_MIN
// terms or more).
enum { RED_PLAIN, RED_GATHER, RED_SLICED };

// v and the terms of the runs a, l and r in that order (run_sum). RED_GATHER: where no run
// has more than eight terms, all of them are loaded together, one memory round trip instead
// of three (one receiver: 6.0 -> 4.8 us; 32 receivers: 6.9 -> 4.6). Not for launches whose
// tiles were not split: they have thousands of blocks to hide the latency and would pay for
// the padding to eight loads (1024 RIRs of 2427 samples: 16 us; term by term 9.7; with one
// item per tile known, so no plan lookups either, 6.3).
template <int MODE, class Red>
__device__ __forceinline__ float add_runs(float v, const Run &a, const Run &l, const Run &r, int slice, int ks,
                                          Red &red) {
  const Run *const runs[3] = {&a, &l, &r};
  if constexpr (MODE == RED_SLICED) {
#pragma unroll
    for (int i = 0; i < 3; ++i) v = run_sum(v, runs[i]->x, runs[i]->stride, runs[i]->n, runs[i]->active, slice, ks, red);
  } else if (MODE == RED_GATHER && max(a.n, max(l.n, r.n)) <= 8) {
    float t[3][8];
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (runs[i]->n > 0 && runs[i]->active) {
#pragma unroll
        for (int u = 0; u < 8; ++u) t[i][u] = runs[i]->x[(size_t)min(u, runs[i]->n - 1) * runs[i]->stride];
      }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (runs[i]->n > 0 && runs[i]->active) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v = u < runs[i]->n ? v + t[i][u] : v;
      }
  } else {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (runs[i]->active) v = ordered_sum(v, runs[i]->x, runs[i]->stride, runs[i]->n);
  }
  return v;
}

template <int MODE>
__global__ __launch_bounds__(256) void reduce_kernel(RoomArgs ra, PlanArgs pa, const float *__restrict__ part,
                                                     const float *__restrict__ marg, float *__restrict__ out) {
  constexpr bool SLICED = MODE == RED_SLICED;
  constexpr int SPB = SLICED ? RED_SAMPLES : 256;  // samples per block
  __shared__ float red[SLICED ? RED_SLICES : 1][SLICED ? RED_SAMPLES : 1];
  const int pos = blockIdx.y;
  const int tile_id = pa.n_tiles - 1 - pos;
  // (plain: one item per tile, so item pos * n_rir is a position's first)
  const int C = MODE == RED_PLAIN ? 1 : pa.chunks[tile_id];
  const int rir = blockIdx.x;
  const int TL = ra.tile, T0 = tile_id * TL;
  const int ks = (int)threadIdx.x % SPB, slice = (int)threadIdx.x / SPB;
  const int k0 = blockIdx.z * SPB, k = k0 + ks;
  const int W = (int)(2.0f * ra.half_w);
  const int LM = W / 2 - 1;
  // block-uniform: which runs exist for some sample of this block
  const bool has_l = tile_id > 0 && k0 < W / 2;                    // right margin of tile t-1
  const bool has_r = tile_id + 1 < pa.n_tiles && k0 + SPB > TL - LM;  // left margin of tile t+1
  if (C <= 1 && !has_l && !has_r) return;
  const bool in = k < ra.n_samples - T0 && k < TL;
  const bool zl = in && has_l && k < W / 2;
  const bool zr = in && has_r && k >= TL - LM;
  float *o = out + (size_t)rir * ra.n_samples + T0 + k;
  Run own{part, (size_t)TL, 0, in}, left{marg, (size_t)W, 0, zl}, right{marg, (size_t)W, 0, zr};
  float v = 0.0f;
  const uint32_t first = MODE == RED_PLAIN ? (uint32_t)pos * (uint32_t)pa.n_rir : plan_first_item(pa, pos);
  if (C > 1) {
    own.x = part + ((size_t)first + (size_t)rir * C) * TL + k;
    own.n = C;
  } else if (in && slice == 0 && (zl || zr)) {
    v = *o;
  }
  if (has_l) {  // tile t-1 is dispatched at pos + 1
    left.n = MODE == RED_PLAIN ? 1 : pa.chunks[tile_id - 1];
    left.x = marg + ((size_t)first + (size_t)pa.n_rir * C + (size_t)rir * left.n) * W + LM + k;
  }
  if (has_r) {  // tile t+1 is dispatched at pos - 1
    right.n = MODE == RED_PLAIN ? 1 : pa.chunks[tile_id + 1];
    right.x = marg + ((size_t)first - (size_t)pa.n_rir * right.n + (size_t)rir * right.n) * W + (k - (TL - LM));
  }
  v = add_runs<MODE>(v, own, left, right, slice, ks, red);
  if (in && slice == 0 && (C > 1 || zl || zr)) *o = v;
}

// Batch mode: grid = (output tile of a batch RIR, segment of the tile).
template <int MODE>
__global__ __launch_bounds__(256) void reduce_batch_kernel(const JobDev *__restrict__ jobs,
                                                           const BatchReduce *__restrict__ red_tab,
                                                           const float *__restrict__ part,
                                                           const float *__restrict__ marg) {
  constexpr bool SLICED = MODE == RED_SLICED;
  constexpr int SPB = SLICED ? RED_SAMPLES : 256;
  __shared__ float red[SLICED ? RED_SLICES : 1][SLICED ? RED_SAMPLES : 1];
  const BatchReduce br = red_tab[blockIdx.x];
  const JobDev &jb = jobs[br.job];
  const int n_samples = jb.ra.n_samples;
  const int TL = jb.ra.tile, T0 = (int)br.tile * TL;
  const int ks = (int)threadIdx.x % SPB, slice = (int)threadIdx.x / SPB;
  const int k0 = blockIdx.y * SPB, k = k0 + ks;
  if (k0 >= TL) return;  // the grid covers the batch's longest tiles
  const int W = (int)(2.0f * jb.ra.half_w);
  const int LM = W / 2 - 1;
  const bool has_l = br.nprev > 0 && k0 < W / 2;
  const bool has_r = br.nnext > 0 && k0 + SPB > TL - LM;
  if (br.chunks <= 1 && !has_l && !has_r) return;
  const bool in = k < n_samples - T0 && k < TL;
  const bool zl = in && has_l && k < W / 2;
  const bool zr = in && has_r && k >= TL - LM;
  float *o = jb.out + (size_t)br.rir * n_samples + T0 + k;
  float v = 0.0f;
  if (br.chunks <= 1 && in && slice == 0 && (zl || zr)) v = *o;
  const Run own{part + (size_t)br.first * TILE + k, (size_t)TL, br.chunks > 1 ? (int)br.chunks : 0, in};
  const Run left{marg + (size_t)br.mprev * MARG_UNIT + LM + k, (size_t)W, has_l ? (int)br.nprev : 0, zl};
  const Run right{marg + (size_t)br.mnext * MARG_UNIT + (k - (TL - LM)), (size_t)W, has_r ? (int)br.nnext : 0, zr};
  v = add_runs<MODE>(v, own, left, right, slice, ks, red);
  if (in && slice == 0 && (br.chunks > 1 || zl || zr)) *o = v;
}

// The fixed order of run_sum on one thread: the slices of a long run summed
// one after the other (each from its first term), then added in order.
__device__ __forceinline__ float run_sum_serial(float v, const float *__restrict__ x, size_t stride, int n) {
  if (n < RED_SLICE_MIN) return ordered_sum(v, x, stride, n);
  const int m = (n + RED_SLICES - 1) / RED_SLICES;
  for (int i = 0; i < RED_SLICES; ++i) v += ordered_sum(0.0f, x + (size_t)(i * m) * stride, stride, min(m, n - i * m));
  return v;
}

// Batch mode, tiles that were not split: their own samples are final, and
// only the W - 1 margin samples (the first W/2 and the last W/2 - 1) take the
// neighbours' margins, in the order of reduce_batch_kernel. One 64-lane block
// per reduce entry.
__global__ __launch_bounds__(64) void reduce_margins_kernel(const JobDev *__restrict__ jobs,
                                                            const BatchReduce *__restrict__ red_tab,
                                                            const float *__restrict__ marg) {
  const BatchReduce br = red_tab[blockIdx.x];
  const JobDev &jb = jobs[br.job];
  const int n_samples = jb.ra.n_samples;
  const int TL = jb.ra.tile, T0 = (int)br.tile * TL;
  const int W = (int)(2.0f * jb.ra.half_w);
  const int LM = W / 2 - 1;
  for (int i = (int)threadIdx.x; i < W - 1; i += 64) {
    const int k = i < W / 2 ? i : TL - LM + (i - W / 2);
    if (k >= n_samples - T0) continue;
    const bool zl = br.nprev > 0 && k < W / 2;
    const bool zr = br.nnext > 0 && k >= TL - LM;
    if (!zl && !zr) continue;
    float *o = jb.out + (size_t)br.rir * n_samples + T0 + k;
    float v = *o;
    if (zl) v = run_sum_serial(v, marg + (size_t)br.mprev * MARG_UNIT + LM + k, W, br.nprev);
    if (zr) v = run_sum_serial(v, marg + (size_t)br.mnext * MARG_UNIT + (k - (TL - LM)), W, br.nnext);
    *o = v;
  }
}

// ---------------------------------------------------------------------------
// Launchers (called from ism_host.cpp).
// ---------------------------------------------------------------------------
int launch_tables(const RoomArgs &ra, const float *src, const float *rcv, const float *orient, AxisEntry *tab,
                  AxisOrigin *origin, int *valid, int n_rir, float W, bool half, float *wc, hipStream_t st) {
  const int64_t total = (int64_t)n_rir * ra.n_tab;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65535) blocks = 65535;
  hipLaunchKernelGGL(tables_kernel, dim3((unsigned)(blocks + (wc ? 1 : 0))), dim3(256), 0, st, ra, src, rcv, orient,
                     tab, origin, valid, n_rir, (int)blocks, W, half ? 1 : 0, wc);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Items [first, first + count) of a call, one workgroup of the given threads each, by as
// many launches as the limit of 2^32 - 1 threads per launch asks for (16.7 million items
// of 256 threads).
template <class Launch>
static int launch_items(uint32_t n_items, int threads, Launch &&launch) {
  const uint32_t most = 0xffffffffu / (uint32_t)threads;
  for (uint32_t first = 0; first < n_items;) {
    const uint32_t count = min(n_items - first, most);
    launch(first, count);
    if (hipGetLastError() != hipSuccess) return -1;
    first += count;
  }
  return 0;
}

template <int WT, int TL, int KIND, bool LUT, bool POLAR, bool GEN>
static int launch_acc_w(const RoomArgs &ra, const PlanArgs &pa, uint32_t n_items, const AxisEntry *tab,
                        const AxisOrigin *origin, const int *valid, float *out, float *part, float *marg,
                        const float *wc, hipStream_t st) {
  return launch_items(n_items, item_threads(KIND), [&](uint32_t first, uint32_t count) {
    hipLaunchKernelGGL((accumulate_kernel<WT, TL, KIND, LUT, POLAR, GEN>), dim3(count), dim3(item_threads(KIND)), 0,
                       st, ra, pa, tab, origin, valid, out, part, marg, wc, first);
  });
}

int launch_dump(bool half, const RoomArgs &ra, const PlanArgs &pa, uint32_t n_items, const AxisEntry *tab,
                const AxisOrigin *origin, const int *valid, DumpArgs dump, hipStream_t st) {
  hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, st, dump.count, 0u, 1);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    fprintf(stderr, "ism_debug_enumerate: fill launch: %s\n", hipGetErrorString(e));
    return -1;
  }
  auto *const kernel = half ? &enumerate_dump_kernel<1> : &enumerate_dump_kernel<MOM_WAVES>;
  const int threads = item_threads(half ? ITEM_FP16 : ITEM_MOMENTS);
  const int rc = launch_items(n_items, threads, [&](uint32_t first, uint32_t count) {
    hipLaunchKernelGGL(kernel, dim3(count), dim3(threads), 0, st, ra, pa, tab, origin, valid, dump, first);
  });
  if (rc != 0) fprintf(stderr, "ism_debug_enumerate: enumeration launch failed\n");
  return rc;
}

bool supported_window(int wt, bool gen) {
  if (gen) return wt >= 32 && wt <= MAX_WINDOW && wt % 32 == 0;
  return wt == 32 || wt == 64 || wt == 96 || wt == 128;
}

// Calls the kernel instance of a window class: exact windows W in {32, 64,
// 96, 128} with every tap mode, general-mode caps 32 .. 256 with FP32 or FP16
// taps; FP32 taps with tiles of TILE or LONG_TILE samples, FP32 and table taps also on
// one-wave items (kind ITEM_FEW). fn is a generic lambda taking the template arguments as
// values.
template <class Fn>
static int dispatch_window(int wt, int tile, bool gen, int kind, bool lut, bool polar, Fn &&fn) {
  if ((kind == ITEM_FP16 && lut) || (tile != TILE && (kind != ITEM_MOMENTS || lut || tile != LONG_TILE))) return -2;
  using F = std::false_type;
  using T = std::true_type;
  auto by_mode = [&](auto W, auto G) -> int {
    using S = std::integral_constant<int, TILE>;
    using LT = std::integral_constant<int, LONG_TILE>;
    using Mom = std::integral_constant<int, ITEM_MOMENTS>;
    using Half = std::integral_constant<int, ITEM_FP16>;
    using Few = std::integral_constant<int, ITEM_FEW>;
    auto by_polar = [&](auto Tl, auto K, auto L) -> int {
      return polar ? fn(W, Tl, K, L, T{}, G) : fn(W, Tl, K, L, F{}, G);
    };
    if (kind == ITEM_FP16) return by_polar(S{}, Half{}, F{});
    if (lut) {
      if constexpr (!decltype(G)::value) return kind == ITEM_FEW ? by_polar(S{}, Few{}, T{}) : by_polar(S{}, Mom{}, T{});
      return -2;
    }
    if (kind == ITEM_FEW) return by_polar(S{}, Few{}, F{});
    return tile == LONG_TILE ? by_polar(LT{}, Mom{}, F{}) : by_polar(S{}, Mom{}, F{});
  };
  if (!gen) {
    switch (wt) {
      case 32: return by_mode(std::integral_constant<int, 32>{}, F{});
      case 64: return by_mode(std::integral_constant<int, 64>{}, F{});
      case 96: return by_mode(std::integral_constant<int, 96>{}, F{});
      case 128: return by_mode(std::integral_constant<int, 128>{}, F{});
      default: return -2;
    }
  }
  switch (wt) {
    case 32: return by_mode(std::integral_constant<int, 32>{}, T{});
    case 64: return by_mode(std::integral_constant<int, 64>{}, T{});
    case 96: return by_mode(std::integral_constant<int, 96>{}, T{});
    case 128: return by_mode(std::integral_constant<int, 128>{}, T{});
    case 160: return by_mode(std::integral_constant<int, 160>{}, T{});
    case 192: return by_mode(std::integral_constant<int, 192>{}, T{});
    case 224: return by_mode(std::integral_constant<int, 224>{}, T{});
    case 256: return by_mode(std::integral_constant<int, 256>{}, T{});
    default: return -2;
  }
}

// polar: directional receivers (any tap mode; FP16 items and lut exclusive).
int launch_accumulate(int wt, bool gen, int kind, bool lut, bool polar, const RoomArgs &ra, const PlanArgs &pa,
                      uint32_t n_items, const AxisEntry *tab, const AxisOrigin *origin, const int *valid, float *out,
                      float *part, float *marg, const float *wc, hipStream_t st) {
  return dispatch_window(wt, ra.tile, gen, kind, lut, polar, [&](auto W, auto Tl, auto H, auto L, auto P, auto G) -> int {
    return launch_acc_w<decltype(W)::value, decltype(Tl)::value, decltype(H)::value, decltype(L)::value,
                        decltype(P)::value, decltype(G)::value>(ra, pa, n_items, tab, origin, valid, out, part, marg, wc, st);
  });
}

// grid: workgroups of the persistent launch (at most n_items; the planner
// sizes it from the tuned workgroups per SIMD).
template <int WT, int TL, int KIND, bool LUT, bool POLAR, bool GEN>
static int launch_acc_batch_w(const JobDev *jobs, const BatchItem *items, uint32_t n_items, uint32_t grid,
                              uint32_t *queue, const AxisEntry *tab, const AxisOrigin *origin, const int *valid,
                              float *part, float *marg, hipStream_t st) {
  hipLaunchKernelGGL((accumulate_batch_kernel<WT, TL, KIND, LUT, POLAR, GEN>),
                     dim3(grid), dim3(item_threads(KIND)), 0, st, jobs, items, n_items, queue, tab, origin, valid, part, marg);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// queue[k] = the first item of class k not taken by a workgroup's first pick.
struct QueueInit {
  uint32_t v[kMaxBatchLaunches];
};
__global__ void queue_init_kernel(uint32_t *queue, QueueInit q) {
  if (threadIdx.x < kMaxBatchLaunches) queue[threadIdx.x] = q.v[threadIdx.x];
}

int launch_batch(const JobDev *jobs, int n_jobs, bool any_gen, const BatchRir *rirs, uint32_t n_rir,
                 const BatchItem *items, const BatchClass *cls, int n_classes, bool half, bool lut, bool polar,
                 const BatchReduce *red, uint32_t n_red, uint32_t n_red_split, bool long_runs, int max_tile, AxisEntry *tab,
                 AxisOrigin *origin, int *valid, float *part, float *marg, uint32_t *queue, hipStream_t st,
                 hipEvent_t ev_start, hipEvent_t ev_stop) {
  hipLaunchKernelGGL(tables_batch_kernel, dim3(n_rir + (any_gen ? (unsigned)n_jobs : 0u)), dim3(256), 0, st, jobs, rirs,
                     tab, origin, valid, n_rir, half ? 1 : 0);
  if (hipGetLastError() != hipSuccess) return -1;
  if (queue) {
    QueueInit q = {};
    for (int k = 0; k < n_classes && k < kMaxBatchLaunches; ++k) q.v[k] = cls[k].grid;
    hipLaunchKernelGGL(queue_init_kernel, dim3(1), dim3(64), 0, st, queue, q);
    if (hipGetLastError() != hipSuccess) return -1;
  }
  if (ev_start && hipEventRecord(ev_start, st) != hipSuccess) return -1;
  for (int k = 0; k < n_classes; ++k) {
    if (cls[k].count == 0) continue;
    const BatchItem *it = items + cls[k].first;
    uint32_t *qk = queue ? queue + k : nullptr;
    const int rc = dispatch_window(cls[k].wt, cls[k].tile, cls[k].gen != 0, cls[k].kind, lut, polar,
                                   [&](auto W, auto Tl, auto H, auto L, auto P, auto G) -> int {
                                     return launch_acc_batch_w<decltype(W)::value, decltype(Tl)::value,
                                                               decltype(H)::value, decltype(L)::value,
                                                               decltype(P)::value, decltype(G)::value>(
                                         jobs, it, cls[k].count, cls[k].grid, qk, tab, origin, valid, part, marg, st);
                                   });
    if (rc != 0) return -1;
  }
  if (ev_stop && hipEventRecord(ev_stop, st) != hipSuccess) return -1;
  if (n_red_split > 0) {
    // split tiles, whole tiles; runs of RED_SLICE_MIN terms or more: RED_SLICES threads per sample
    if (long_runs)
      hipLaunchKernelGGL(reduce_batch_kernel<RED_SLICED>, dim3(n_red_split, max_tile / RED_SAMPLES), dim3(256), 0, st, jobs, red,
                         part, marg);
    else
      hipLaunchKernelGGL(reduce_batch_kernel<RED_GATHER>, dim3(n_red_split, max_tile / 256), dim3(256), 0, st, jobs, red, part,
                         marg);
    if (hipGetLastError() != hipSuccess) return -1;
  }
  if (n_red > n_red_split) {  // the other tiles: their margin samples only
    hipLaunchKernelGGL(reduce_margins_kernel, dim3(n_red - n_red_split), dim3(64), 0, st, jobs, red + n_red_split,
                       marg);
    if (hipGetLastError() != hipSuccess) return -1;
  }
  return 0;
}

int launch_reduce(const RoomArgs &ra, const PlanArgs &pa, int n_rir, const float *part, const float *marg,
                  float *out, hipStream_t st) {
  int max_c = 0;  // longest run: the most items of any tile (its own, or a neighbour's margins)
  for (int t = 0; t < pa.n_tiles; ++t) max_c = max(max_c, (int)pa.chunks[t]);
  const int spb = max_c >= RED_SLICE_MIN ? RED_SAMPLES : 256;
  const dim3 grid((unsigned)n_rir, (unsigned)pa.n_tiles, ra.tile / spb);
  auto *const kernel = max_c >= RED_SLICE_MIN ? &reduce_kernel<RED_SLICED>
                       : max_c > 1            ? &reduce_kernel<RED_GATHER>
                                              : &reduce_kernel<RED_PLAIN>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, ra, pa, part, marg, out);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ism
