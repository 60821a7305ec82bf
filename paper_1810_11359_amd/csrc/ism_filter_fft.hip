// Moving-source filtering (Sec. 3.4) by partitioned FFT convolution: the
// paper filters the signal through the trajectory's RIRs with batched FFTs;
// this is that path, written for gfx950 (real transforms through half-size
// complex Stockham transforms in LDS).
//
// The signal x is cut into segments of L = ceil(n_x / n_pos) samples and
// segment p goes through RIR p (y_m[n] = sum_k x[n - k] h_{p(n-k), m}[k]).
// Two plans:
//
// Segment blocks (segments of at most half a transform): input block p is
// segment p as it is, and partition q of an RIR is c L taps long, with (c + 1) L
// - 1 <= N points, so that the product of segment p with partition q lies in
// output block p + c q of the same grid of multiples of L. Every RIR partition
// then meets exactly one input spectrum: a workgroup takes one output block of
// one microphone, transforms the partitions that end there one after the other in
// LDS, multiplies each spectrum by its segment's and adds it up in registers, and
// transforms the sum back. RIRs are read once and no RIR spectrum is written.
// y_m[n] is the sum of the up to c + 1 blocks that cover n.
//
// Fixed blocks (longer segments, whose RIR spectra several blocks use): blocks
// of B samples, N = 2B point transforms:
//   - RIR partition q of point p and microphone m, h_{p,m}[qB, qB + B), has
//     the spectrum H[p][m][q];
//   - input block i, x[iB, iB + B), is split into pieces, one per segment it
//     touches (samples of other segments zeroed); piece r (segment p0(i) + r)
//     has the spectrum X[i][r];
//   - piece (i, r) times partition q is the linear convolution of two B-sample
//     sequences placed at (i + q) B: 2B - 1 samples, exact in an N-point
//     circular convolution. Output block b collects, in the frequency domain,
//     Y[m][b] = sum_q sum_r X[b - q][r] H[p(b - q, r)][m][q] (q, then r, in
//     increasing order), and
//   - y_m[bB + t] = z_b[t] + z_{b-1}[B + t], z_b = IFFT(Y[m][b]) (overlap-add).
// Every sum has a fixed order, so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "ism_internal.h"
#include "ism_math.h"

namespace ism {

// Transforms: the real N-point transform of each block (N = 2B, the second
// half zero) is taken as an M = N/2-point complex transform of the packed
// sequence z[n] = x[2n] + i x[2n+1], then split into the spectrum of x: with
// W = exp(-2 pi i / N),
//   X[k] = (Z[k] + conj Z[M-k]) / 2 + W^k (Z[k] - conj Z[M-k]) / (2i), 0 < k < M,
//   X[0] = Re Z[0] + Im Z[0], X[M] = Re Z[0] - Im Z[0] (both real),
// stored as M complex bins, bin 0 holding (X[0], X[M]). The inverse runs the
// same steps backwards (Z[k] = E[k] + i O[k] from Y[k] and conj Y[M-k], then
// an inverse M-point transform scaled by 1/M gives y[2n] + i y[2n+1]).
// The complex transforms are Stockham passes of radix 16 and 8, each thread holding
// its butterflies' points (16 in all) in registers between two barriers; the data
// stay in LDS (M complex per transform). A pass's constants are consecutive in the lanes:
// read from one table of roots they were a cache line per lane. 8 microphones, 100
// segments of 4800 samples, RIRs of 96000 taps: 428 us so, with radix 8 and 4; 355 us
// with a table per pass and radix 16; 313 us with the padded LDS places as well; 305 us
// with the upper half's twiddles in the butterflies' first sums.

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(__builtin_fmaf(a.x, b.x, -a.y * b.y), __builtin_fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// c + a b and c - a b (one rounding less than with the product apart)
__device__ __forceinline__ float2 cfma(float2 c, float2 a, float2 b) {
  return make_float2(__builtin_fmaf(a.x, b.x, __builtin_fmaf(-a.y, b.y, c.x)),
                     __builtin_fmaf(a.x, b.y, __builtin_fmaf(a.y, b.x, c.y)));
}
__device__ __forceinline__ float2 cneg(float2 a) { return make_float2(-a.x, -a.y); }
// a times -i (forward) or +i (inverse)
__device__ __forceinline__ float2 rot_i(float2 a, bool inv) {
  return inv ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// T[n] = exp(-2 pi i n / N), n < N, computed in double by the compiler (the first
// octant by repeated rotation, to 1e-12; the others by symmetry) and rounded once.
template <int N>
struct alignas(8) Roots {
  float t[N][2];
};
constexpr double root_sin(double x) {  // 0 <= x <= pi/4
  double term = x, sum = x;
  for (int k = 1; k < 12; ++k) {
    term *= -x * x / ((2.0 * k) * (2.0 * k + 1.0));
    sum += term;
  }
  return sum;
}
constexpr double root_cos(double x) {
  double term = 1.0, sum = 1.0;
  for (int k = 1; k < 12; ++k) {
    term *= -x * x / ((2.0 * k - 1.0) * (2.0 * k));
    sum += term;
  }
  return sum;
}
template <int N>
constexpr Roots<N> make_roots() {
  Roots<N> r{};
  constexpr double step = 2.0 * 3.14159265358979323846 / N;
  const double cs = root_cos(step), sn = root_sin(step);
  double c = 1.0, s = 0.0;  // cos, sin of 2 pi n / N
  for (int n = 0; n <= N / 8; ++n) {
    const float cf = (float)c, sf = (float)s;
    // the octants by symmetry
    const int h = N / 2, q = N / 4;
    const int at[8] = {n, q - n, (q + n) % N, h - n, (h + n) % N, h + q - n, (h + q + n) % N, (N - n) % N};
    const float re[8] = {cf, sf, -sf, -cf, -cf, -sf, sf, cf}, im[8] = {-sf, -cf, -cf, -sf, sf, cf, cf, sf};
    for (int i = 0; i < 8; ++i) {
      r.t[at[i]][0] = re[i];
      r.t[at[i]][1] = im[i];
    }
    const double c2 = c * cs - s * sn;
    s = s * cs + c * sn;
    c = c2;
  }
  return r;
}

// The transforms' constants, all taken from the 16384-point roots:
// pass[R][Ns]: exp(-2 pi i t k / (R Ns)) at [t - 1][k], 1 <= t < R, k < Ns, so that the
// lanes of a wave (consecutive k) read consecutive elements; split<M>: exp(-2 pi i k / 2M),
// k < M.
template <int R, int Ns> struct PassTable {
  float t[(R - 1) * Ns][2];
};
template <int M> struct SplitTable {
  float t[M][2];
};
struct alignas(16) FftTables {
  PassTable<8, 8> p8_8;
  PassTable<8, 16> p8_16;
  PassTable<8, 64> p8_64;
  PassTable<8, 128> p8_128;
  PassTable<8, 256> p8_256;
  PassTable<8, 1024> p8_1024;
  PassTable<16, 16> p16_16;
  PassTable<16, 256> p16_256;
  SplitTable<256> s256;
  SplitTable<512> s512;
  SplitTable<1024> s1024;
  SplitTable<2048> s2048;
  SplitTable<4096> s4096;
  SplitTable<8192> s8192;
};
constexpr int kRoots = 16384;
template <int R, int Ns>
constexpr void fill_pass(PassTable<R, Ns> &p, const Roots<kRoots> &r) {
  for (int t = 1; t < R; ++t)
    for (int k = 0; k < Ns; ++k)
      for (int i = 0; i < 2; ++i) p.t[(t - 1) * Ns + k][i] = r.t[t * k * (kRoots / (R * Ns))][i];
}
template <int M>
constexpr void fill_split(SplitTable<M> &p, const Roots<kRoots> &r) {
  for (int k = 0; k < M; ++k)
    for (int i = 0; i < 2; ++i) p.t[k][i] = r.t[k * (kRoots / (2 * M))][i];
}
constexpr FftTables make_tables() {
  const Roots<kRoots> r = make_roots<kRoots>();
  FftTables f{};
  fill_pass(f.p8_8, r);
  fill_pass(f.p8_16, r);
  fill_pass(f.p8_64, r);
  fill_pass(f.p8_128, r);
  fill_pass(f.p8_256, r);
  fill_pass(f.p8_1024, r);
  fill_pass(f.p16_16, r);
  fill_pass(f.p16_256, r);
  fill_split(f.s256, r);
  fill_split(f.s512, r);
  fill_split(f.s1024, r);
  fill_split(f.s2048, r);
  fill_split(f.s4096, r);
  fill_split(f.s8192, r);
  return f;
}
__constant__ FftTables kTables = make_tables();

// Offsets (bytes) of a pass's and of a split's constants.
template <int R, int Ns> constexpr int pass_offset() {
  if constexpr (R == 8 && Ns == 8) return offsetof(FftTables, p8_8);
  else if constexpr (R == 8 && Ns == 16) return offsetof(FftTables, p8_16);
  else if constexpr (R == 8 && Ns == 64) return offsetof(FftTables, p8_64);
  else if constexpr (R == 8 && Ns == 128) return offsetof(FftTables, p8_128);
  else if constexpr (R == 8 && Ns == 256) return offsetof(FftTables, p8_256);
  else if constexpr (R == 8 && Ns == 1024) return offsetof(FftTables, p8_1024);
  else if constexpr (R == 16 && Ns == 16) return offsetof(FftTables, p16_16);
  else return offsetof(FftTables, p16_256);
}
template <int M> constexpr int split_offset() {
  return M == 256 ? offsetof(FftTables, s256) : M == 512 ? offsetof(FftTables, s512) :
         M == 1024 ? offsetof(FftTables, s1024) : M == 2048 ? offsetof(FftTables, s2048) :
         M == 4096 ? offsetof(FftTables, s4096) : offsetof(FftTables, s8192);
}

// Element i (a 32-bit offset) of the constants at byte offset off of T.
typedef const char *Tables;
__device__ __forceinline__ float2 at32(const float2 *__restrict__ t, int i) {
  return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(t) + (uint32_t)(i << 3));
}
__device__ __forceinline__ float2 root(Tables T, int off, int i) {
  return *reinterpret_cast<const float2 *>(T + off + (uint32_t)(i << 3));
}

// LDS place of point i: one slot in 17 stays empty, so that the strided writes of the
// first pass spread over the banks.
__device__ __forceinline__ constexpr int pad(int i) { return i + (i >> 4); }
template <int M> constexpr int kBufLen = M + M / 16;

// 4-point DFT in place, kernel exp(-+2 pi i t s / 4); TW: points 2 and 3 times w2 and w3.
template <bool TW>
__device__ __forceinline__ void dft4(float2 *v, float2 w2, float2 w3, bool inv) {
  const float2 t0 = TW ? cfma(v[0], v[2], w2) : cadd(v[0], v[2]);
  const float2 t1 = TW ? cfma(v[0], cneg(v[2]), w2) : csub(v[0], v[2]);
  const float2 t2 = TW ? cfma(v[1], v[3], w3) : cadd(v[1], v[3]);
  const float2 t3 = rot_i(TW ? cfma(v[1], cneg(v[3]), w3) : csub(v[1], v[3]), inv);
  v[0] = cadd(t0, t2);
  v[2] = csub(t0, t2);
  v[1] = cadd(t1, t3);
  v[3] = csub(t1, t3);
}

// R-point DFT of v in place (R = 8, 16), kernel exp(-+2 pi i t s / R); TW: point t times
// w[t - 1] first (points R/2 and on within their first sums).
template <int R, bool TW>
__device__ __forceinline__ void dft_small(float2 *v, const float2 *w, bool inv) {
  const float2 one = make_float2(1.0f, 0.0f);
  if constexpr (TW)
#pragma unroll
    for (int t = 1; t < R / 2; ++t) v[t] = cmul(v[t], w[t - 1]);
  if constexpr (R == 16) {
    // 4 x 4: DFTs over t1 of the points t = 4 t1 + t2, times exp(-+2 pi i t2 s1 / 16),
    // DFTs over t2: points s = s1 + 4 s2
    constexpr float c1 = 0.92387953251128676f, s1 = 0.38268343236508977f, h = 0.70710678118654752f;
    constexpr float re[10] = {1.0f, c1, h, s1, 0.0f, 0.0f, -h, 0.0f, 0.0f, -c1};
    constexpr float im[10] = {0.0f, -s1, -h, -c1, -1.0f, 0.0f, -h, 0.0f, 0.0f, s1};
    float2 u[4][4];
#pragma unroll
    for (int t2 = 0; t2 < 4; ++t2) {
#pragma unroll
      for (int t1 = 0; t1 < 4; ++t1) u[t2][t1] = v[4 * t1 + t2];
      dft4<TW>(u[t2], TW ? w[7 + t2] : one, TW ? w[11 + t2] : one, inv);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float2 x[4] = {u[0][i], u[1][i], u[2][i], u[3][i]};
      float2 k[4];
#pragma unroll
      for (int t2 = 0; t2 < 4; ++t2) k[t2] = make_float2(re[t2 * i], inv ? -im[t2 * i] : im[t2 * i]);
      if (i == 0) {
        dft4<false>(x, one, one, inv);
      } else {
        x[1] = cmul(x[1], k[1]);
        if (i == 2) {  // k[2] = -+i
          x[2] = rot_i(x[2], inv);
          x[3] = cmul(x[3], k[3]);
          dft4<false>(x, one, one, inv);
        } else {
          dft4<true>(x, k[2], k[3], inv);
        }
      }
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) v[i + 4 * s2] = x[s2];
    }
  } else {
    // DFTs of the even and odd points, combined with exp(-+2 pi i s / 8)
    float2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft4<TW>(e, TW ? w[3] : one, TW ? w[5] : one, inv);
    dft4<TW>(o, TW ? w[4] : one, TW ? w[6] : one, inv);
    constexpr float h = 0.70710678118654752f;  // 1 / sqrt(2)
    // h o1 and h o3 are the products
    const float2 o1 = inv ? make_float2(o[1].x - o[1].y, o[1].x + o[1].y)
                          : make_float2(o[1].x + o[1].y, o[1].y - o[1].x);
    const float2 o2 = rot_i(o[2], inv);
    const float2 o3 = inv ? make_float2(-(o[3].x + o[3].y), o[3].x - o[3].y)
                          : make_float2(o[3].y - o[3].x, -(o[3].x + o[3].y));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = make_float2(__builtin_fmaf(h, o1.x, e[1].x), __builtin_fmaf(h, o1.y, e[1].y));
    v[5] = make_float2(__builtin_fmaf(-h, o1.x, e[1].x), __builtin_fmaf(-h, o1.y, e[1].y));
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = make_float2(__builtin_fmaf(h, o3.x, e[3].x), __builtin_fmaf(h, o3.y, e[3].y));
    v[7] = make_float2(__builtin_fmaf(-h, o3.x, e[3].x), __builtin_fmaf(-h, o3.y, e[3].y));
  }
}

// Threads per transform: 16 points (one radix-16 or two radix-8 butterflies of a pass,
// or eight bin pairs (k, M - k)) each. A workgroup holds one transform of 8192 points on
// 512 threads (two workgroups per CU, 16 waves), smaller ones in half the LDS on 256.
template <int M> struct FftShape {
  static constexpr int TPF = M / 16;
  static constexpr int FPB = TPF < 256 ? 256 / TPF : 1;
  static constexpr int NT = TPF * FPB;
  static constexpr int PAIRS = M / 2 / TPF;
};

// A thread's twiddles of one pass (radix R, span Ns).
template <int M, int R, int Ns> struct PassRoots {
  static constexpr int TPF = FftShape<M>::TPF, NB = M / R / TPF;  // butterflies per thread
  static_assert(NB >= 1 && NB * R * TPF == M, "pass shape");
  float2 w[NB][R - 1];
  __device__ __forceinline__ void load(Tables T, int tid) {
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
      for (int t = 1; t < R; ++t)
        w[u][t - 1] = root(T, pass_offset<R, Ns>() + (t - 1) * Ns * 8, (tid + u * TPF) & (Ns - 1));
  }
};

// One Stockham pass of radix R and span Ns over the M points at a (LDS): the
// butterfly j (k = j mod Ns) takes point j + t M/R, t < R, twiddles it by
// exp(-+2 pi i t k / (R Ns)), and writes its DFT to the points (j - k) R + k + s Ns.
// All LDS reads of the pass happen before the first barrier and all writes after it.
template <int M, int R, int Ns>
__device__ __forceinline__ void fft_pass(float2 *a, int tid, const PassRoots<M, R, Ns> &p, bool inv) {
  constexpr int TPF = FftShape<M>::TPF, NB = M / R / TPF;
  float2 v[NB][R];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int t = 0; t < R; ++t) v[u][t] = a[pad(tid) + pad(u * TPF + t * (M / R))];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int j = tid + u * TPF;
    const int k = j & (Ns - 1);
    float2 w[R - 1];
#pragma unroll
    for (int t = 0; t < R - 1; ++t) w[t] = make_float2(p.w[u][t].x, inv ? -p.w[u][t].y : p.w[u][t].y);
    dft_small<R, true>(v[u], w, inv);
    const int o = (j - k) * R + k;
#pragma unroll
    for (int s = 0; s < R; ++s) a[Ns % 16 ? pad(o + s * Ns) : pad(o) + pad(s * Ns)] = v[u][s];
  }
  __syncthreads();
}

// The first pass (span 1, no twiddles): points from load, which may read a (IN_LDS).
template <int M, int R, bool IN_LDS, class Load>
__device__ __forceinline__ void fft_first(Load &&load, float2 *a, int tid, bool inv) {
  constexpr int TPF = FftShape<M>::TPF, NB = M / R / TPF;
  float2 v[NB][R];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int t = 0; t < R; ++t) v[u][t] = load(tid + u * TPF + t * (M / R));
  if constexpr (IN_LDS) __syncthreads();
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    dft_small<R, false>(v[u], nullptr, inv);
    const int o = R * (tid + u * TPF);
#pragma unroll
    for (int s = 0; s < R; ++s) a[pad(o) + s] = v[u][s];
  }
  __syncthreads();
}

// M-point complex transform into a (LDS), natural order in and out; point n
// of the input is load(n). The passes after the first (radix R0) work in a. KEEP: all
// twiddles are fetched at init (one round trip to memory beside the input's, where
// fetching them pass by pass takes one each), else with their pass.
template <int M, bool KEEP> struct Fft;
template <int M, int R0, bool KEEP, class... Passes> struct FftPasses;
template <int M, int R0, bool KEEP> struct FftPasses<M, R0, KEEP> {
  __device__ __forceinline__ void init(Tables, int) {}
  __device__ __forceinline__ void rest(float2 *, int, Tables, bool) {}
};
template <int M, int R0, bool KEEP, class P, class... Passes>
struct FftPasses<M, R0, KEEP, P, Passes...> : FftPasses<M, R0, KEEP, Passes...> {
  typedef FftPasses<M, R0, KEEP, Passes...> Next;
  P p;
  __device__ __forceinline__ void init(Tables T, int tid) {
    if constexpr (KEEP) p.load(T, tid);
    Next::init(T, tid);
  }
  __device__ __forceinline__ void rest(float2 *a, int tid, Tables T, bool inv) {
    if constexpr (!KEEP) p.load(T, tid);
    fft_pass(a, tid, p, inv);
    Next::rest(a, tid, T, inv);
  }
  template <bool IN_LDS = false, class Load>
  __device__ __forceinline__ void run(Load &&load, float2 *a, int tid, Tables T, bool inv) {
    fft_first<M, R0, IN_LDS>(load, a, tid, inv);
    rest(a, tid, T, inv);
  }
};
template <bool KEEP> struct Fft<256, KEEP> : FftPasses<256, 16, KEEP, PassRoots<256, 16, 16>> {};
template <bool KEEP> struct Fft<512, KEEP> : FftPasses<512, 8, KEEP, PassRoots<512, 8, 8>, PassRoots<512, 8, 64>> {};
template <bool KEEP>
struct Fft<1024, KEEP> : FftPasses<1024, 16, KEEP, PassRoots<1024, 8, 16>, PassRoots<1024, 8, 128>> {};
template <bool KEEP>
struct Fft<2048, KEEP> : FftPasses<2048, 16, KEEP, PassRoots<2048, 16, 16>, PassRoots<2048, 8, 256>> {};
template <bool KEEP>
struct Fft<4096, KEEP> : FftPasses<4096, 16, KEEP, PassRoots<4096, 16, 16>, PassRoots<4096, 16, 256>> {};
template <bool KEEP>
struct Fft<8192, KEEP>
    : FftPasses<8192, 16, KEEP, PassRoots<8192, 8, 16>, PassRoots<8192, 8, 128>, PassRoots<8192, 8, 1024>> {};

// Spectrum bins k < M of the real sequence packed in a (transformed) to o.
template <int M>
__device__ __forceinline__ void real_split(const float2 *a, int tid, Tables T, float2 *__restrict__ o) {
  for (int k = tid; k < M; k += FftShape<M>::TPF) {
    if (k == 0) {
      o[0] = make_float2(a[0].x + a[0].y, a[0].x - a[0].y);
      continue;
    }
    const float2 zk = a[pad(k)], am = a[pad(M - k)], zm = make_float2(am.x, -am.y);  // conj Z[M-k]
    const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
    const float2 d = csub(zk, zm);
    const float2 od = make_float2(0.5f * d.y, -0.5f * d.x);  // d / (2i)
    o[k] = cfma(e, root(T, split_offset<M>(), k), od);
  }
}

// Point k of the packed sequence Z whose inverse transform gives a real
// block, from its packed spectrum Y (M bins, bin 0 holding bins 0 and M).
template <int M>
__device__ __forceinline__ float2 real_merge(const float2 *__restrict__ Y, int k, Tables T) {
  if (k == 0) {
    const float2 y0 = Y[0];
    return make_float2(0.5f * (y0.x + y0.y), 0.5f * (y0.x - y0.y));
  }
  const float2 yk = Y[k], ym = make_float2(Y[M - k].x, -Y[M - k].y);  // conj Y[M-k]
  const float2 e = make_float2(0.5f * (yk.x + ym.x), 0.5f * (yk.y + ym.y));
  const float2 tk = root(T, split_offset<M>(), k), w = make_float2(tk.x, -tk.y);  // exp(+2 pi i k / N)
  const float2 d = csub(yk, ym);
  return cfma(e, make_float2(-0.5f * d.y, 0.5f * d.x), w);  // e + i W^-k d / 2
}

// Segment of input block i's piece r, or -1 when the piece is empty.
__device__ __forceinline__ int piece_segment(int i, int r, int B, int L, int n_x, int n_pos) {
  const int lo = i * B, hi = min(lo + B, n_x);  // samples [lo, hi)
  const int p = lo / L + r;
  if (p >= n_pos || p * L >= hi) return -1;
  return p;
}

// Spectra of the RIR partitions (workgroups below rir_wgs), transform row =
// (p * n_mic + m) * P + q, and of the input pieces, transform i * R + r (empty pieces
// are skipped: their spectra are never read). One launch: a transform kernel of a few
// workgroups takes 5 .. 9 us, most of it the fetch of its code.
template <int M>
__global__ __launch_bounds__(FftShape<M>::NT) void fft_parts_kernel(const float *__restrict__ rir, int n_rir, int P,
                                                                  int n_rir_rows, int rir_wgs,
                                                                  float2 *__restrict__ H, const float *__restrict__ x,
                                                                  int n_x, int n_pos, int L, int R, int n_in_rows,
                                                                  float2 *__restrict__ X) {
  const Tables T = reinterpret_cast<Tables>(&kTables);
  constexpr int TPF = FftShape<M>::TPF, FPB = FftShape<M>::FPB;
  __shared__ float2 buf[FPB][kBufLen<M>];
  const int f = threadIdx.x / TPF, tid = threadIdx.x % TPF;
  // samples [lo, hi) of the M at s, the rest is zero
  const float *s;
  int lo, hi;
  float2 *o = nullptr;
  if ((int)blockIdx.x < rir_wgs) {
    const int row = blockIdx.x * FPB + f, q = row % P;
    s = rir + (size_t)(row / P) * n_rir + (size_t)q * M;  // B = M samples per partition
    lo = 0;
    hi = row < n_rir_rows ? min(M, n_rir - q * M) : 0;
    if (row < n_rir_rows) o = H + (size_t)row * M;
  } else {
    const int row = ((int)blockIdx.x - rir_wgs) * FPB + f, i = row / R;
    const int p = row < n_in_rows ? piece_segment(i, row % R, M, L, n_x, n_pos) : -1;
    // samples of the block (B = M) inside segment p
    s = x + (size_t)i * M;
    lo = p >= 0 ? max(p * L - i * M, 0) : 0;
    hi = p >= 0 ? min(min(p * L + L, n_x) - i * M, M) : 0;
    if (p >= 0) o = X + (size_t)row * M;
  }
  Fft<M, true> fft;
  fft.init(T, tid);
  fft.run([&](int n) {
    const int i0 = 2 * n, i1 = 2 * n + 1;
    return make_float2(i0 >= lo && i0 < hi ? s[i0] : 0.0f, i1 >= lo && i1 < hi ? s[i1] : 0.0f);
  }, buf[f], tid, T, false);
  if (o) real_split<M>(buf[f], tid, T, o);
}

// Y[m][b][k] = sum over q, then r of X[b - q][r][k] H[p][m][q][k], k < M
// (bin 0 holds the two real bins 0 and M: their products are taken apart).
// grid = (M / 256, n_out_blocks, n_mic).
__global__ __launch_bounds__(256) void spectrum_mac_kernel(const float2 *__restrict__ X, const float2 *__restrict__ H,
                                                           int n_x, int n_pos, int n_mic, int L, int B, int M, int P,
                                                           int R, int n_in_blocks, float2 *__restrict__ Y) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y, m = blockIdx.z;
  const float2 *__restrict__ Xk = X + k;
  const float2 *__restrict__ Hk = H + (size_t)m * P * M + k;
  float2 acc = make_float2(0.0f, 0.0f);
  // input blocks i = b - q that exist: q in [q0, q1]; the pieces of block i
  // are the segments p0(i), p0(i) + 1, ... up to the first empty one
  const int q0 = max(0, b - (n_in_blocks - 1)), q1 = min(P - 1, b);
  for (int q = q0; q <= q1; ++q) {
    const int i = b - q;
    const int lo = i * B, hi = min(lo + B, n_x);
    const int p0 = lo / L;
    for (int r = 0; r < R; ++r) {
      const int p = p0 + r;
      if (p >= n_pos || p * L >= hi) break;  // uniform over the block
      const float2 xv = Xk[((size_t)i * R + r) * M];
      const float2 hv = Hk[((size_t)p * n_mic * P + q) * M];
      if (k == 0) {
        acc.x = __builtin_fmaf(xv.x, hv.x, acc.x);
        acc.y = __builtin_fmaf(xv.y, hv.y, acc.y);
      } else {
        acc.x = __builtin_fmaf(xv.x, hv.x, acc.x);
        acc.x = __builtin_fmaf(-xv.y, hv.y, acc.x);
        acc.y = __builtin_fmaf(xv.x, hv.y, acc.y);
        acc.y = __builtin_fmaf(xv.y, hv.x, acc.y);
      }
    }
  }
  Y[((size_t)m * gridDim.y + b) * M + k] = acc;
}

// z[m][b] = IFFT(Y[m][b]) (N real samples); transform row = m * n_out_blocks + b.
template <int M>
__global__ __launch_bounds__(FftShape<M>::NT) void ifft_block_kernel(const float2 *__restrict__ Y, int n_rows,
                                                               float *__restrict__ z) {
  const Tables T = reinterpret_cast<Tables>(&kTables);
  constexpr int TPF = FftShape<M>::TPF, FPB = FftShape<M>::FPB;
  __shared__ float2 buf[FPB][kBufLen<M>];
  const int f = threadIdx.x / TPF, tid = threadIdx.x % TPF;
  const int row = blockIdx.x * FPB + f;
  const bool live = row < n_rows;
  const float2 *Yr = Y + (size_t)(live ? row : 0) * M;
  Fft<M, true> fft;
  fft.init(T, tid);
  fft.run([&](int n) { return live ? real_merge<M>(Yr, n, T) : make_float2(0.0f, 0.0f); }, buf[f], tid, T, true);
  if (live) {
    constexpr float inv_m = 1.0f / (float)M;
    const float2 *a = buf[f];
    float2 *o = reinterpret_cast<float2 *>(z + (size_t)row * 2 * M);
    for (int n = tid; n < M; n += TPF) o[n] = make_float2(a[pad(n)].x * inv_m, a[pad(n)].y * inv_m);
  }
}

// y[m][bB + t] = z[m][b][t] + z[m][b - 1][B + t]; grid = (ceil(n_y / 256), n_mic).
__global__ __launch_bounds__(256) void overlap_add_kernel(const float *__restrict__ z, int B, int N, int n_out_blocks,
                                                          float *__restrict__ y, int n_y) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  if (n >= n_y) return;
  const int b = n / B, t = n % B;
  const float *zm = z + (size_t)m * n_out_blocks * N;
  float v = zm[(size_t)b * N + t];
  if (b > 0) v += zm[(size_t)(b - 1) * N + B + t];
  y[(size_t)m * n_y + n] = v;
}

// ---------------------------------------------------------------------------
// Segment blocks.
// ---------------------------------------------------------------------------
// Spectra of the segments: row p, samples [p L, min(p L + L, n_x)).
template <int M>
__global__ __launch_bounds__(FftShape<M>::NT) void seg_input_kernel(const float *__restrict__ x, int n_x, int L,
                                                                    int n_seg, float2 *__restrict__ X) {
  typedef FftShape<M> Sh;
  const Tables T = reinterpret_cast<Tables>(&kTables);
  __shared__ float2 buf[Sh::FPB][kBufLen<M>];
  const int f = threadIdx.x / Sh::TPF, tid = threadIdx.x % Sh::TPF;
  const int p = blockIdx.x * Sh::FPB + f;
  const int len = p < n_seg ? min(L, n_x - p * L) : 0;
  const float *xs = x + (size_t)p * L;
  Fft<M, true> fft;
  fft.init(T, tid);
  fft.run([&](int n) {
    const int i0 = 2 * n, i1 = 2 * n + 1;
    return make_float2(i0 < len ? xs[i0] : 0.0f, i1 < len ? xs[i1] : 0.0f);
  }, buf[f], tid, T, false);
  if (p < n_seg) real_split<M>(buf[f], tid, T, X + (size_t)p * M);
}

// Transforms whose twiddles seg_filter_kernel holds in registers over its partitions, with
// two workgroups per CU at 256 VGPRs: up to 4096 points. That is faster than four
// workgroups that fetch them (8 microphones, 100 segments of 1600, RIRs of 8000 taps: the
// call 50.2 us against 59.5); 8192 points do not have the registers for it.
template <int M> constexpr bool kKeepRoots = M <= 4096;

// z[row] of row = (m n_blk + b) S + g: the inverse transform of the sum over the
// partitions q of group g (PS of them) of X[b - c q] H_{b - c q, m}[q], with
// 2M points of which the first (c + 1) L are kept. q counts from 0, or (window: signals of
// fewer segments than the RIR's partitions span) from the first that meets a segment. RIRs are read once and no RIR spectrum
// goes to memory (fixed blocks write and read twice the RIRs). Bounded by the transforms:
// VALU issue (0.47 of the slots) and waits for the LDS passes and their barriers. 8 microphones, 100 segments of 4800 samples, RIRs of 96000 taps (307
// MB): 293 us with the launches around it 310, fixed blocks of radix 8 677; segments of
// 1600, RIRs of 8000 taps: 35 and 47.5 against 81.
template <int M>
__global__ __launch_bounds__(FftShape<M>::NT) __attribute__((amdgpu_waves_per_eu(kKeepRoots<M> ? 2 : 4))) void seg_filter_kernel(
    const float *__restrict__ rir, int n_mic, int n_rir, const float2 *__restrict__ X, int n_seg, int L, int c, int P,
    int S, int PS, bool window, int n_blk, int n_rows, float *__restrict__ z) {
  typedef FftShape<M> Sh;
  constexpr int TPF = Sh::TPF, PAIRS = Sh::PAIRS;
  Tables T = reinterpret_cast<Tables>(&kTables);
  __shared__ float2 buf[Sh::FPB][kBufLen<M>];
  const int f = Sh::FPB == 1 ? 0 : threadIdx.x / TPF, tid0 = Sh::FPB == 1 ? threadIdx.x : threadIdx.x % TPF;
  const int row = blockIdx.x * Sh::FPB + f;
  const bool live = row < n_rows;
  const int g = row % S, b = (row / S) % n_blk, m = row / S / n_blk;
  float2 *const a = buf[f];
  // bins k = tid + u TPF and M - k; in place of bins 0 and M: the packed bin 0
  // (bins 0 and M, both real) and bin M/2
  float2 y1[PAIRS], y2[PAIRS];
#pragma unroll
  for (int u = 0; u < PAIRS; ++u) y1[u] = y2[u] = make_float2(0.0f, 0.0f);
  const int part = c * L;
  int q0 = g * PS;
  if (window) q0 += max(b - n_seg + c, 0) / c;
  Fft<M, kKeepRoots<M>> fft;
  fft.init(T, tid0);
  // (every transform of the workgroup takes PS turns: the barriers are the workgroup's)
  for (int i = 0; i < PS; ++i) {
    // keeps twiddles and addresses in the loop: held across it they take 100 registers
    int tid = tid0;
    if constexpr (!kKeepRoots<M>) __asm__ volatile("" : "+s"(T), "+v"(tid));
    const int q = q0 + i, p = b - c * q;
    const bool has = live && q < P && p >= 0 && p < n_seg;
    if (Sh::FPB == 1 && !has) continue;  // uniform over the workgroup
    const int len = has ? min(part, n_rir - q * part) : 0;
    const float *h = rir + (has ? ((size_t)p * n_mic + m) * n_rir + (size_t)q * part : 0);
    fft.run([&](int n) {
      const int i0 = 2 * n, i1 = 2 * n + 1;
      return make_float2(i0 < len ? h[i0] : 0.0f, i1 < len ? h[i1] : 0.0f);
    }, a, tid, T, false);
    if (has) {
      const float2 *__restrict__ Xp = X + (size_t)p * M;
#pragma unroll
      for (int u = 0; u < PAIRS; ++u) {
        const int k = tid + u * TPF;
        if (k == 0) {
          const float2 x0 = Xp[0], a0 = a[0];
          y1[0].x = __builtin_fmaf(x0.x, a0.x + a0.y, y1[0].x);
          y1[0].y = __builtin_fmaf(x0.y, a0.x - a0.y, y1[0].y);
          const float2 hm = make_float2(a[pad(M / 2)].x, -a[pad(M / 2)].y);
          y2[0] = cfma(y2[0], Xp[M / 2], hm);
          continue;
        }
        if (u % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // two pairs in flight
        const float2 zk = a[pad(k)], am = a[pad(M - k)], zm = make_float2(am.x, -am.y);  // conj Z[M-k]
        const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y + zm.y));
        const float2 d = csub(zk, zm);
        const float2 w = root(T, split_offset<M>(), k), od = make_float2(0.5f * d.y, -0.5f * d.x);  // W^k, d / (2i)
        const float2 hk = cfma(e, w, od), hc = cfma(e, w, cneg(od));  // H[k], conj H[M-k]
        y1[u] = cfma(y1[u], at32(Xp, k), hk);
        y2[u] = cfma(y2[u], at32(Xp, M - k), make_float2(hc.x, -hc.y));
      }
    }
    __syncthreads();  // a is used up
  }
  // packed sequence of the block's spectrum (real_merge, both bins of a pair)
  const int tid = tid0;
#pragma unroll
  for (int u = 0; u < PAIRS; ++u) {
    const int k = tid + u * TPF;
    if (k == 0) {
      a[0] = make_float2(0.5f * (y1[0].x + y1[0].y), 0.5f * (y1[0].x - y1[0].y));
      a[pad(M / 2)] = make_float2(y2[0].x, -y2[0].y);
      continue;
    }
    const float2 ym = make_float2(y2[u].x, -y2[u].y);  // conj Y[M-k]
    const float2 e = make_float2(0.5f * (y1[u].x + ym.x), 0.5f * (y1[u].y + ym.y));
    const float2 d = csub(y1[u], ym);
    const float2 tk = root(T, split_offset<M>(), k);
    const float2 id = make_float2(-0.5f * d.y, 0.5f * d.x), w = make_float2(tk.x, -tk.y);  // i d / 2
    const float2 zk = cfma(e, id, w), zm = cfma(e, cneg(id), w);
    a[pad(k)] = zk;
    a[pad(M - k)] = make_float2(zm.x, -zm.y);
  }
  __syncthreads();
  fft.template run<true>([&](int n) { return a[pad(n)]; }, a, tid, T, true);
  if (live) {
    constexpr float inv_m = 1.0f / (float)M;
    float2 *o = reinterpret_cast<float2 *>(z + (size_t)row * 2 * M);
    const int keep = ((c + 1) * L + 1) / 2;
    for (int n = tid; n < min(M, keep); n += TPF) o[n] = make_float2(a[pad(n)].x * inv_m, a[pad(n)].y * inv_m);
  }
}

// y[m][n]: sum of z over the blocks that cover n, block by block, group by group; eight
// reads in flight (one after the other the up to (c + 1) S of them made this launch as
// long as the transforms of a short signal).
// CONTAIN (calls that take segment blocks in place of the direct sum): a sample or tap that
// is not finite makes every output of the blocks it enters so, in a transform; the outputs
// that come out infinite or NaN are therefore summed directly, each by its wave, so that
// only those that use such a value keep it (and sums that overflow in a transform alone
// are finite again). Nothing but a test of the value otherwise.
template <bool CONTAIN>
__global__ __launch_bounds__(256) void seg_overlap_kernel(const float *__restrict__ z, int N, int L, int c, int S,
                                                          int n_blk, float *__restrict__ y, int n_y,
                                                          const float *__restrict__ x, int n_x,
                                                          const float *__restrict__ rir, int n_mic, int n_rir) {
  const uint32_t at = blockIdx.x * 256u + threadIdx.x;
  const int m = blockIdx.y;
  const bool in = at < (uint32_t)n_y;
  if (!CONTAIN && !in) return;
  const int n = in ? (int)at : n_y - 1;  // (lanes past the end repeat the last output)
  const int top = n / L, hi = min(top, n_blk - 1);
  // block top - c ends one sample before the next multiple of L
  const int lo = max(0, top - c + (n - top * L == L - 1 ? 1 : 0));
  const float *zb = z + ((size_t)m * n_blk + lo) * S * N + (n - lo * L);
  int left = (hi - lo + 1) * S, g = 0;
  float v = 0.0f;
  while (left > 0) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      t[u] = 0.0f;
      if (u < left) {
        t[u] = *zb;
        zb += N;
        if (++g == S) {  // next block
          g = 0;
          zb -= L;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < left) v += t[u];
    left -= 8;
  }
  if constexpr (CONTAIN) {
    const int lane = threadIdx.x & 63;
    uint64_t bad = __ballot(in && !(__builtin_fabsf(v) <= 3.402823466e38f));
    while (bad) {
      const int l = __builtin_ctzll(bad);
      bad &= bad - 1;
      const int nn = __builtin_amdgcn_readlane(n, l);
      // taps whose sample nn - k is in the signal
      const int k1 = min(n_rir - 1, nn);
      float s = 0.0f;
      for (int k = max(0, nn - (n_x - 1)) + lane; k <= k1; k += 64) {
        const int i = nn - k;
        s = __builtin_fmaf(x[i], rir[((size_t)(i / L) * n_mic + m) * n_rir + k], s);
      }
#pragma unroll
      for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
      if (lane == l) v = s;
    }
  }
  if (in) y[(size_t)m * n_y + n] = v;
}

static size_t fft_align(size_t v) { return (v + 255) & ~(size_t)255; }

// A transform of 16384 points takes a workgroup 15 us where one of 8192 takes 11, so few
// of them end later than the work they save: from 128 RIR partitions on (1 microphone, 20
// segments of 8000 samples, RIRs of 24000 taps, 60 partitions: 33.5 us, fixed blocks
// 28.5; 8 microphones, 480: 56.4 and 61.6; 8 microphones, 8000 taps, 160: 39.5 and 46.3).
constexpr int64_t kSegLongRows = 128;

// Segment-block plan: transform size N (512 .. 16384, least work), partitions of
// c L taps, groups of partitions so that the launch holds up to 512 workgroups, two per
// CU, in one round (8 microphones, 100 segments of 1600, RIRs of 8000 taps: 47.6 us; up to
// 1024 57.4, up to 2048 63.4).
// False when a segment is longer than half the longest transform or the sizes leave
// a grid.
bool seg_plan(int n_x, int n_pos, int n_mic, int n_rir, FftPlan &f) {
  f.L = (n_x + n_pos - 1) / n_pos;
  const int n_seg = (n_x + f.L - 1) / f.L;
  double best = 0.0;
  f.N = 0;
  for (int N = 512; N <= 16384; N <<= 1) {
    const int64_t c = ((int64_t)N + 1) / f.L - 1;
    if (c < 1) continue;
    // a partition is at most the RIR long
    const int64_t cc = std::min<int64_t>(c, (n_rir + f.L - 1) / f.L);
    const int64_t P = (n_rir + cc * f.L - 1) / (cc * f.L), blk = n_seg + cc * (P - 1);
    if (N == 16384 && (int64_t)n_mic * n_seg * P < kSegLongRows) continue;
    const double work = (double)N * (std::log2((double)N) + 6.0) * ((double)n_seg * P + (double)blk);
    if (f.N == 0 || work < best) {
      best = work;
      f.N = N;
      f.c = (int)cc;
      f.P = (int)P;
      f.n_out_blocks = (int)blk;
    }
  }
  if (f.N == 0) return false;
  f.B = f.N / 2;
  f.n_in_blocks = n_seg;
  const int fpb = f.B < 4096 ? 4096 / f.B : 1;
  const int64_t rows = (int64_t)n_mic * f.n_out_blocks;
  // an output block meets at most ceil(n_seg / c) partitions: groups of those where that is
  // fewer (3 segments of 101 samples, 8 microphones, RIRs of 20 879 taps: 52 partitions, one
  // per block; 54 us with groups of all of them, most of it transforms of nothing)
  const int met = (n_seg + f.c - 1) / f.c;
  f.window = met < f.P;
  const int K = f.window ? met : f.P;
  f.S = (int)std::min<int64_t>(K, std::max<int64_t>(1, 512 * fpb / std::max<int64_t>(rows, 1)));
  f.PS = (K + f.S - 1) / f.S;
  f.S = (K + f.PS - 1) / f.PS;
  if (rows * f.S > 0x7fffff00LL) return false;
  size_t o = 0;
  f.off_X = o;
  o = fft_align(o + sizeof(float2) * (size_t)n_seg * f.B);
  f.off_z = o;
  f.bytes = fft_align(o + sizeof(float) * (size_t)(rows * f.S) * f.N);
  return true;
}

template <int M>
static int launch_seg_m(const float *x, int n_x, const float *rir, int n_mic, int n_rir, float *y, const FftPlan &f,
                        bool contain, char *w, hipStream_t st) {
  typedef FftShape<M> Sh;
  float2 *X = (float2 *)(w + f.off_X);
  float *z = (float *)(w + f.off_z);
  const int n_seg = f.n_in_blocks, rows = n_mic * f.n_out_blocks * f.S;
  hipLaunchKernelGGL(seg_input_kernel<M>, dim3((n_seg + Sh::FPB - 1) / Sh::FPB), dim3(Sh::NT), 0, st, x, n_x, f.L,
                     n_seg, X);
  hipLaunchKernelGGL(seg_filter_kernel<M>, dim3((rows + Sh::FPB - 1) / Sh::FPB), dim3(Sh::NT), 0, st, rir, n_mic,
                     n_rir, X, n_seg, f.L, f.c, f.P, f.S, f.PS, f.window, f.n_out_blocks, rows, z);
  const int n_y = n_x + n_rir - 1;
  auto *const overlap = contain ? &seg_overlap_kernel<true> : &seg_overlap_kernel<false>;
  hipLaunchKernelGGL(overlap, dim3((n_y + 255) / 256, n_mic), dim3(256), 0, st, z, f.N, f.L, f.c, f.S,
                     f.n_out_blocks, y, n_y, x, n_x, rir, n_mic, n_rir);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Block size: B = 4096 for RIRs of 16384 taps and more, else a quarter of
// the next power of two of n_rir (at least 256). R: pieces per input block.
// Returns false when the pieces per block exceed max_pieces.
bool fft_plan(int n_x, int n_pos, int n_mic, int n_rir, int max_pieces, FftPlan &f) {
  f.c = 0;
  f.window = false;
  int np2 = 1;
  while (np2 < n_rir) np2 <<= 1;
  f.B = np2 >= 16384 ? 4096 : (np2 / 4 < 256 ? 256 : np2 / 4);
  f.N = 2 * f.B;
  f.P = (n_rir + f.B - 1) / f.B;
  f.L = (n_x + n_pos - 1) / n_pos;
  f.R = (f.B + f.L - 1) / f.L + 1;  // segments one block can touch
  if (f.R > n_pos) f.R = n_pos;
  if (f.R > max_pieces) return false;
  f.n_in_blocks = (n_x + f.B - 1) / f.B;
  const int64_t n_y = (int64_t)n_x + n_rir - 1;
  if ((n_y + f.B - 1) / f.B > 65535) return false;  // one grid dimension per output block
  f.n_out_blocks = (int)((n_y + f.B - 1) / f.B);
  size_t o = 0;
  f.off_H = o;
  o = fft_align(o + sizeof(float2) * (size_t)n_pos * n_mic * f.P * f.B);
  f.off_X = o;
  o = fft_align(o + sizeof(float2) * (size_t)f.n_in_blocks * f.R * f.B);
  f.off_Y = o;
  o = fft_align(o + sizeof(float2) * (size_t)n_mic * f.n_out_blocks * f.B);
  f.off_z = o;
  o = fft_align(o + sizeof(float) * (size_t)n_mic * f.n_out_blocks * f.N);
  f.bytes = o;
  return true;
}

template <int M>
static int launch_fft_m(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, float *y,
                        const FftPlan &f, char *w, hipStream_t st) {
  constexpr int FPB = FftShape<M>::FPB;
  float2 *H = (float2 *)(w + f.off_H), *X = (float2 *)(w + f.off_X),
         *Y = (float2 *)(w + f.off_Y);
  float *z = (float *)(w + f.off_z);
  const int rir_rows = n_pos * n_mic * f.P, in_rows = f.n_in_blocks * f.R;
  const int rir_wgs = (rir_rows + FPB - 1) / FPB;
  hipLaunchKernelGGL(fft_parts_kernel<M>, dim3(rir_wgs + (in_rows + FPB - 1) / FPB), dim3(FftShape<M>::NT), 0, st,
                     rir, n_rir, f.P, rir_rows, rir_wgs, H, x, n_x, n_pos, f.L, f.R, in_rows, X);
  hipLaunchKernelGGL(spectrum_mac_kernel, dim3(M / 256, f.n_out_blocks, n_mic), dim3(256), 0, st, X, H, n_x, n_pos,
                     n_mic, f.L, f.B, M, f.P, f.R, f.n_in_blocks, Y);
  const int out_rows = n_mic * f.n_out_blocks;
  hipLaunchKernelGGL(ifft_block_kernel<M>, dim3((out_rows + FPB - 1) / FPB), dim3(FftShape<M>::NT), 0, st, Y, out_rows,
                     z);
  const int n_y = n_x + n_rir - 1;
  hipLaunchKernelGGL(overlap_add_kernel, dim3((n_y + 255) / 256, n_mic), dim3(256), 0, st, z, f.B, f.N,
                     f.n_out_blocks, y, n_y);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_filter_fft(const float *x, int n_x, const float *rir, int n_pos, int n_mic, int n_rir, float *y,
                      const FftPlan &f, bool contain, void *ws, hipStream_t st) {
  char *w = (char *)ws;
  if (f.c > 0) {  // segment blocks
    switch (f.B) {
      case 256: return launch_seg_m<256>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      case 512: return launch_seg_m<512>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      case 1024: return launch_seg_m<1024>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      case 2048: return launch_seg_m<2048>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      case 4096: return launch_seg_m<4096>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      case 8192: return launch_seg_m<8192>(x, n_x, rir, n_mic, n_rir, y, f, contain, w, st);
      default: return -1;
    }
  }
  switch (f.B) {  // M = B complex points per transform
    case 256: return launch_fft_m<256>(x, n_x, rir, n_pos, n_mic, n_rir, y, f, w, st);
    case 512: return launch_fft_m<512>(x, n_x, rir, n_pos, n_mic, n_rir, y, f, w, st);
    case 1024: return launch_fft_m<1024>(x, n_x, rir, n_pos, n_mic, n_rir, y, f, w, st);
    case 2048: return launch_fft_m<2048>(x, n_x, rir, n_pos, n_mic, n_rir, y, f, w, st);
    case 4096: return launch_fft_m<4096>(x, n_x, rir, n_pos, n_mic, n_rir, y, f, w, st);
    default: return -1;
  }
}

}  // namespace ism
