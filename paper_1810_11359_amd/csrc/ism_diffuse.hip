// Diffuse reverberation tail (Sec. 2.2, Eq. (8); Sec. 3.3): after t_diff the
// RIR is logistic noise times the square root of an exponential power envelope,
//   P(t) = A 10^(-6 (t - t_diff) / T60)      (-60 dB of power in T60, Sabine),
// whose level A is estimated from the ISM part of the same RIR: the mean of
// h[k]^2 / 10^(-6 (t_k - t_diff) / T60) over the last fifth of the ISM part.
// The noise of sample k of RIR i is the unit-variance logistic variate of one
// 32-bit word of the Philox4x32-10 counter-based generator (Salmon et al.,
// SC'11) with counter (k / 4, i, 0, 0) and key (seed low, seed high), word
// k % 4: any sample can be drawn independently, so the tail is one pass of
// independent threads and a result does not depend on the launch shape.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace ism {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Philox4x32 with 10 rounds: a round maps (c0, c1, c2, c3) with key (k0, k1)
// to (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)); the key
// advances by two Weyl increments before every round but the first.
__device__ __forceinline__ u32x4 philox4x32_10(u32x4 c, uint32_t k0, uint32_t k1) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += W0;
      k1 += W1;
    }
    // both halves by one 64-bit multiplication (a quarter of the FP32 rate each)
    const uint64_t p0 = (uint64_t)M0 * c.x, p1 = (uint64_t)M1 * c.z;
    c = u32x4{(uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0};
  }
  return c;
}

// Unit-variance logistic variate of a word x: log(u / (1 - u)) sqrt(3)/pi at
// u = (x + 1/2) / 2^32, with u and 1 - u both formed from exact integers.
__device__ __forceinline__ float logistic_from_bits(uint32_t x) {
  const float a = (float)x + 0.5f;
  const float b = (float)(0xFFFFFFFFu - x) + 0.5f;
  constexpr float kScale = 0.69314718055994531f * 0.55132889542179204f;  // ln 2 * sqrt(3)/pi
  return (__log2f(a) - __log2f(b)) * kScale;
}

// 2^e for the envelope: its integer part apart, so that the rounding of e to FP32 is
// that of its fraction.
__device__ __forceinline__ float exp2_split(double e) {
  e = __builtin_fmin(__builtin_fmax(e, -1000.0), 1000.0);
  const double r = __builtin_rint(e);
  return __builtin_ldexpf(__builtin_amdgcn_exp2f((float)(e - r)), (int)r);
}

// Amplitude envelope sqrt(P / A) at sample k: 2^(slope (k - k0)).
struct Envelope {
  double slope, k0;
  float step[4];  // 2^(slope j)
};

// grid = n_rir x n_blk blocks (block b: RIR b / n_blk, its share of SEGS segments of
// 256 SPT samples); each block computes the level A of its RIR (a fixed-order sum over
// the window) and writes SPT consecutive samples per thread and segment: the ISM part
// copied for k < k_diff, the tail after it. Bounded by the random words and logarithms
// (about 50 instructions per sample) and by writing the RIRs; one exponential and no
// division or square root per SPT samples. 1024 RIRs of 11200 samples, ISM part 2427:
// 30.4 us with a segment per block, each with the level, a division, an exponential and
// a square root per sample; now 17.8 us.
constexpr int SPT = 4;
__global__ __launch_bounds__(256) void diffuse_kernel(const float *__restrict__ ism, int k_diff, int k_w,
                                                      float *__restrict__ out, int n_samples, int n_blk, int segs,
                                                      Envelope env, uint32_t key0, uint32_t key1) {
  const int rir = (int)(blockIdx.x / (unsigned)n_blk);
  const int64_t first = (int64_t)(blockIdx.x % (unsigned)n_blk) * segs * (256 * SPT);
  const float *h = ism + (size_t)rir * k_diff;
  __shared__ float red[4];
  float acc = 0.0f;
  for (int k = k_w + (int)threadIdx.x; k < k_diff; k += 256) {
    const float v = h[k];
    acc += v * v * exp2_split(-2.0 * env.slope * ((double)k - env.k0));
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) acc += __shfl_down(acc, s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  const float level = sqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)(k_diff - k_w));
  float *o = out + (size_t)rir * n_samples;
  for (int s = 0; s < segs; ++s) {
    const int64_t at = first + ((int64_t)s * 256 + threadIdx.x) * SPT;  // one Philox block
    if (at >= n_samples) return;
    const int k0 = (int)at;
    float v[SPT];
    if (k0 + SPT > k_diff) {
      const u32x4 bits = philox4x32_10(u32x4{(uint32_t)(k0 / 4), (uint32_t)rir, 0u, 0u}, key0, key1);
      if (k0 >= k_diff) {
        const float amp = level * exp2_split(env.slope * ((double)k0 - env.k0));
#pragma unroll
        for (int j = 0; j < SPT; ++j) v[j] = logistic_from_bits(bits[j]) * (amp * env.step[j]);
      } else {
        // the tail begins inside: before it the envelope is above the level, and for T60
        // of a fraction of a sample beyond FP32
#pragma unroll
        for (int j = 0; j < SPT; ++j)
          v[j] = logistic_from_bits(bits[j]) * (level * exp2_split(env.slope * ((double)max(k0 + j, k_diff) - env.k0)));
      }
    }
#pragma unroll
    for (int j = 0; j < SPT; ++j)
      if (k0 + j < k_diff) v[j] = h[k0 + j];
    if (k0 + SPT <= n_samples && ((uintptr_t)(o + k0) & 15) == 0) {
      *reinterpret_cast<float4 *>(o + k0) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int j = 0; j < SPT; ++j)
        if (k0 + j < n_samples) o[k0 + j] = v[j];
    }
  }
}

int launch_diffuse(const float *ism, int k_diff, float *out, int n_samples, int n_rir, double fs, double t_diff,
                   double t60, uint64_t seed, hipStream_t st) {
  const int k_w = k_diff - (k_diff / 5 > 1 ? k_diff / 5 : 1);
  const int n_seg = (int)(((int64_t)n_samples + 256 * SPT - 1) / (256 * SPT));
  // segments per block: one level per block, as long as 2048 blocks fill the chip
  const int segs = (int)std::max<int64_t>(1, std::min<int64_t>(n_seg, (int64_t)n_seg * n_rir / 2048));
  const int n_blk = (n_seg + segs - 1) / segs;
  const uint64_t blocks = (uint64_t)n_blk * (uint64_t)n_rir;
  if (blocks == 0 || (uint64_t)n_seg * (uint64_t)n_rir > 0x7fffffffu) return -1;
  Envelope env;
  env.slope = -3.0 * 3.32192809488736235 / (t60 * fs);  // log2 of the amplitude per sample
  env.k0 = t_diff * fs;
  for (int j = 0; j < SPT; ++j) env.step[j] = (float)std::exp2(env.slope * j);
  hipLaunchKernelGGL(diffuse_kernel, dim3((unsigned)blocks), dim3(256), 0, st, ism, k_diff, k_w, out, n_samples,
                     n_blk, segs, env, (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32));
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ism
