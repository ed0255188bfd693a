// Plain initialisation and optimisation metrics.
//
// Ram-Lak filtering: the paper's Radon baseline filters each parallel-beam
// sinogram with a Ram-Lak filter and clips negative values (Sec. 2.3).  Here
// the filter is applied along u as the exact spatial-domain convolution with
// the band-limited ramp kernel sampled at the pixel pitch (Ramachandran and
// Lakshminarayanan; see Kak and Slaney, "Principles of Computerized
// Tomographic Imaging", ch. 3):
//   h[0] = 1 / (4 tau^2),  h[n] = 0 for even n != 0,
//   h[n] = -1 / (n^2 pi^2 tau^2) for odd n,
// scaled by tau so that a unit-pitch discrete convolution approximates the
// continuous filter, followed by clipping at zero.
//
// Export: see k_eq_map below.
//
// Dose error: the termination test of Sec. 2.7 compares simulated and target
// dose; here E = ||sigmoid(kappa (d - thr)) - t||_1 / ||t||_1 together with
// the fraction of voxels whose thresholded dose (d >= thr) differs from the
// binary target, both reduced in FP64.

#include <cmath>

#include "vam_internal.h"

namespace vam {

// out = in * h for 32 rows and 64 NB columns of them: a product of the rows with
// the banded (Toeplitz) matrix of h.  h is zero at even distances, so even
// columns take only odd ones and the other way round: with u = 2 a + e and
// u' = 2 b + 1 - e, out(u) = in(u) / 4 + sum_b T(a - b + e) in(u'), where
// T(d) = h[2 d - 1] (h is even).
//
// What bounds it: n_u / 2 multiplications a value, 6 GFLOP for 92160 rows of
// 256 (39 us at the rate of a large FP32 product; moving the rows takes 36 us).
// One thread an output read two values and a weight from LDS for each pair of
// taps, 660 us.  Here the FP32 matrix instructions multiply: a wave has 32 rows
// x 64 columns (even and odd), and per 8 products of 32 x 32 x 2 it reads two
// times four values and five weights a lane, a third of the LDS's time.
// 82 us; 12000 rows of 1024 133 us.
//
// Precision: the filter all but cancels the value itself and its neighbours,
// so a sum over ascending b carries large partial sums through most of its
// roundings (six times the error of adding pairs from the middle outwards).
// The kNear nearest pairs are therefore added apart, from the middle outwards,
// and the matrix instructions add the rest from both ends towards the middle.
// The error against FP64 is then that of adding pairs, or less, for rows of 64
// to 1000 values of noise, smooth bumps, boxes and waves.
//
// Infinities and NaN: the matrix instructions multiply the nearest values by
// zero, which makes NaN of an infinity that is added apart.  A sum that is not
// finite when they are done is therefore formed again, pair by pair; one that
// is finite had no such value at any odd distance.
//
// Columns go in groups of 512 (above that NB is 8 and blockIdx.y is the group)
// and so does the sum over u', its own group last.  Rows in LDS are K + 12
// floats apart, so 16 rows read at 16 bytes a lane cover all 64 banks.
constexpr int kRampRows = 32, kRampMax = 8, kNear = 4;
__device__ inline constexpr float ramp_weight(int m) {
  const float n = (float)(2 * m + 1);
  return -1.0f / ((float)(M_PI * M_PI) * n * n);
}
// One output of a row, adding pairs from the middle outwards.
__device__ inline float ramp_pairs(const float* __restrict__ row, int u, int nu) {
  float acc = 0.25f * row[u];
  for (int m = 0; 2 * m + 1 < nu; ++m) {
    const int l = u - (2 * m + 1), r = u + 2 * m + 1;
    acc = fmaf(ramp_weight(m), (l >= 0 ? row[l] : 0.0f) + (r < nu ? row[r] : 0.0f), acc);
  }
  return acc;
}

template <int NB>
__global__ __launch_bounds__(64 * NB) void k_ramlak(const float* __restrict__ in, float* __restrict__ out, int n_rows,
                                                    int nu, float tau, int clip) {
  typedef float f32x16 __attribute__((ext_vector_type(16)));
  constexpr int K = 32 * NB, P = K + 12;  // columns of one parity in a group; row pitch
  // columns of one parity of a group with four more on each side (the last 32
  // floats put a wave's even and odd columns into different banks)
  __shared__ __attribute__((aligned(16))) float x[2][kRampRows * P + 32];
  __shared__ float ramp[2 * K];  // T(i - (K - 1) + (group - c) K), zero for the nearest
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int r0 = blockIdx.x * kRampRows, group = blockIdx.y, groups = gridDim.y;
  const bool any = 2 * K * group + 64 * wave < nu;
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.0f;
  for (int i = 0; i < groups; ++i) {
    const int c = i < group ? i : groups - 1 - (i - group), u0 = 2 * K * c;
    if (i) __syncthreads();
    // (the reads past the last row or column are of the last one)
#pragma unroll 4
    for (int r = wave; r < kRampRows; r += NB) {
      const float* src = in + (int64_t)min(r0 + r, n_rows - 1) * nu;
      float v[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k) v[k] = src[min(u0 + 64 * k + lane, nu - 1)];
#pragma unroll
      for (int k = 0; k < NB; ++k)
        x[lane & 1][r * P + 4 + 32 * k + (lane >> 1)] = u0 + 64 * k + lane < nu ? v[k] : 0.0f;
    }
    if (c == group)
      for (int e = threadIdx.x; e < 16 * kRampRows; e += 64 * NB) {
        const int r = e >> 4, at = (e & 15) < 8 ? (e & 15) : 2 * K + (e & 15), u = u0 - 8 + at;
        x[at & 1][r * P + (at >> 1)] = u >= 0 && u < nu ? in[(int64_t)min(r0 + r, n_rows - 1) * nu + u] : 0.0f;
      }
    for (int e = threadIdx.x; e < 2 * K; e += 64 * NB) {
      const int d = e - (K - 1) + (group - c) * K, m = d > 0 ? d - 1 : -d;
      ramp[e] = m < kNear ? 0.0f : ramp_weight(m);
    }
    __syncthreads();
    if (!any) continue;
    const float *xe = x[0] + col * P + 4 + 4 * half, *xo = x[1] + col * P + 4 + 4 * half;
    const float* t = ramp + 32 * wave + col - 4 * half + K - 1;
    // 8 columns at a time, of the two ends left the one further from the wave's 32
    const int middle = 2 * (32 * wave + (group - c) * K + 12);
    for (int lo = 0, hi = (min(K, (nu + 1) / 2 - K * c) - 1) & ~7; lo <= hi;) {
      const bool left = middle >= lo + hi;
      const int b = left ? lo : hi;
      lo += left ? 8 : 0;
      hi -= left ? 0 : 8;
      const float4 o = *(const float4*)(xo + b), e = *(const float4*)(xe + b);
      const float vo[4] = {o.x, o.y, o.z, o.w}, ve[4] = {e.x, e.y, e.z, e.w};
      float w[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) w[j] = t[1 - j - b];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vo[j], w[j + 1], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ve[j], w[j], acc[1], 0, 0, 0);
      }
    }
  }
  if (!any) return;
  const int u = 2 * (K * group + 32 * wave + col);
  float not_finite[4] = {};  // NaN if one of the sums is not finite (four chains)
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = 8 * (i >> 2) + 4 * half + (i & 3);
    not_finite[i & 1] = fmaf(acc[0][i], 0.0f, not_finite[i & 1]);
    not_finite[2 + (i & 1)] = fmaf(acc[1][i], 0.0f, not_finite[2 + (i & 1)]);
    const float *e = x[0] + r * P + 4 + 32 * wave + col, *o = x[1] + r * P + 4 + 32 * wave + col;
    float v[2] = {0.25f * e[0], 0.25f * o[0]};
#pragma unroll
    for (int m = 0; m < kNear; ++m) {
      v[0] = fmaf(ramp_weight(m), o[-1 - m] + o[m], v[0]);
      v[1] = fmaf(ramp_weight(m), e[-m] + e[1 + m], v[1]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      v[k] = (v[k] + acc[k][i]) / tau;
      if (clip) v[k] = fmaxf(v[k], 0.0f);
    }
    if (r0 + r >= n_rows) continue;
    float* to = out + (int64_t)(r0 + r) * nu + u;
    if (u + 1 < nu)
      __builtin_memcpy(to, v, 8);
    else if (u < nu)
      *to = v[0];
  }
  if (not_finite[0] + not_finite[1] + not_finite[2] + not_finite[3] == 0.0f) return;
  unsigned again = 0u;
#pragma unroll
  for (int i = 0; i < 32; ++i) again |= acc[i & 1][i >> 1] * 0.0f == 0.0f ? 0u : 1u << i;
  for (; again != 0u; again &= again - 1u) {
    const int i = __ffs(again) - 1, r = r0 + 8 * (i >> 3) + 4 * half + (i >> 1 & 3), at = u + (i & 1);
    if (r >= n_rows || at >= nu) continue;
    const float v = ramp_pairs(in + (int64_t)r * nu, at, nu) / tau;
    out[(int64_t)r * nu + at] = clip ? fmaxf(v, 0.0f) : v;
  }
}

// (NB of the narrowest kernel that has all columns, or the widest)
template <int NB>
void launch_ramlak(const float* in, float* out, int n_rows, int nu, float tau, int clip, hipStream_t s) {
  if constexpr (NB < kRampMax)
    if (64 * NB < nu) return launch_ramlak<NB + 1>(in, out, n_rows, nu, tau, clip, s);
  hipLaunchKernelGGL((k_ramlak<NB>), dim3((n_rows + kRampRows - 1) / kRampRows, (nu + 64 * NB - 1) / (64 * NB)),
                     dim3(64 * NB), 0, s, in, out, n_rows, nu, tau, clip);
}

// The whole-array kernels below take four values a lane and load (any
// alignment: an unaligned 16-byte load costs no more than the lines it
// touches), kAhead loads ahead of the arithmetic; the last n % 4 values go one a
// lane in the first workgroup.  (One value a lane and load: dose error of 256^3
// 40 us, export statistics of 360 x 256^2 31, its bytes 39; so 35, 17 and 21.
// The arrays take 26, 18 and 23 at the rate of a large copy, which the last two
// beat where the projections are still in the last cache; the dose error's FP64
// exponential and division take about as long as its loads.)
constexpr int kAhead = 4;
template <class F4, class F1>
__device__ inline void for_quads(int64_t n, F4 quads, F1 one) {
  const int64_t n4 = n / 4, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += kAhead * stride) quads(i, stride, n4);
  if (blockIdx.x == 0 && (int64_t)threadIdx.x < n - 4 * n4) one(4 * n4 + threadIdx.x);
}
// Values 4 i .. 4 i + 3 of p, and of the quads i + stride, ... (k < kAhead) that exist.
__device__ inline void load_quads(const float* p, int64_t i, int64_t stride, int64_t n4, float (&v)[kAhead][4]) {
#pragma unroll
  for (int k = 0; k < kAhead; ++k) __builtin_memcpy(v[k], p + 4 * min(i + k * stride, n4 - 1), 16);
}

constexpr int kErrThreads = 256;
constexpr int kErrBlocks = 1024;

__global__ __launch_bounds__(kErrThreads) void k_dose_error(const float* __restrict__ dose,
                                                            const float* __restrict__ target, int64_t n, float thr,
                                                            float kappa, double* __restrict__ part) {
  __shared__ double red[3][kErrThreads / 64];
  double l1 = 0.0, tsum = 0.0, wrong = 0.0;
  auto add = [&](double d, double t) {
    const double sig = 1.0 / (1.0 + exp(-(double)kappa * (d - thr)));
    l1 += fabs(sig - t);
    tsum += fabs(t);
    wrong += ((d >= thr) != (t >= 0.5)) ? 1.0 : 0.0;
  };
  for_quads(
      n,
      [&](int64_t i, int64_t stride, int64_t n4) {
        float d[kAhead][4], t[kAhead][4];
        load_quads(dose, i, stride, n4, d);
        load_quads(target, i, stride, n4, t);
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
          if (i + k * stride < n4)
#pragma unroll
            for (int j = 0; j < 4; ++j) add(d[k][j], t[k][j]);
      },
      [&](int64_t i) { add(dose[i], target[i]); });
  for (int off = 32; off > 0; off >>= 1) {
    l1 += __shfl_down(l1, off, 64);
    tsum += __shfl_down(tsum, off, 64);
    wrong += __shfl_down(wrong, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = l1;
    red[1][threadIdx.x >> 6] = tsum;
    red[2][threadIdx.x >> 6] = wrong;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0.0;
    for (int w = 0; w < kErrThreads / 64; ++w) s += red[threadIdx.x][w];
    part[3 * blockIdx.x + threadIdx.x] = s;
  }
}

// The block sums in a fixed order by one workgroup (a single thread walking
// the 1024 x 3 sums took 122 us of waiting for loads, this 5 us).
__global__ __launch_bounds__(kSumThreads) void k_dose_error_final(const double* __restrict__ part, int nblocks,
                                                                  int64_t n, double* __restrict__ out) {
  double s[3];
  block_sum_rows<3>(part, nblocks, s);
  if (threadIdx.x == 0) {
    out[0] = s[1] > 0.0 ? s[0] / s[1] : 0.0;
    out[1] = s[2] / (double)n;
  }
}

// Projection export (Sec. 2.7): values above mean + 3 std over all pixels of
// all angles are clipped, then the range [0, clip] is rescaled to 8 bits.
// Statistics in FP64; the scaled value v = x * (255 / clip) is formed in FP64
// and rounded to nearest even.
constexpr int kEqThreads = 256;
constexpr int kEqBlocks = 1024;
constexpr int kMapBlocks = 2048;  // a whole CU's waves on every CU

__global__ __launch_bounds__(kEqThreads) void k_eq_stats(const float* __restrict__ p, int64_t n,
                                                         double* __restrict__ part) {
  __shared__ double red[2][kEqThreads / 64];
  double s1 = 0.0, s2 = 0.0;
  auto add = [&](double x) {
    s1 += x;
    s2 += x * x;
  };
  for_quads(
      n,
      [&](int64_t i, int64_t stride, int64_t n4) {
        float v[kAhead][4];
        load_quads(p, i, stride, n4, v);
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
          if (i + k * stride < n4)
#pragma unroll
            for (int j = 0; j < 4; ++j) add(v[k][j]);
      },
      [&](int64_t i) { add(p[i]); });
  for (int off = 32; off > 0; off >>= 1) {
    s1 += __shfl_down(s1, off, 64);
    s2 += __shfl_down(s2, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s1;
    red[1][threadIdx.x >> 6] = s2;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double s = 0.0;
    for (int w = 0; w < kEqThreads / 64; ++w) s += red[threadIdx.x][w];
    part[2 * blockIdx.x + threadIdx.x] = s;
  }
}

// stats[0] mean, stats[1] population std, stats[2] clip = mean + 3 std (one
// workgroup: 84 us on one thread, 5 us so)
__global__ __launch_bounds__(kSumThreads) void k_eq_final(const double* __restrict__ part, int nblocks, int64_t n,
                                                          double* __restrict__ stats) {
  double s[2];
  block_sum_rows<2>(part, nblocks, s);
  if (threadIdx.x == 0) {
    const double mean = s[0] / (double)n;
    const double var = fmax(s[1] / (double)n - mean * mean, 0.0);
    const double sd = sqrt(var);
    stats[0] = mean;
    stats[1] = sd;
    stats[2] = mean + 3.0 * sd;
  }
}

__global__ __launch_bounds__(kEqThreads) void k_eq_map(const float* __restrict__ p, int64_t n,
                                                       const double* __restrict__ stats, uint8_t* __restrict__ out) {
  const double clip = stats[2], scale = 255.0 / clip;
  auto byte = [&](float x) {
    double v = 0.0;
    if (clip > 0.0) v = rint(fmin(fmax((double)x, 0.0), clip) * scale);
    return (uint8_t)fmin(fmax(v, 0.0), 255.0);
  };
  for_quads(
      n,
      [&](int64_t i, int64_t stride, int64_t n4) {
        float v[kAhead][4];
        load_quads(p, i, stride, n4, v);
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
          const int64_t q = i + k * stride;
          if (q >= n4) break;
          const uint8_t b[4] = {byte(v[k][0]), byte(v[k][1]), byte(v[k][2]), byte(v[k][3])};
          __builtin_memcpy(out + 4 * q, b, 4);
        }
      },
      [&](int64_t i) { out[i] = byte(p[i]); });
}

}  // namespace vam

using namespace vam;

extern "C" {

vam_status vam_ramlak_filter(const float* proj_in, float* proj_out, int32_t n_rows, int32_t n_u, double pitch,
                             int32_t clip_negative, hipStream_t stream) {
  clear_error();
  if (!proj_in || !proj_out) return fail(VAM_ERR_INVALID_ARG, "NULL buffer");
  if (n_rows < 0 || n_u < 1 || n_u > 8192) return fail(VAM_ERR_INVALID_ARG, "bad sizes %d x %d", n_rows, n_u);
  if (!(pitch > 0) || !std::isfinite(pitch)) return fail(VAM_ERR_INVALID_ARG, "pitch must be finite and > 0");
  if (proj_in == proj_out) return fail(VAM_ERR_INVALID_ARG, "in-place filtering is not supported");
  if (n_rows == 0) return VAM_OK;
  launch_ramlak<1>(proj_in, proj_out, n_rows, n_u, (float)pitch, clip_negative, stream);
  VAM_HIP_TRY(hipGetLastError(), "launching the Ram-Lak filter");
  return VAM_OK;
}

vam_status vam_dose_error(const float* dose, const float* target, int64_t n, double threshold, double sharpness,
                          double* out2, hipStream_t stream) {
  clear_error();
  if (!dose || !target || !out2) return fail(VAM_ERR_INVALID_ARG, "NULL argument");
  if (n < 1) return fail(VAM_ERR_INVALID_ARG, "n must be >= 1");
  if (!(sharpness > 0) || !std::isfinite(sharpness) || !std::isfinite(threshold))
    return fail(VAM_ERR_INVALID_ARG, "sharpness must be finite and > 0");
  double* part = nullptr;
  const int blocks = (int)std::min<int64_t>(kErrBlocks, (n + kErrThreads - 1) / kErrThreads);
  VAM_HIP_TRY(hipMallocAsync((void**)&part, (3 * blocks + 2) * sizeof(double), stream), "allocating partials");
  hipLaunchKernelGGL(k_dose_error, dim3(blocks), dim3(kErrThreads), 0, stream, dose, target, n, (float)threshold,
                     (float)sharpness, part);
  hipLaunchKernelGGL(k_dose_error_final, dim3(1), dim3(kSumThreads), 0, stream, part, blocks, n, part + 3 * blocks);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = hipMemcpyAsync(out2, part + 3 * blocks, 2 * sizeof(double), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  (void)hipFreeAsync(part, stream);
  if (e != hipSuccess) return hip_check(e, "dose error");
  return VAM_OK;
}

vam_status vam_equalize_u8(const float* proj, int64_t n, uint8_t* out, double* stats3, hipStream_t stream) {
  clear_error();
  if (!proj || !out) return fail(VAM_ERR_INVALID_ARG, "NULL buffer");
  if (n < 1) return fail(VAM_ERR_INVALID_ARG, "n must be >= 1");
  double* part = nullptr;
  const int blocks = (int)std::min<int64_t>(kEqBlocks, (n + kEqThreads - 1) / kEqThreads);
  VAM_HIP_TRY(hipMallocAsync((void**)&part, (2 * blocks + 3) * sizeof(double), stream), "allocating partials");
  double* st = part + 2 * blocks;
  const int map_blocks = (int)std::max<int64_t>(1, std::min<int64_t>(kMapBlocks, (n / 4 + kEqThreads - 1) / kEqThreads));
  hipLaunchKernelGGL(k_eq_stats, dim3(blocks), dim3(kEqThreads), 0, stream, proj, n, part);
  hipLaunchKernelGGL(k_eq_final, dim3(1), dim3(kSumThreads), 0, stream, part, blocks, n, st);
  hipLaunchKernelGGL(k_eq_map, dim3(map_blocks), dim3(kEqThreads), 0, stream, proj, n, st, out);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && stats3) e = hipMemcpyAsync(stats3, st, 3 * sizeof(double), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess && stats3) e = hipStreamSynchronize(stream);
  (void)hipFreeAsync(part, stream);
  if (e != hipSuccess) return hip_check(e, "equalisation");
  return VAM_OK;
}

}  // extern "C"
