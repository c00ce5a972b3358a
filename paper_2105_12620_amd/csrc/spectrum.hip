// Radially averaged power spectrum of the error tile (the |FFT(e)|^2 insets
// of Fig. 1b), as a diagnostic beside the blur criterion of Sec. 3.3.  A
// direct separable DFT over the W x H torus, chunks of 64 integrand rows:
// first along x, then along y with |.|^2 summed over a chunk's integrands per
// frequency (u, v) and over the chunks in order.  FP32 twiddles and sums within
// a row or column, FP64 across integrands.
//
// A lane owns one integrand and 8 consecutive frequencies, so that a value is
// loaded once for 8 of them; their twiddles, uniform over the wave, come from a
// matrix [position][frequency] through the scalar cache, 8 in one load.
// Several chunks go in one launch, as many as give about 16384 waves.  Bound by
// the vector ALUs and the scalar loads.  At 128^2 and 1024 integrands 180 us
// along x and 296 along y for all 16 chunks; 1430 and 2090 with one frequency
// a lane, its twiddle gathered, and a launch per chunk.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

constexpr uint32_t SPEC_CHUNK = 64;
constexpr int F = 8;   // frequencies of a lane

#define BN_UNIFORM __attribute__((address_space(4)))
// cos and -sin of F frequencies at one position
typedef float Twiddles __attribute__((ext_vector_type(2 * F), aligned(8)));
static_assert(F == 8, "the twiddles of a lane are one vector");

inline uint32_t padded(uint32_t n) { return (n + F - 1) / F * F; }

// mat[x][u] = tw[u x mod n], u < padded(n).
__global__ __launch_bounds__(256) void k_twiddles(const float2* __restrict__ tw, uint32_t n, uint32_t np,
                                                  float2* __restrict__ mat) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * np) return;
  const uint32_t x = i / np, u = i - x * np;
  mat[i] = tw[(uint32_t)(((uint64_t)u * x) % n)];
}

// rows[c][y][u][64] of chunk c, integrands t0 + 64 c ..
__global__ __launch_bounds__(256) void k_dft_x(const float* __restrict__ field, uint32_t pitch, uint32_t valid,
                                               uint32_t t0, uint32_t chunks, uint32_t w, uint32_t h,
                                               const float2* __restrict__ mat, float2* __restrict__ rows) {
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t np = (w + F - 1) / F * F, nb = np / F;
  const uint32_t ub = wave % nb, rest = wave / nb, y = rest % h, c = rest / h;
  if (c >= chunks) return;
  const uint32_t t = t0 + c * SPEC_CHUNK;
  const float* row = field + (size_t)y * w * pitch + t;
  const BN_UNIFORM float* m = (const BN_UNIFORM float*)(mat + ub * F);
  float re[F], im[F];
#pragma unroll
  for (int f = 0; f < F; ++f) re[f] = im[f] = 0.0f;
  if (t + lane < valid) {
#pragma unroll 4
    for (uint32_t x = 0; x < w; ++x) {
      const float e = (row + (size_t)x * pitch)[lane];
      const Twiddles q = *(const BN_UNIFORM Twiddles*)(m + (size_t)x * 2 * np);
#pragma unroll
      for (int f = 0; f < F; ++f) {
        re[f] = fmaf(e, q[2 * f], re[f]);
        im[f] = fmaf(e, q[2 * f + 1], im[f]);
      }
    }
  }
  float2* o = rows + (((size_t)c * h + y) * w + ub * F) * SPEC_CHUNK;
#pragma unroll
  for (int f = 0; f < F; ++f)
    if (ub * F + f < w) (o + f * SPEC_CHUNK)[lane] = make_float2(re[f], im[f]);
}

// power[c][v][u] of chunk c; one wave per u and F values of v.
__global__ __launch_bounds__(256) void k_dft_y_power(const float2* __restrict__ rows, uint32_t chunks, uint32_t w,
                                                     uint32_t h, const float2* __restrict__ mat,
                                                     double* __restrict__ power) {
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t np = (h + F - 1) / F * F, nb = np / F;
  const uint32_t vb = wave % nb, rest = wave / nb, u = rest % w, c = rest / w;
  if (c >= chunks) return;
  const float2* col = rows + ((size_t)c * h * w + u) * SPEC_CHUNK;
  const BN_UNIFORM float* m = (const BN_UNIFORM float*)(mat + vb * F);
  float re[F], im[F];
#pragma unroll
  for (int f = 0; f < F; ++f) re[f] = im[f] = 0.0f;
#pragma unroll 4
  for (uint32_t y = 0; y < h; ++y) {
    const float2 a = (col + (size_t)y * w * SPEC_CHUNK)[lane];
    const Twiddles q = *(const BN_UNIFORM Twiddles*)(m + (size_t)y * 2 * np);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      re[f] = fmaf(a.x, q[2 * f], fmaf(-a.y, q[2 * f + 1], re[f]));
      im[f] = fmaf(a.x, q[2 * f + 1], fmaf(a.y, q[2 * f], im[f]));
    }
  }
#pragma unroll
  for (int f = 0; f < F; ++f) {
    double pw = (double)re[f] * re[f] + (double)im[f] * im[f];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) pw += __shfl_xor(pw, off);
    if (lane == 0 && vb * F + f < h) power[((size_t)c * h + vb * F + f) * w + u] = pw;
  }
}

// sum += the chunks' powers, in order.
__global__ __launch_bounds__(256) void k_power_sum(const double* __restrict__ power, uint32_t chunks, uint32_t n,
                                                   double* __restrict__ sum) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = sum[i];
  for (uint32_t c = 0; c < chunks; ++c) s += power[(size_t)c * n + i];
  sum[i] = s;
}

}  // namespace

uint32_t spectrum_chunk() { return SPEC_CHUNK; }

uint32_t spectrum_chunks(const DevView& v, uint32_t rows) {
  const uint64_t waves = std::min((uint64_t)v.h * padded(v.w), (uint64_t)v.w * padded(v.h)) / F;
  const uint64_t want = std::max<uint64_t>(1, (16384 + waves - 1) / waves);
  return (uint32_t)std::min<uint64_t>(want, std::max(1u, (rows + SPEC_CHUNK - 1) / SPEC_CHUNK));
}

SpectrumScratch spectrum_scratch(const DevView& v, uint32_t chunks) {
  const size_t n = (size_t)v.w * v.h;
  return {n * SPEC_CHUNK * chunks, n * chunks, (size_t)v.w * padded(v.w), (size_t)v.h * padded(v.h)};
}

hipError_t launch_twiddles(const float2* tw, uint32_t n, float2* mat, hipStream_t s) {
  const uint32_t np = padded(n);
  hipLaunchKernelGGL(k_twiddles, dim3((n * np + 255) / 256), dim3(256), 0, s, tw, n, np, mat);
  return hipGetLastError();
}

hipError_t launch_spectrum_chunks(const DevView& v, const float* field, uint32_t pitch, uint32_t valid, uint32_t t0,
                                  uint32_t chunks, const float2* matx, const float2* maty, float2* rows, double* power,
                                  double* sum, hipStream_t s) {
  const uint64_t wx = (uint64_t)chunks * v.h * (padded(v.w) / F), wy = (uint64_t)chunks * v.w * (padded(v.h) / F);
  hipLaunchKernelGGL(k_dft_x, dim3((unsigned)((wx + 3) / 4)), dim3(256), 0, s, field, pitch, valid, t0, chunks, v.w,
                     v.h, matx, rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dft_y_power, dim3((unsigned)((wy + 3) / 4)), dim3(256), 0, s, (const float2*)rows, chunks, v.w,
                     v.h, maty, power);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const uint32_t n = v.w * v.h;
  hipLaunchKernelGGL(k_power_sum, dim3((n + 255) / 256), dim3(256), 0, s, (const double*)power, chunks, n, sum);
  return hipGetLastError();
}

}  // namespace bnlat
