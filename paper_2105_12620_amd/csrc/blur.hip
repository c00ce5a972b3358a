// gfx950 blur criterion: separable periodised Gaussian blur of an error tile
// (Sec. 3.3), then the sum of squares.  Taps (d, k) on a ring of n pixels:
// b(x) = sum_d k_d e((x - d) mod n), in runs of consecutive d (the taps above
// the negligible level are those near 0 from either side, or all).
//
// A lane owns one integrand and 16 consecutive outputs of a row (or column).
// The 16 values that they meet at tap d move on by one at d + 1, so they stay
// in registers (slots named by the unrolled tap number) and each tap loads one
// value for its 16 FMAs; every output still adds its taps in ascending order.
// Bound by the vector ALUs for wide blurs and by memory for narrow ones.  At
// 128^2, T = 1024, on average over blur sizes 0.25 .. 20, 62 us along x and 57
// along y; loading each output's own value per tap took 430 and 604 (16 times
// as many loads from L1 and L2).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

constexpr int B = (int)BLUR_BLOCK;

#define BN_UNIFORM __attribute__((address_space(4)))
typedef float Taps __attribute__((ext_vector_type(16), aligned(4)));
static_assert(B == 16, "a block of taps is one vector");

// acc[j] = sum of the taps at output s0 + j, j < 16.  Entry i of a lane's ring
// is ring[i * stride + lane] (all else uniform); runs: first d and count; taps one run after the other,
// readable up to 15 past the last.
__device__ __forceinline__ void blur16(const float* __restrict__ ring, uint32_t lane, size_t stride,
                                       int n, int s0,
                                       const float* __restrict__ taps,
                                       const int2* __restrict__ runs, uint32_t nruns, float acc[B]) {
#pragma unroll
  for (int j = 0; j < B; ++j) acc[j] = 0.0f;
  const BN_UNIFORM float* k = (const BN_UNIFORM float*)taps;
  auto at = [&](int i) {   // entry i mod n, -16 - n < i < n + 16
    while (i < 0) i += n;
    while (i >= n) i -= n;
    return (ring + (size_t)i * stride)[lane];
  };
#pragma unroll 1
  for (uint32_t r = 0; r < nruns; ++r) {
    const BN_UNIFORM int* run = (const BN_UNIFORM int*)(runs + r);
    const int count = run[1];
    int pos = s0 - run[0];   // entry of output 0 at the current tap
    if (pos < 0) pos += n;
    float w[B];
#pragma unroll
    for (int j = 0; j < B; ++j) w[j] = at(pos + j);
#pragma unroll 1
    for (int b = 0; b < count; b += B) {
      const Taps t = *(const BN_UNIFORM Taps*)(k + b);
      float next[B];
#pragma unroll
      for (int q = 0; q < B; ++q) next[q] = at(pos - q - 1);
      if (b + B <= count) {
#pragma unroll
        for (int q = 0; q < B; ++q) {
#pragma unroll
          for (int j = 0; j < B; ++j) acc[j] = fmaf(t[q], w[(j - q) & (B - 1)], acc[j]);
          w[B - 1 - q] = next[q];
        }
      } else {
#pragma unroll
        for (int q = 0; q < B; ++q) {
          if (b + q < count) {
#pragma unroll
            for (int j = 0; j < B; ++j) acc[j] = fmaf(t[q], w[(j - q) & (B - 1)], acc[j]);
          }
          w[B - 1 - q] = next[q];
        }
      }
      pos -= B;
      while (pos < 0) pos += n;
    }
    k += count;
  }
}

// The field is float [P][pitch] with `valid` meaningful columns; one wave per
// row, 16 outputs and 64 columns.
__global__ __launch_bounds__(256) void k_blur_x(DevView v, const float* __restrict__ field, uint32_t pitch,
                                                const float* __restrict__ taps, const int2* __restrict__ runs,
                                                uint32_t nruns, float* __restrict__ out) {
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t nch = pitch >> 6, nb = (v.w + B - 1) / B;
  const uint32_t ch = wave % nch, rest = wave / nch, y = rest / nb, x0 = (rest - y * nb) * B;
  if (y >= v.h) return;
  const size_t base = (size_t)y * v.w * pitch + ch * 64;
  float acc[B];
  blur16(field + base, lane, pitch, (int)v.w, (int)x0, taps, runs, nruns, acc);
#pragma unroll
  for (int j = 0; j < B; ++j)
    if (x0 + j < v.w) (out + base + (size_t)(x0 + j) * pitch)[lane] = acc[j];
}

__global__ __launch_bounds__(256) void k_blur_y_sq(DevView v, uint32_t pitch, uint32_t valid,
                                                   const float* __restrict__ taps, const int2* __restrict__ runs,
                                                   uint32_t nruns, const float* __restrict__ in,
                                                   double* __restrict__ partial) {
  __shared__ double red[4];
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t nch = pitch >> 6, nb = (v.h + B - 1) / B;
  // waves walk down one column (and 64-integrand chunk) at a time, so the
  // waves in flight share the column's values in L2
  const uint32_t y0 = wave % nb * B, rest = wave / nb;
  const uint32_t x = rest / nch, ch = rest - x * nch;
  double sq = 0.0;
  if (x < v.w) {
    const uint32_t t = ch * 64 + lane;
    float acc[B];
    blur16(in + (size_t)x * pitch + ch * 64, lane, (size_t)v.w * pitch, (int)v.h, (int)y0, taps, runs, nruns, acc);
#pragma unroll
    for (int j = 0; j < B; ++j)
      if (t < valid && y0 + j < v.h) sq += (double)acc[j] * (double)acc[j];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
  if (lane == 0) red[threadIdx.x >> 6] = sq;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

uint32_t blocks_of(uint32_t rows, uint32_t n, uint32_t pitch) {
  return (uint32_t)(((uint64_t)rows * ((n + B - 1) / B) * (pitch >> 6) + 3) / 4);
}

}  // namespace

uint32_t blur_partials(const DevView& v, uint32_t pitch) { return blocks_of(v.w, v.h, pitch); }

hipError_t launch_blur(const DevView& v, const float* field, uint32_t pitch, uint32_t valid, const BlurTaps& x,
                       const BlurTaps& y, float* tmp, double* partial, uint32_t* npartial, hipStream_t s) {
  hipLaunchKernelGGL(k_blur_x, dim3(blocks_of(v.h, v.w, pitch)), dim3(256), 0, s, v, field, pitch, x.taps, x.runs,
                     x.nruns, tmp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  *npartial = blur_partials(v, pitch);
  hipLaunchKernelGGL(k_blur_y_sq, dim3(*npartial), dim3(256), 0, s, v, pitch, valid, y.taps, y.runs, y.nruns,
                     (const float*)tmp, partial);
  return hipGetLastError();
}

}  // namespace bnlat
