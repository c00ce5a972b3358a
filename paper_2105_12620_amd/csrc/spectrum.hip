// Radially averaged power spectrum of the error tile (the |FFT(e)|^2 insets
// of Fig. 1b), as a diagnostic beside the blur criterion of Sec. 3.3.  A
// direct separable DFT over the W x H torus, chunks of 64 integrand rows:
// first along x, then along y with |.|^2 summed over a chunk's integrands per
// frequency (u, v) and over the chunks in order.  FP32 twiddles and sums within
// a row or column, FP64 across integrands.
//
// A lane owns one integrand and 8 consecutive frequencies, so that a value is
// loaded once for 8 of them; their twiddles tw[u x mod n], uniform over the wave,
// come by scalar loads: from a matrix [position][frequency], 8 in one load, or
// from the n values themselves, their indexes stepped by u in scalar registers.
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
typedef float Twiddle __attribute__((ext_vector_type(2), aligned(8)));        // cos and -sin
typedef float Twiddles __attribute__((ext_vector_type(2 * F), aligned(8)));   // of F frequencies at one position
static_assert(F == 8, "the twiddles of a lane are one vector");

// blocks of F frequencies
__host__ __device__ inline uint32_t blocks(uint32_t n) { return (n + F - 1) / F; }

// mat[x][u] = tw[u x mod n], u < F blocks(n) (n <= MATRIX_SIDE).
__global__ __launch_bounds__(256) void k_twiddles(const float2* __restrict__ tw, uint32_t n, float2* __restrict__ mat) {
  const uint32_t np = F * blocks(n), i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * np) return;
  const uint32_t x = i / np, u = i - x * np;
  mat[i] = tw[u * x % n];
}

// The twiddles of frequencies u0 .. u0 + F - 1 at the positions of a ring of n,
// from 0 on (frequencies past n - 1 repeat the first ones; they are not stored).
// MATRIX: tw is the matrix, else the n values.
template <bool MATRIX>
struct Frequencies;

template <>
struct Frequencies<true> {
  const BN_UNIFORM float* at;
  uint32_t pitch;
  __device__ __forceinline__ Frequencies(const float2* tw, uint32_t n, uint32_t u0)
      : at((const BN_UNIFORM float*)(tw + u0)), pitch(2 * F * blocks(n)) {}
  __device__ __forceinline__ Twiddles next() {
    const Twiddles q = *(const BN_UNIFORM Twiddles*)at;
    at += pitch;
    return q;
  }
};

template <>
struct Frequencies<false> {
  const BN_UNIFORM Twiddle* tw;
  uint32_t n, step[F], at[F];
  __device__ __forceinline__ Frequencies(const float2* t, uint32_t n_, uint32_t u0)
      : tw((const BN_UNIFORM Twiddle*)t), n(n_) {
#pragma unroll
    for (int f = 0; f < F; ++f) step[f] = (u0 + f) % n, at[f] = 0;
  }
  __device__ __forceinline__ Twiddles next() {
    Twiddles q;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const Twiddle t = tw[at[f]];
      q[2 * f] = t[0];
      q[2 * f + 1] = t[1];
      at[f] += step[f];
      at[f] = min(at[f], at[f] - n);   // (at - n wraps where at < n)
    }
    return q;
  }
};

// rows[c][y][u][64] of chunk c, integrands t0 + 64 c ..
template <bool MATRIX>
__global__ __launch_bounds__(256) void k_dft_x(const float* __restrict__ field, uint32_t pitch, uint32_t valid,
                                               uint32_t t0, uint32_t chunks, uint32_t w, uint32_t h,
                                               const float2* __restrict__ tw, float2* __restrict__ rows) {
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t nb = blocks(w);
  const uint32_t ub = wave % nb, rest = wave / nb, y = rest % h, c = rest / h;
  if (c >= chunks) return;
  const uint32_t t = t0 + c * SPEC_CHUNK;
  const float* row = field + (size_t)y * w * pitch + t;
  Frequencies<MATRIX> fr(tw, w, ub * F);
  float re[F], im[F];
#pragma unroll
  for (int f = 0; f < F; ++f) re[f] = im[f] = 0.0f;
  if (t + lane < valid) {
#pragma unroll 4
    for (uint32_t x = 0; x < w; ++x) {
      const float e = (row + (size_t)x * pitch)[lane];
      const Twiddles q = fr.next();
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
template <bool MATRIX>
__global__ __launch_bounds__(256) void k_dft_y_power(const float2* __restrict__ rows, uint32_t chunks, uint32_t w,
                                                     uint32_t h, const float2* __restrict__ tw,
                                                     double* __restrict__ power) {
  const uint32_t lane = threadIdx.x & 63, wave = wave_id();
  const uint32_t nb = blocks(h);
  const uint32_t vb = wave % nb, rest = wave / nb, u = rest % w, c = rest / w;
  if (c >= chunks) return;
  const float2* col = rows + ((size_t)c * h * w + u) * SPEC_CHUNK;
  Frequencies<MATRIX> fr(tw, h, vb * F);
  float re[F], im[F];
#pragma unroll
  for (int f = 0; f < F; ++f) re[f] = im[f] = 0.0f;
#pragma unroll 4
  for (uint32_t y = 0; y < h; ++y) {
    const float2 a = (col + (size_t)y * w * SPEC_CHUNK)[lane];
    const Twiddles q = fr.next();
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

// sum += the chunks' powers, in order (first: sum = theirs).
__global__ __launch_bounds__(256) void k_power_sum(const double* __restrict__ power, uint32_t chunks, uint32_t n,
                                                   bool first, double* __restrict__ sum) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = first ? 0.0 : sum[i];
  for (uint32_t c = 0; c < chunks; ++c) s += power[(size_t)c * n + i];
  sum[i] = s;
}

}  // namespace

uint32_t spectrum_chunk() { return SPEC_CHUNK; }

uint32_t spectrum_chunks(const DevView& v, uint32_t rows) {
  const uint64_t waves = std::min((uint64_t)v.h * blocks(v.w), (uint64_t)v.w * blocks(v.h));
  const uint64_t want = std::max<uint64_t>(1, (16384 + waves - 1) / waves);
  return (uint32_t)std::min<uint64_t>(want, std::max(1u, (rows + SPEC_CHUNK - 1) / SPEC_CHUNK));
}

// A matrix of the twiddles along a side of n, for spectra of `rows` integrand
// rows?  It halves the time of the transforms (128^2, 1024 rows: 620 us a spectrum
// against 1090; 64^2, 256 rows: 121 against 105), costs a launch to fill it, and
// grows as n^2 (128 MiB at the largest side taken).
constexpr uint32_t MATRIX_SIDE = 4096;
bool spectrum_matrix(const DevView& v, uint32_t n, uint32_t rows) {
  const uint64_t chunks = (rows + SPEC_CHUNK - 1) / SPEC_CHUNK;
  return n <= MATRIX_SIDE && chunks * v.w * v.h * ((uint64_t)v.w + v.h) >= 1u << 22;
}

size_t spectrum_matrix_size(uint32_t n) { return (size_t)n * F * blocks(n); }

hipError_t launch_twiddles(const float2* tw, uint32_t n, float2* mat, hipStream_t s) {
  hipLaunchKernelGGL(k_twiddles, dim3((unsigned)((spectrum_matrix_size(n) + 255) / 256)), dim3(256), 0, s, tw, n, mat);
  return hipGetLastError();
}

SpectrumScratch spectrum_scratch(const DevView& v, uint32_t chunks) {
  const size_t n = (size_t)v.w * v.h;
  return {n * SPEC_CHUNK * chunks, n * chunks};
}

hipError_t launch_spectrum_chunks(const DevView& v, const float* field, uint32_t pitch, uint32_t valid, uint32_t t0,
                                  uint32_t chunks, bool first, const SpectrumTwiddles& x, const SpectrumTwiddles& y,
                                  float2* rows, double* power, double* sum, hipStream_t s) {
  const uint64_t wx = (uint64_t)chunks * v.h * blocks(v.w), wy = (uint64_t)chunks * v.w * blocks(v.h);
  hipLaunchKernelGGL(x.matrix ? k_dft_x<true> : k_dft_x<false>, dim3((unsigned)((wx + 3) / 4)), dim3(256), 0, s, field,
                     pitch, valid, t0, chunks, v.w, v.h, x.tw, rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool one = first && chunks == 1;   // the chunk's power is the sum so far
  hipLaunchKernelGGL(y.matrix ? k_dft_y_power<true> : k_dft_y_power<false>, dim3((unsigned)((wy + 3) / 4)), dim3(256), 0,
                     s, (const float2*)rows, chunks, v.w, v.h, y.tw, one ? sum : power);
  if ((e = hipGetLastError()) != hipSuccess || one) return e;
  const uint32_t n = v.w * v.h;
  hipLaunchKernelGGL(k_power_sum, dim3((n + 255) / 256), dim3(256), 0, s, (const double*)power, chunks, n, first, sum);
  return hipGetLastError();
}

}  // namespace bnlat
