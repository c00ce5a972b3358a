// gfx950 Gaussian estimates along lattice lines (Sec. 3.5 integrands on the
// rank-1 lattice of Sec. 3.2).
//
// Estimate of one Gaussian at one pixel: (1 / N) sum_k 2^E(s^k), E the base-2
// exponent a |x|^2 + bx x + by y + c.  The samples lie on lines O_l + j b1
// (lattice_lines.h), where E is a quadratic in j with the same second
// difference on every line, so a line's sum is
//   2^E(O_l) sum_j w_j z_l^j,   w_j = 2^(a |b1|^2 j^2),  z_l = 2^(slope at O_l):
// a polynomial in z_l with coefficients that depend on the Gaussian alone.
// Horner's rule takes one FP64 FMA per sample where evaluating each sample's
// exponential took 8.4 issue slots (3 FMAs, a conversion, v_exp_f32, an add);
// z_l and 2^E(O_l) follow from line to line by multiplication, so a pixel and
// Gaussian cost four FP64 exponentials in all.  The terms are FP64 throughout
// (the relative error of a term, about j^2 2^-52, is far below the FP32
// result's), where the exponentials were FP32 before.
//
// A lane owns one pixel and a wave four Gaussians (four independent chains),
// their interleaved tables in scalar registers; the four waves of a workgroup
// share the pixels.  Which steps of a line a pixel
// has depends on the class of its shift: the few steps at either end that not
// every class has run under the execution mask (one comparison for the four
// Gaussians), those in between without.  The classes' rows are kept in LDS, and
// the results change hands there so that whole runs of a pixel's row are
// written.  Bound by the vector ALUs (1.7 slots per sample at N = 1024, 12 ms of
// issue) and the latency of the scalar loads (five waves a SIMD).
// Measured at 512^2, N = 1024, 1024 Gaussians: 13.8 ms per estimate of all
// pixels against 57.4 sample by sample; 15.6 with 16 Gaussians a wave, one four
// after the other, and a launch over few pixels took four times as long (256
// listed moves: 283 us the call against 141); four lines at a time in place of
// four Gaussians, whose common steps are fewer, took 41.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

#define BN_UNIFORM __attribute__((address_space(4)))
template <class T>
__device__ inline const BN_UNIFORM T* uniform(const T* p) {
  return (const BN_UNIFORM T*)p;
}

constexpr uint32_t GC = 4;           // Gaussians per wave
constexpr uint32_t OUT_PITCH = GC + 1;

typedef double Two __attribute__((ext_vector_type(8), aligned(8)));   // two steps' entries of four tables

// p z + w, w in scalar registers.  Left to itself the compiler takes the
// accumulating form, which first moves w to vector registers: two more
// instructions per step.
__device__ __forceinline__ void horner(double& p, double z, double w) {
  asm("v_fma_f64 %0, %0, %1, %2" : "+v"(p) : "v"(z), "s"(w));
}

// Sum over the samples one by one (exponents beyond FP64's range).
__device__ double gauss_by_sample(const DevView& v, uint32_t u, uint32_t t) {
  const BN_UNIFORM double* c = uniform(v.gcoef) + 4 * t;
  double s = 0.0;
#pragma unroll 1
  for (uint32_t i = 0; i < v.n; ++i) {
    const uint32_t sv = wrap_add(uniform(v.lat)[i], u);
    const double x = (double)(sv & 0xFFFFu) * 0x1p-16, y = (double)(sv >> 16) * 0x1p-16;
    const double e = __fma_rn(c[0], __fma_rn(x, x, y * y), __fma_rn(c[1], x, __fma_rn(c[2], y, c[3])));
    s += exp2(e);
  }
  return s;
}

// LDS words per workgroup: class rows [lines][64] and results [4][64][OUT_PITCH].
inline size_t lds_words(uint32_t lines) { return (size_t)lines * 64 + 4 * 64 * OUT_PITCH; }

template <bool ALL>
__global__ __launch_bounds__(256, 5) void k_gauss_lines(DevView v, uint32_t m) {
  extern __shared__ uint32_t rows[];
  const uint32_t lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t ng = (v.tg + 4 * GC - 1) / (4 * GC);   // workgroups per 64 pixels
  const uint32_t jg = blockIdx.x / ng, t0 = ((blockIdx.x - jg * ng) * 4 + w) * GC;
  float* outs = (float*)(rows + v.glines * 64) + w * 64 * OUT_PITCH;
  const uint32_t j = min(jg * 64 + lane, m - 1);
  const uint32_t u = ALL ? v.U[j] : v.u_new[j];

  const uint32_t sh = 16 - v.log2n, ux = u & 0xFFFFu, uy = u >> 16;
  const uint32_t cls = ((uy >> sh) * v.gx - (ux >> sh) * v.gy) & (v.n - 1);
  const uint32_t* row = v.grow + (size_t)cls * (1 + v.glines);
  const uint32_t aw = row[0], fm = (1u << sh) - 1;
  for (uint32_t l = w; l < v.glines; l += 4) rows[l * 64 + lane] = row[1 + l];
  __syncthreads();
  // A in the unit square's coordinates (exact)
  const double ax = (double)((int)(int16_t)(aw & 0xFFFFu) * (1 << sh) + (int)(ux & fm)) * 0x1p-16;
  const double ay = (double)(((int)aw >> 16) * (1 << sh) + (int)(uy & fm)) * 0x1p-16;
  const double a2 = __fma_rn(ax, ax, ay * ay);
  const double inv_n = 1.0 / (double)v.n;

  double total[4] = {0.0, 0.0, 0.0, 0.0};
  if (t0 < v.tg) {
    const BN_UNIFORM double* tab = uniform(v.gtab) + (size_t)t0 * v.gwords;
    double y[4], za[4], zi[4], ys[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = exp2(__fma_rn(tab[e], a2, __fma_rn(tab[4 + e], ax, __fma_rn(tab[8 + e], ay, tab[12 + e]))));
      const double le = __fma_rn(tab[16 + e], ax, __fma_rn(tab[20 + e], ay, tab[24 + e]));
      za[e] = exp2(le);
      zi[e] = exp2(-le);
      ys[e] = exp2(__fma_rn(tab[28 + e], ax, __fma_rn(tab[32 + e], ay, tab[36 + e])));
    }
    const BN_UNIFORM double* wt = tab + 4 * (GAUSS_HEAD + 2 * v.glines);
#pragma unroll 1
    for (uint32_t l = 0; l < v.glines; ++l) {
      const uint32_t r = rows[l * 64 + lane];
      const int lo = (int)(r & 0xFFFFu), hi = (int)(r >> 16);
      const BN_UNIFORM int* span = uniform(v.gspans) + 4 * l;
      const BN_UNIFORM double* kc = tab + 4 * (GAUSS_HEAD + 2 * l);
      double z[4], f[4], p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        z[e] = za[e] * kc[e];
        f[e] = y[e] * kc[4 + e];
        p[e] = 0.0;
      }
      const int flo = span[1], fhi = span[2], d = span[3];
      int s = span[0] - 1;
      const BN_UNIFORM double* wp = wt + 4 * (s - 1);
      // (the empty asm keeps the steps under the execution mask; as selects
      // they would cost two instructions each)
#pragma unroll 1
      for (; s >= fhi; s -= 2, wp -= 8) {
        const Two w = *(const BN_UNIFORM Two*)wp;
        if (s < hi) {
#pragma unroll
          for (int e = 0; e < 4; ++e) horner(p[e], z[e], w[4 + e]);
          asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]));
        }
        if (s == fhi) {
          --s;
          wp -= 4;
          break;
        }
        if (s <= hi) {
#pragma unroll
          for (int e = 0; e < 4; ++e) horner(p[e], z[e], w[e]);
          asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]));
        }
      }
#pragma unroll 1
      for (; s >= flo + 3; s -= 4, wp -= 16) {
        const Two w0 = *(const BN_UNIFORM Two*)wp, w1 = *(const BN_UNIFORM Two*)(wp - 8);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w0[4 + e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w0[e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w1[4 + e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w1[e]);
      }
      if (s > flo) {
        const Two w = *(const BN_UNIFORM Two*)wp;
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w[4 + e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w[e]);
        s -= 2;
        wp -= 8;
      }
      if (s >= flo) {   // one common step left
        const Two w = *(const BN_UNIFORM Two*)wp;
#pragma unroll
        for (int e = 0; e < 4; ++e) horner(p[e], z[e], w[4 + e]);
        --s;
        wp -= 4;
      }
#pragma unroll 1
      for (; s >= 0; s -= 2, wp -= 8) {
        const Two w = *(const BN_UNIFORM Two*)wp;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (s >= k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] *= z[e];
            if (s - k >= lo && s - k < hi) {
#pragma unroll
              for (int e = 0; e < 4; ++e) p[e] = __dadd_rn(p[e], w[4 - 4 * k + e]);
              asm volatile("" : "+v"(p[0]), "+v"(p[1]), "+v"(p[2]), "+v"(p[3]));
            }
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        total[e] = __fma_rn(f[e], p[e], total[e]);
        y[e] *= ys[e];   // origin of the next line: b2 and d steps of b1 further
      }
#pragma unroll 1
      for (int k = 0; k < d; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] *= za[e];
#pragma unroll 1
      for (int k = 0; k > d; --k)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] *= zi[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (tab[44 + e] != 0.0) total[e] = gauss_by_sample(v, u, t0 + e);
  }
#pragma unroll
  for (uint32_t e = 0; e < 4; ++e) {
    if (t0 + e >= v.tg) total[e] = (double)v.n;   // padding: estimate 1
    outs[lane * OUT_PITCH + e] = (float)(total[e] * inv_n);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  float* out = (ALL ? v.gest : v.g_new) + t0;
#pragma unroll
  for (uint32_t r = 0; r < 64; r += 64 / GC) {
    const uint32_t px = r + lane / GC, jp = jg * 64 + px;
    if (jp < m) out[(size_t)jp * v.tgp + lane % GC] = outs[px * OUT_PITCH + lane % GC];
  }
  // the padding past the last workgroup's Gaussians
  const uint32_t pad = v.tgp - ng * 4 * GC;
  if (pad && (blockIdx.x + 1) % ng == 0)
    for (uint32_t i = threadIdx.x; i < 64 * pad; i += 256) {
      const uint32_t jp = jg * 64 + i / pad;
      if (jp < m) (ALL ? v.gest : v.g_new)[(size_t)jp * v.tgp + (v.tgp - pad) + i % pad] = 1.0f;
    }
}

}  // namespace

hipError_t launch_gauss_lines(const DevView& v, bool all, uint32_t m, hipStream_t s) {
  const size_t lds = 4 * lds_words(v.glines);
  const dim3 grid((m + 63) / 64 * ((v.tg + 4 * GC - 1) / (4 * GC))), block(256);
  if (all) hipLaunchKernelGGL(k_gauss_lines<true>, grid, block, lds, s, v, m);
  else hipLaunchKernelGGL(k_gauss_lines<false>, grid, block, lds, s, v, m);
  return hipGetLastError();
}

}  // namespace bnlat
