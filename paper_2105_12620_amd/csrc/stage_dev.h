// LDS-staged energy change of one colour phase (gfx950), in three forms of its
// operands; each form is compiled by its own source (stage_wide.hip,
// stage_narrow.hip, stage_split.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

// A workgroup owns a block of 32 x (BY V) class pixels; thread (tx, ty) owns
// the V class pixels of column tx in class rows ty V .. ty V + V - 1.  Their
// windows overlap, so each field word the thread reads from LDS serves all of
// them.  The workgroup also owns a slice of the integrands: for one 16-byte
// word of integrands at a time it stages the field of its block plus the window
// halo (region of RH x RW pixels) and the class pixels' recounted rows in LDS.
// Region columns are grouped by residue mod K, so the 32 lanes of a class row
// read 32 consecutive words for every window offset, each with one
// ds_read_b128 at a compile-time offset from the thread's base.  Where the
// staging words fit in registers, the next stage's global loads are issued
// before the current stage is evaluated.  Class sums stay in int32 over a
// slice: its length is bounded so that |sum_t dc_t f_q,t| < 2^31 for every
// class; they are added into xsum[class][pixel] with 64-bit integer atomics
// (exact, so the order of the slices does not matter); the decision clears
// them.
template <int R, int K, int BY, int V>
struct StageGeom {
  static constexpr int BX = 32;
  static constexpr int CR = BY * V;                                // class rows per block
  static constexpr int RH = K * (CR - 1) + 2 * R + 1;
  static constexpr int RW = ((K * (BX - 1) + 2 * R + 1 + K - 1) / K) * K;
  static constexpr int RWK = RW / K;
  static constexpr int RA = RH * RW;                               // region pixels
  static constexpr int NB = BX * CR;                               // class pixels per block
  static constexpr int NT = BX * BY;                               // threads per block
  static constexpr int DR = K * (V - 1) + 2 * R + 1;               // region rows one thread reads
  static constexpr int LDS_BYTES = 16 * (RA + NB);
  // word of region column K tx + R + ox relative to that of column K tx
  static constexpr int dcol(int ox) { return ((R + ox) % K) * RWK + (R + ox) / K; }
};

// Block shape of the staged kernel for K colour classes per axis and radius R:
// class rows per thread (V) and thread rows (BY), within 64 KiB of LDS.
// Shape 0 is the single-problem default; the batched form's tuner also tries
// shape 1 (twice the waves per workgroup for K = 4, half for K = 1, 2).
template <int R, int K, int SH = 0>
struct StageShape {
  static constexpr int V = (K == 4) ? 1 : 2;
  static constexpr int BY = (K == 4) ? (SH ? 4 : 2) : (SH ? 4 : 8);
};

// The operands of the exact integer class sums
//   X_d = |class d| sum_t dc_t (f'_t + f_t) - 2 sum_{o in class d} sum_t dc_t f_{p+o,t},
// which are the same for any field f = c - b_t with b_t fixed per integrand
// (dc = c' - c; the terms of b_t cancel class by class).
//   FIELD_WIDE    f = c as uint16, 8 integrands a word; products of int16 pairs.
//   FIELD_NARROW  f = c - b_t as int8, 16 integrands a word, where |c - b_t| and
//                 |dc| stay within 127 for every shift (host's bound,
//                 lattice_lines.h): half the bytes, half the words and stages,
//                 four products an instruction.
//   FIELD_SPLIT   the same where only |c - b_t| does: sum f'_t f_q - sum f_t f_q,
//                 the wide form's number of products at half its bytes.
// Measured at 256^2, N = 256, T = 1024, r = 4, one phase alone: wide 60 us,
// narrow 39 us.
template <int FORM>
struct StageOps;

template <>
struct StageOps<FIELD_WIDE> {
  static constexpr uint32_t IPW = 8;   // integrands per word
  struct Op {
    uint32_t d[4];
  };
  // operand of one moved pixel; returns sum_t dc_t (f'_t + f_t) of the word
  static __device__ __forceinline__ int change(const u32x4 cn, const u32x4 co, Op& o) {
    int z = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int n0 = (int)(cn[k] & 0xFFFFu), n1 = (int)(cn[k] >> 16);
      const int o0 = (int)(co[k] & 0xFFFFu), o1 = (int)(co[k] >> 16);
      o.d[k] = ((uint32_t)(n0 - o0) & 0xFFFFu) | ((uint32_t)(n1 - o1) << 16);
      z += (n0 - o0) * (n0 + o0) + (n1 - o1) * (n1 + o1);
    }
    return z;
  }
  static __device__ __forceinline__ int add(const Op& o, const u32x4 f, int x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) x = dot2(o.d[k], f[k], x);
    return x;
  }
  // a class has at most 12 offsets for radii up to 6
  static uint64_t per_integrand(uint32_t n) { return (uint64_t)12 * n * n; }
};

template <>
struct StageOps<FIELD_NARROW> {
  static constexpr uint32_t IPW = 16;
  struct Op {
    uint32_t d[4];
  };
  static __device__ __forceinline__ int change(const u32x4 cn, const u32x4 co, Op& o) {
    int zn = 0, zo = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      o.d[k] = sub_bytes(cn[k], co[k]);
      zn = dot4(cn[k], cn[k], zn);
      zo = dot4(co[k], co[k], zo);
    }
    return zn - zo;
  }
  static __device__ __forceinline__ int add(const Op& o, const u32x4 f, int x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) x = dot4(o.d[k], f[k], x);
    return x;
  }
  static uint64_t per_integrand(uint32_t) { return (uint64_t)12 * 127 * 127; }
};

template <>
struct StageOps<FIELD_SPLIT> {
  static constexpr uint32_t IPW = 16;
  struct Op {
    uint32_t n[4], m[4];   // f' and -f
  };
  static __device__ __forceinline__ int change(const u32x4 cn, const u32x4 co, Op& o) {
    int zn = 0, zo = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      o.n[k] = cn[k];
      o.m[k] = sub_bytes(0u, co[k]);
      zn = dot4(cn[k], cn[k], zn);
      zo = dot4(co[k], co[k], zo);
    }
    return zn - zo;
  }
  static __device__ __forceinline__ int add(const Op& o, const u32x4 f, int x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) x = dot4(o.m[k], f[k], dot4(o.n[k], f[k], x));
    return x;
  }
  static uint64_t per_integrand(uint32_t) { return (uint64_t)2 * 12 * 127 * 127; }
};

// Largest slice (a multiple of a word's integrands) whose class sums fit int32.
template <int FORM>
inline uint32_t stage_max_slice(uint32_t n) {
  constexpr uint32_t G = StageOps<FORM>::IPW;
  const uint64_t t = 0x7FFFFFFFull / StageOps<FORM>::per_integrand(n) / G * G;
  return t < G ? G : (t > 0x40000000u ? 0x40000000u : (uint32_t)t);
}

template <int FORM, int R, int K, int BY, int V>
__device__ __forceinline__ void delta_stage_body(const DevView& v, uint32_t kappa, uint32_t trlen,
                                                 long long* __restrict__ xpart, uint32_t bkx,
                                                 uint32_t bky, uint32_t bkz) {
  using G = StageGeom<R, K, BY, V>;
  using Ops = StageOps<FORM>;
  constexpr uint32_t IPW = Ops::IPW;
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  constexpr int ITER = (G::RA + G::NT - 1) / G::NT;
  constexpr bool PREFETCH = ITER <= 16;
  constexpr int WS = 2 * R + 1;
  extern __shared__ u32x4 lds4[];
  u32x4* reg = lds4;                 // [RA] region field
  u32x4* cnb = lds4 + G::RA;         // [NB] recounted rows of the class pixels
  const uint32_t tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const uint32_t a0 = bky * G::CR, b0 = bkx * G::BX;
  const uint32_t b = b0 + tx;
  const uint32_t ky = kappa / K, kx = kappa - ky * K;
  // top-left region pixel, made non-negative modulo the tile
  const uint32_t ys = (ky + K * a0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (kx + K * b0 + v.w * (R / v.w + 1) - R) % v.w;
  const uint32_t P = v.w * v.h;

  // staging byte offsets: the region is the same for every stage.  Lanes past
  // the region load pixel 0 and do not store it.
  uint32_t poff[ITER], wi[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const uint32_t i = threadIdx.x + it * G::NT;
    poff[it] = 0;
    wi[it] = 0xFFFFFFFFu;
    if (i < (uint32_t)G::RA) {
      const uint32_t rr = i / G::RW, cc = i - rr * G::RW;
      uint32_t gy = ys + rr, gx = xs + cc;
      while (gy >= v.h) gy -= v.h;
      while (gx >= v.w) gx -= v.w;
      poff[it] = (gy * v.w + gx) * 16;
      wi[it] = rr * G::RW + (cc % K) * G::RWK + cc / K;
    }
  }
  uint32_t coff[V];
  bool act[V];
#pragma unroll
  for (int vv = 0; vv < V; ++vv) {
    const uint32_t a = a0 + ty * V + vv;
    act[vv] = (a < v.ch) && (b < v.cw);
    coff[vv] = act[vv] ? (a * v.cw + b) * 16 : 0;
  }
  const uint32_t top = K * ty * V * G::RW + tx;

  int z0[V];
  int part[V][NCLS];
#pragma unroll
  for (int vv = 0; vv < V; ++vv) {
    z0[vv] = 0;
#pragma unroll
    for (int c = 0; c < NCLS; ++c) part[vv][c] = 0;
  }

  const uint32_t t_begin = bkz * trlen, t_end = min(t_begin + trlen, v.tp);
  const char* fld = FORM == FIELD_WIDE ? (const char*)v.cnt : (const char*)v.d8;
  const char* nfl = FORM == FIELD_WIDE ? (const char*)v.c_new : (const char*)v.n8;
  u32x4 q[ITER], qc[V];
  auto issue = [&](uint32_t t0) {
    const char* cs = fld + (size_t)(t0 / IPW) * P * 16;
    const char* ns = nfl + (size_t)(t0 / IPW) * v.pc * 16;
#pragma unroll
    for (int it = 0; it < ITER; ++it) q[it] = *(const u32x4*)(cs + poff[it]);
#pragma unroll
    for (int vv = 0; vv < V; ++vv) qc[vv] = *(const u32x4*)(ns + coff[vv]);
  };
  if (PREFETCH && t_begin < t_end) issue(t_begin);
  for (uint32_t t0 = t_begin; t0 < t_end; t0 += IPW) {
    __syncthreads();
    if (!PREFETCH) issue(t0);
#pragma unroll
    for (int it = 0; it < ITER; ++it)
      if (wi[it] != 0xFFFFFFFFu) reg[wi[it]] = q[it];
#pragma unroll
    for (int vv = 0; vv < V; ++vv) cnb[(ty * V + vv) * G::BX + tx] = qc[vv];
    __syncthreads();
    if (PREFETCH && t0 + IPW < t_end) issue(t0 + IPW);
    typename Ops::Op d[V];
#pragma unroll
    for (int vv = 0; vv < V; ++vv)
      z0[vv] += Ops::change(cnb[(ty * V + vv) * G::BX + tx], reg[top + (R + K * vv) * G::RW + G::dcol(0)], d[vv]);
#pragma unroll
    for (int dr = 0; dr < G::DR; ++dr) {
      // a row's words are loaded together, so their LDS latencies overlap
      u32x4 row[WS];
#pragma unroll
      for (int ox = -R; ox <= R; ++ox) row[ox + R] = reg[top + dr * G::RW + G::dcol(ox)];
#pragma unroll
      for (int ox = -R; ox <= R; ++ox) {
        const u32x4 cq = row[ox + R];
#pragma unroll
        for (int vv = 0; vv < V; ++vv) {
          const int oy = dr - R - K * vv;
          if (oy < -R || oy > R || (ox == 0 && oy == 0)) continue;
          const int c = W.cmap[(oy + R) * WS + ox + R];
          part[vv][c] = Ops::add(d[vv], cq, part[vv][c]);
        }
      }
    }
  }
#pragma unroll
  for (int vv = 0; vv < V; ++vv) {
    if (act[vv]) {
      const uint32_t j = (a0 + ty * V + vv) * v.cw + b;
#pragma unroll
      for (int c = 0; c < NCLS; ++c)
        atomicAdd((unsigned long long*)&xpart[(size_t)c * v.pc + j],
                  (unsigned long long)((long long)W.csize[c] * z0[vv] - 2 * (long long)part[vv][c]));
    }
  }
}

// One-dimensional grid of gx x gy blocks x slices, renumbered per XCD: the
// blocks one L2 serves at a time are whole rows of blocks of one slice, whose
// window halos are then read from HBM once.
template <int FORM, int R, int K, int BY, int V>
__global__ __launch_bounds__(32 * BY) void k_delta_stage(DevView v, uint32_t kappa, uint32_t trlen,
                                                         long long* __restrict__ xpart, uint32_t gx,
                                                         uint32_t gy) {
  // the colour phases' waves issue ahead of the sweep-wide recount running
  // beside them (k_decide_commit, k_delta_finish, k_commit and the BF16 form's k_delta_bf
  // and k_delta_refine likewise), which fills the remaining issue slots
  __builtin_amdgcn_s_setprio(2);
  const uint32_t wk = xcd_block(blockIdx.x, gridDim.x), bxy = wk % (gx * gy);
  delta_stage_body<FORM, R, K, BY, V>(v, kappa, trlen, xpart, bxy % gx, bxy / gx, wk / (gx * gy));
}

// Batched form: member i owns blocks pre[i] .. pre[i+1]-1, laid out as its own
// (x, y, slice) grid; its slice length is in trl[i].
template <int FORM, int R, int K, int BY, int V>
__global__ __launch_bounds__(32 * BY) void k_delta_stage_batch(const DevView* __restrict__ views,
                                                               const uint32_t* __restrict__ pre,
                                                               const uint32_t* __restrict__ geo,
                                                               uint32_t nmem, uint32_t kappa) {
  // like the single problem's phase kernels: issue ahead of the recount
  __builtin_amdgcn_s_setprio(2);
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  const DevView v = views[i];
  const uint32_t lb = blockIdx.x - pre[i];
  const uint32_t gx = geo[3 * i], gy = geo[3 * i + 1], trlen = geo[3 * i + 2];
  delta_stage_body<FORM, R, K, BY, V>(v, kappa, trlen, v.xpart, lb % gx, (lb / gx) % gy, lb / (gx * gy));
}

// Integrand slices of a staged launch: about slice_target workgroups in total
// (512 by default), each slice a whole number of words, at least 64 integrands
// long (a slice adds its class sums with atomics and restages the window
// halo), shorter where the launch would leave CUs idle otherwise, and within
// the int32 bound.
template <int FORM>
inline uint32_t stage_slices(const DevView& v, uint32_t blocks, uint32_t* trlen) {
  constexpr uint32_t G = StageOps<FORM>::IPW;
  const uint32_t chunks = (v.t + G - 1) / G;
  const uint32_t target = v.slice_target ? v.slice_target : 512;
  const uint32_t want = min(chunks, (target + blocks - 1) / blocks);
  uint32_t per = (chunks + want - 1) / want;
  uint32_t min_per = min(chunks, 64 / G);
  if (blocks * ((chunks + min_per - 1) / min_per) < 256) min_per = max(1u, chunks * blocks / 256);
  per = min(max(per, min_per), max(1u, stage_max_slice<FORM>(v.n) / G));
  *trlen = per * G;
  return (chunks + per - 1) / per;
}

template <int FORM, int R, int K>
hipError_t stage_rk(const DevView& v, uint32_t kappa, hipStream_t s) {
  using S = StageShape<R, K>;
  using G = StageGeom<R, K, S::BY, S::V>;
  static_assert(G::LDS_BYTES <= 65536, "staged block exceeds 64 KiB of LDS");
  uint32_t trlen = 0;
  const uint32_t gx = (v.cw + G::BX - 1) / G::BX, gy = (v.ch + G::CR - 1) / G::CR;
  const uint32_t ns = stage_slices<FORM>(v, gx * gy, &trlen);
  hipLaunchKernelGGL((k_delta_stage<FORM, R, K, S::BY, S::V>), dim3(gx * gy * ns), dim3(G::NT), (size_t)G::LDS_BYTES, s,
                     v, kappa, trlen, v.xpart, gx, gy);
  return hipGetLastError();
}

template <int FORM, int R>
hipError_t stage_r(const DevView& v, uint32_t kappa, hipStream_t s) {
  switch (v.k) {
    case 1: return stage_rk<FORM, R, 1>(v, kappa, s);
    case 2: return stage_rk<FORM, R, 2>(v, kappa, s);
    case 4: return stage_rk<FORM, R, 4>(v, kappa, s);
    default: return hipErrorInvalidValue;
  }
}

template <int FORM>
hipError_t stage_form(const DevView& v, uint32_t kappa, hipStream_t s) {
  switch (v.radius) {
    case 1: return stage_r<FORM, 1>(v, kappa, s);
    case 2: return stage_r<FORM, 2>(v, kappa, s);
    case 3: return stage_r<FORM, 3>(v, kappa, s);
    case 4: return stage_r<FORM, 4>(v, kappa, s);
    case 5: return stage_r<FORM, 5>(v, kappa, s);
    case 6: return stage_r<FORM, 6>(v, kappa, s);
    default: return hipErrorInvalidValue;
  }
}

template <int FORM, int R, int K, int SH>
hipError_t stage_batch_rk(const DevView* views, const uint32_t* pre, const uint32_t* geo, uint32_t nmem,
                          uint32_t blocks, uint32_t kappa, hipStream_t s) {
  using S = StageShape<R, K, SH>;
  using G = StageGeom<R, K, S::BY, S::V>;
  static_assert(G::LDS_BYTES <= 65536, "staged block exceeds 64 KiB of LDS");
  static_assert(G::CR == StageShape<1, K == 4 ? 4 : 2, SH>::BY * StageShape<1, K == 4 ? 4 : 2, SH>::V,
                "batched geometry assumes one block shape per (K, shape)");
  hipLaunchKernelGGL((k_delta_stage_batch<FORM, R, K, S::BY, S::V>), dim3(blocks), dim3(G::NT), (size_t)G::LDS_BYTES, s,
                     views, pre, geo, nmem, kappa);
  return hipGetLastError();
}

template <int FORM, int R>
hipError_t stage_batch_r(uint32_t k, uint32_t shape, const DevView* views, const uint32_t* pre, const uint32_t* geo,
                         uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s) {
  switch (k * 2 + (shape ? 1 : 0)) {
    case 2: return stage_batch_rk<FORM, R, 1, 0>(views, pre, geo, nmem, blocks, kappa, s);
    case 3: return stage_batch_rk<FORM, R, 1, 1>(views, pre, geo, nmem, blocks, kappa, s);
    case 4: return stage_batch_rk<FORM, R, 2, 0>(views, pre, geo, nmem, blocks, kappa, s);
    case 5: return stage_batch_rk<FORM, R, 2, 1>(views, pre, geo, nmem, blocks, kappa, s);
    case 8: return stage_batch_rk<FORM, R, 4, 0>(views, pre, geo, nmem, blocks, kappa, s);
    case 9: return stage_batch_rk<FORM, R, 4, 1>(views, pre, geo, nmem, blocks, kappa, s);
    default: return hipErrorInvalidValue;
  }
}

template <int FORM>
hipError_t stage_batch_form(uint32_t radius, uint32_t k, uint32_t shape, const DevView* views, const uint32_t* pre,
                            const uint32_t* geo, uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s) {
  switch (radius) {
    case 1: return stage_batch_r<FORM, 1>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    case 2: return stage_batch_r<FORM, 2>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    case 3: return stage_batch_r<FORM, 3>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    case 4: return stage_batch_r<FORM, 4>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    case 5: return stage_batch_r<FORM, 5>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    case 6: return stage_batch_r<FORM, 6>(k, shape, views, pre, geo, nmem, blocks, kappa, s);
    default: return hipErrorInvalidValue;
  }
}

template <int FORM>
void stage_geometry_form(const DevView& v, uint32_t shape, uint32_t* gx, uint32_t* gy, uint32_t* gz, uint32_t* trlen) {
  using A = StageShape<1, 2, 0>;
  using B = StageShape<1, 2, 1>;
  using C = StageShape<1, 4, 0>;
  using D = StageShape<1, 4, 1>;
  const uint32_t cr = v.k == 4 ? (shape ? D::BY * D::V : C::BY * C::V) : (shape ? B::BY * B::V : A::BY * A::V);
  *gx = (v.cw + 31) / 32;
  *gy = (v.ch + cr - 1) / cr;
  *gz = stage_slices<FORM>(v, *gx * *gy, trlen);
}

}  // namespace

// The entry points of one form (one source each).
#define BN_STAGE_FORM(FORM, NAME)                                                                                      \
  hipError_t launch_stage_##NAME(const DevView& v, uint32_t kappa, hipStream_t s) {                                    \
    return stage_form<FORM>(v, kappa, s);                                                                              \
  }                                                                                                                    \
  hipError_t launch_stage_batch_##NAME(uint32_t radius, uint32_t k, uint32_t shape, const DevView* views,              \
                                       const uint32_t* pre, const uint32_t* geo, uint32_t nmem, uint32_t blocks,       \
                                       uint32_t kappa, hipStream_t s) {                                                \
    return stage_batch_form<FORM>(radius, k, shape, views, pre, geo, nmem, blocks, kappa, s);                          \
  }                                                                                                                    \
  void stage_geometry_##NAME(const DevView& v, uint32_t shape, uint32_t* gx, uint32_t* gy, uint32_t* gz,               \
                             uint32_t* trlen) {                                                                        \
    stage_geometry_form<FORM>(v, shape, gx, gy, gz, trlen);                                                            \
  }

}  // namespace bnlat
