// gfx950 energy change and decision of one colour phase on an int8 field, by
// the matrix cores.
//
// The exact integer class sums of a move,
//   X_d = |class d| sum_t dc_t (f'_t + f_t) - 2 sum_{o in class d} sum_t dc_t f_{p+o,t},
// are the same for any field f = c - b_t with b_t fixed per integrand (dc =
// c' - c; the terms of b_t cancel class by class).  Two forms, each compiled by
// its own source (phase_narrow.hip, phase_split.hip):
//   FIELD_NARROW  |c - b_t| and |dc| stay within 127 for every shift (the
//                 host's bound, lattice_lines.h): one product per pair;
//   FIELD_SPLIT   only |c - b_t| does: sum f'_t f_q - sum f_t f_q.
//
// The products are a Gram block: v_mfma_i32_16x16x64_i8 multiplies 64
// integrands of 16 class pixels of a row (A) with those of 16 consecutive
// pixels of a region row (B), exactly.  A lane's operand is one 16-byte word of
// 16 integrands of one pixel, which is how the field lies in memory
// ([Tp/16][P][16]), so words go from memory into LDS as they are
// (global_load_lds_dwordx4) and from there into the matrix cores: the vector
// ALUs are left to the sweep-wide recount running beside this kernel.
// A workgroup owns BY class rows of 16 pixels; for 64 integrands at a time (one
// stage) the window region of RH x RW pixels (four planes of words) and the
// class pixels' recounted words are in one half of its LDS while the next
// stage's load into the other, with one barrier a stage (three buffers were no
// faster for one problem and left no room for a second workgroup on the CU in
// batches of small ones: 1250 against 1042 us).  A wave owns one class row, or
// the offsets with |oy| = part mod S of one where the LDS holds fewer rows;
// offsets +-oy share their accumulators (their distances agree).
// 9 of the 48 columns of a row's products are used at r = 4, K = 2, yet the
// matrix cores need 3 us per phase at 256^2, T = 1024, where the vector ALUs
// (v_dot4) need 12.  The accumulators are gathered into 64-bit class sums
// through LDS and a lane per pixel decides.
//
// Measured at 256^2, N = 256, T = 1024, r = 4, decision included: 23 us per
// phase alone and 24 beside the recount (84 MB read, 3.6 TB/s: bound by memory
// and, at the ends, latency), against 42 with v_dot4 on integrand slices
// added by 64-bit atomics (which all go to memory on this part: 13 us of it),
// 30 alone and 56 beside the recount with v_dot4 and whole sums (two waves a
// SIMD with 250 registers), and 34 with the B words loaded straight into
// registers (4.1 times the tile through the L1s).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int R, int K>
struct GramGeom {
  static constexpr int NCLS = WinConst<R>::NCLS;
  static constexpr int CT = (15 * K + 2 * R + 1 + 15) / 16;        // column tiles of a region row
  static constexpr int RW = 15 * K + 2 * R + 1;                    // region columns
  static constexpr int rows(int by) { return K * (by - 1) + 2 * R + 1; }
  // words of one plane: the last row's tiles read past RW, whole 64-lane loads
  static constexpr int plane(int by) { return (rows(by) * RW + 16 * CT - RW + 63) / 64 * 64; }
  static constexpr int stage(int by) { return 4 * plane(by) + 64 * by; }
  static constexpr int LDS_MAX = 163840 - 1024;
  // four class rows, or the fewer whose stages fit twice
  static constexpr int BY = 32 * stage(4) <= LDS_MAX ? 4 : 32 * stage(2) <= LDS_MAX ? 2 : 1;
  static constexpr int NW = 4, S = NW / BY;                        // waves; waves per class row
  static constexpr int RH = rows(BY), PLANE = plane(BY), STAGE = stage(BY);
  static constexpr int PX = 16 * BY;                               // class pixels per workgroup
  static constexpr int NO = (R + S) / S;                           // |oy| values of a wave
  static constexpr int CHUNKS = PLANE / 64;                        // 64-word loads of a plane
  static constexpr int NC = (CHUNKS + NW - 1) / NW;                // of a wave (of all four planes)
  static constexpr int PITCH = 16 * CT + 4;                        // words of a row of products in LDS
  static constexpr int ENTRIES = (R + 1) * (2 * R + 1);            // window offsets with oy >= 0
  // after the stages, in their place: products [BY][R + 1][16][PITCH], then class sums
  static constexpr int PROD = BY * (R + 1) * 16 * PITCH;
  static constexpr int END_BYTES = 4 * PROD + 8 * (NCLS + 1) * PX + 16;
  static constexpr int RING_BYTES = 32 * STAGE;
  static constexpr int LDS_BYTES = RING_BYTES > END_BYTES ? RING_BYTES : END_BYTES;
  static_assert(LDS_BYTES <= 163840, "phase block exceeds the LDS");
};

template <int FORM, int R, int K, bool SLICED>
__device__ __forceinline__ void gram_body(const DevView& v, uint32_t kappa, const SliceBlock<SLICED> sb, uint32_t gx) {
  using G = GramGeom<R, K>;
  constexpr Window<R> WN = WinConst<R>::w;
  constexpr int NCLS = G::NCLS, CT = G::CT, WS = 2 * R + 1, S = G::S;
  extern __shared__ u32x4 lds4[];
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t c16 = lane & 15, g = lane >> 4;
  const uint32_t m = w / S, part = w % S;      // class row of the wave, its offsets
  const uint32_t a0 = sb.b / gx * G::BY, b0 = sb.b % gx * 16;
  const uint32_t ky = kappa / K, kx = kappa - ky * K;
  const uint32_t P = v.w * v.h;

  // chunk w + NW k of the four planes' region words: word u = 64 chunk + lane
  // (words past the region read its last pixel) of planes ps bytes apart; an
  // accepted move of an earlier class waits among the sweep's proposals
  const uint32_t ys = (ky + K * a0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (kx + K * b0 + v.w * (R / v.w + 1) - R) % v.w;
  const char* src[G::NC];
  uint32_t ps[G::NC], prop[G::NC], moved[G::NC];
#pragma unroll
  for (int k = 0; k < G::NC; ++k) {
    const uint32_t u = min((w + G::NW * k) * 64 + lane, (uint32_t)(G::RH * G::RW) - 1);
    const uint32_t rr = u / G::RW, cc = u - rr * G::RW;
    uint32_t y = ys + rr, x = xs + cc;
    while (y >= v.h) y -= v.h;
    while (x >= v.w) x -= v.w;
    src[k] = (const char*)v.d8 + (size_t)(y * v.w + x) * 16;
    const uint32_t cls = (y % K) * K + x % K, j = (y / K) * v.cw + x / K;
    prop[k] = cls * v.pc * (v.tp >> 4) + j;
    moved[k] = cls < v.decided ? v.accepts[cls * v.pc + j] : 0u;
  }
#pragma unroll
  for (int k = 0; k < G::NC; ++k) {
    if (moved[k]) src[k] = (const char*)v.n8_sweep + (size_t)prop[k] * 16;
    ps[k] = (moved[k] ? v.pc : P) * 16;
  }
  // the class pixels' recounted words: wave w loads words 64 w .. of row
  // w mod BY (class pixels past the tile read pixel 0; their products are not
  // read back)
  const bool in = a0 + w % G::BY < v.ch && b0 + c16 < v.cw;
  const uint32_t nsrc = (g * v.pc + (in ? (a0 + w % G::BY) * v.cw + b0 + c16 : 0)) * 16;
  const uint32_t first = sb.first, last = sb.last;   // Tp is a multiple of 128, padded integrands are 0
  if (SLICED) {
#pragma unroll
    for (int k = 0; k < G::NC; ++k) src[k] += (size_t)first * 4 * ps[k];
  }
  auto issue = [&](uint32_t st, uint32_t buf) {   // stages in order
    const char* nb = (const char*)v.n8 + (size_t)st * 64 * v.pc;
    u32x4* to = lds4 + buf * G::STAGE;
#pragma unroll
    for (int k = 0; k < G::NC; ++k) {
      if (w + G::NW * k >= (uint32_t)G::CHUNKS) break;   // wave-uniform
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) {
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)src[k],
            (__attribute__((address_space(3))) void*)(to + pl * G::PLANE + 64 * (w + G::NW * k)), 16, 0, 0);
        src[k] += ps[k];
      }
    }
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(nb + nsrc),
                                     (__attribute__((address_space(3))) void*)(to + 4 * G::PLANE + 64 * (w % G::BY)),
                                     16, 0, 0);
  };

  i32x4 acc[G::NO][CT];
#pragma unroll
  for (int o = 0; o < G::NO; ++o)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[o][ct] = (i32x4){0, 0, 0, 0};
  int zn = 0, zo = 0;

  issue(first, 0);
  // words of the lane in a stage: its class pixel's, and column c16 of the
  // wave's first region row, in plane g
  const uint32_t nword = 4 * G::PLANE + 64 * m + lane, fword = g * G::PLANE + K * m * G::RW + c16;
  const uint32_t own = g * G::PLANE + (K * m + R) * G::RW + K * c16 + R;
  for (uint32_t st = first; st < last; ++st) {
    // stage st has landed in every wave, and the other half is read
    barrier_vm<0>();
    if (st + 1 < last) issue(st + 1, (st + 1 - first) & 1);
    const u32x4* bf = lds4 + ((st - first) & 1) * G::STAGE;
    const u32x4 cn = bf[nword], cp = bf[own];
    i32x4 an, am;   // A operands: dc, or f' and -f
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (FORM == FIELD_NARROW) {
        an[k] = (int)sub_bytes(cn[k], cp[k]);
      } else {
        an[k] = (int)cn[k];
        am[k] = (int)sub_bytes(0u, cp[k]);
      }
      zn = dot4(cn[k], cn[k], zn);
      zo = dot4(cp[k], cp[k], zo);
    }
#pragma unroll
    for (int rr = 0; rr < WS; ++rr) {
      const int o = rr < R ? R - rr : rr - R;
      if (S > 1 && o % S != (int)part) continue;   // wave-uniform
      i32x4 f[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) f[ct] = __builtin_bit_cast(i32x4, bf[fword + rr * G::RW + 16 * ct]);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        acc[o / S][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(an, f[ct], acc[o / S][ct], 0, 0, 0);
        if (FORM == FIELD_SPLIT)
          acc[o / S][ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(am, f[ct], acc[o / S][ct], 0, 0, 0);
      }
    }
  }
  barrier_vm<0>();   // the stages are read: their LDS now holds products and class sums
  int* prod = (int*)lds4;
  unsigned long long* sums = (unsigned long long*)((char*)lds4 + (4 * G::PROD + 15) / 16 * 16);
  for (uint32_t i = tid; i < (uint32_t)(NCLS + 1) * G::PX; i += 64 * G::NW) sums[i] = 0;
  // row 4 g + k, column 16 ct + c16 (pitch 4 past a multiple of 16: the four
  // row groups meet different banks)
#pragma unroll
  for (int o = 0; o < G::NO; ++o) {
    if (o * S + (int)part > R) continue;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        prod[((m * (R + 1) + o * S + part) * 16 + 4 * g + k) * G::PITCH + 16 * ct + c16] = acc[o][ct][k];
  }
  __syncthreads();
  if (part == 0) atomicAdd(&sums[NCLS * G::PX + 16 * m + c16], (unsigned long long)((long long)zn - zo));
  // window entries into classes: class pixel b of a row finds offset ox in
  // column K b + R + ox
  {
    constexpr uint32_t SHARE = 64 * G::NW / G::PX;   // threads per class pixel
    const uint32_t px = tid % G::PX, b = px & 15;
#pragma unroll
    for (uint32_t e0 = 0; e0 < (uint32_t)G::ENTRIES; e0 += SHARE) {
      const uint32_t e = e0 + tid / G::PX, o = e / WS, ox = e - o * WS;
      const int dx = (int)ox - R;
      if (o > (uint32_t)R || (o == 0 && dx == 0)) continue;
      // index of the class of squared distance d: the distances below it
      const int cl = v.dcls[dx * dx + (int)(o * o)];
      atomicAdd(&sums[cl * G::PX + px],
                (unsigned long long)(long long)prod[(((px >> 4) * (R + 1) + o) * 16 + b) * G::PITCH + K * b + ox]);
    }
  }
  __syncthreads();
  auto pixel = [&](uint32_t px) {
    const uint32_t a = a0 + (px >> 4), b = b0 + (px & 15);
    return a < v.ch && b < v.cw ? a * v.cw + b : v.pc;
  };
  if (SLICED && v.slices > 1) {
    store_slice<NCLS, G::PX>(v, sb.z, sums, 64 * G::NW, pixel);
    return;
  }
  if (tid >= (uint32_t)G::PX) return;
  const uint32_t j = pixel(tid);
  if (j == v.pc) return;
  const long long z = (long long)sums[NCLS * G::PX + tid];
  double sum = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    const long long x = (long long)WN.csize[c] * z - 2 * (long long)sums[c * G::PX + tid];
    sum = __dadd_rn(sum, __dmul_rn(v.wd[c], (double)x));
  }
  decide_move(v, kappa, j, (ky + K * (a0 + (tid >> 4))) * v.w + kx + K * (b0 + (tid & 15)), sum);
}

// One-dimensional grid of gx blocks a row, slice after slice, renumbered per XCD:
// an L2 then serves whole rows of blocks and their halos are read from memory once.
template <int FORM, int R, int K, bool SLICED>
__global__ __launch_bounds__(64 * (GramGeom<R, K>::NW)) void k_gram(DevView v, uint32_t kappa, uint32_t gx) {
  // the colour phases' waves issue ahead of the sweep-wide recount running
  // beside them (k_commit and the BF16 form's kernels likewise), which fills
  // the remaining issue slots
  __builtin_amdgcn_s_setprio(2);
  gram_body<FORM, R, K, SLICED>(v, kappa, SliceBlock<SLICED>(v, xcd_block(blockIdx.x, gridDim.x), gridDim.x), gx);
}

// Batched form: member i owns blocks pre[i] .. pre[i+1]-1, laid out as its own
// grid.
template <int FORM, int R, int K, bool SLICED>
__global__ __launch_bounds__(64 * (GramGeom<R, K>::NW)) void k_gram_batch(const DevView* __restrict__ views,
                                                                          const uint32_t* __restrict__ pre,
                                                                          uint32_t nmem, uint32_t kappa) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t wk = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t i = batch_member(pre, nmem, wk);
  const DevView v = views[i];
  gram_body<FORM, R, K, SLICED>(v, kappa, SliceBlock<SLICED>(v, wk - pre[i], SLICED ? pre[i + 1] - pre[i] : 0),
                                (v.cw + 15) / 16);
}

// Raises the LDS launch limit (gfx950 has 160 KiB per CU), once per kernel.
template <class F>
hipError_t gram_lds(F kernel, int bytes) {
  return bytes > 65536 ? hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)
                       : hipSuccess;
}

}  // namespace

// The entry points of one form (one source each).
#define BN_GRAM_FORM(FORM, NAME)                                                                                       \
  hipError_t launch_phase_##NAME(const DevView& v, uint32_t kappa, hipStream_t s) {                                    \
    const hipError_t e = by_radius_k(v.radius, v.k, [&](auto r, auto k) {                                              \
      using G = GramGeom<r(), k()>;                                                                                    \
      auto launch = [&](auto sliced) {                                                                                 \
        static const hipError_t ready = gram_lds(k_gram<FORM, r(), k(), sliced()>, G::LDS_BYTES);                      \
        if (ready != hipSuccess) return ready;                                                                         \
        hipLaunchKernelGGL((k_gram<FORM, r(), k(), sliced()>), dim3(phase_blocks_##NAME(v)), dim3(64 * G::NW),         \
                           (size_t)G::LDS_BYTES, s, v, kappa, (v.cw + 15) / 16);                                       \
        return hipGetLastError();                                                                                      \
      };                                                                                                               \
      return v.slices > 1 ? launch(std::true_type()) : launch(std::false_type());                                      \
    });                                                                                                                \
    return e != hipSuccess || v.slices == 1 ? e : launch_phase_decide(v, kappa, s);                                    \
  }                                                                                                                    \
  hipError_t launch_phase_batch_##NAME(uint32_t radius, uint32_t k, bool sliced, const DevView* views,                 \
                                       const uint32_t* pre, uint32_t nmem, uint32_t blocks, uint32_t kappa,            \
                                       hipStream_t s) {                                                                \
    return by_radius_k(radius, k, [&](auto r, auto kk) {                                                               \
      using G = GramGeom<r(), kk()>;                                                                                   \
      auto launch = [&](auto sl) {                                                                                     \
        static const hipError_t ready = gram_lds(k_gram_batch<FORM, r(), kk(), sl()>, G::LDS_BYTES);                   \
        if (ready != hipSuccess) return ready;                                                                         \
        hipLaunchKernelGGL((k_gram_batch<FORM, r(), kk(), sl()>), dim3(blocks), dim3(64 * G::NW),                      \
                           (size_t)G::LDS_BYTES, s, views, pre, nmem, kappa);                                          \
        return hipGetLastError();                                                                                      \
      };                                                                                                               \
      return sliced ? launch(std::true_type()) : launch(std::false_type());                                            \
    });                                                                                                                \
  }                                                                                                                    \
  uint32_t phase_blocks_##NAME(const DevView& v) {                                                                     \
    uint32_t rows = 1;                                                                                                 \
    (void)by_radius_k(v.radius, v.k, [&](auto r, auto k) {                                                             \
      rows = (uint32_t)GramGeom<r(), k()>::BY;                                                                         \
      return hipSuccess;                                                                                               \
    });                                                                                                                \
    return ((v.cw + 15) / 16) * ((v.ch + rows - 1) / rows) * v.slices;                                                 \
  }

}  // namespace bnlat
