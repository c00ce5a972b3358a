// gfx950 energy change and decision of one colour phase on the uint16 counts,
// by the vector ALUs: the FP32 form where no int8 field is known to hold the
// counts (phase_gram.h), and the approximate BF16 form's re-evaluation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

// A workgroup owns a block of 8 x 8 class pixels and every integrand: it ends
// with their whole class sums and decides them.  A 16-byte word of integrands
// of the block is one wave's (K = 4) or half a wave's work (K = 1, 2, where a
// thread owns V = 2 vertically adjacent class pixels, whose windows overlap, so
// that each field word it reads from LDS serves both); W words are in work at
// a time.  A wave copies the words it evaluates, the block plus the window
// halo (RH x RW pixels each), into LDS planes of its own through registers,
// loading the next words before it evaluates the current ones where their
// registers fit: no barrier is needed until the end, and the waves of a CU overlap their loads, LDS traffic
// and arithmetic freely.
//
// A plane groups its columns by residue mod K, so the 8 lanes of a class row
// read 8 consecutive words for every window offset, each with one ds_read_b128
// at a compile-time offset from the thread's base; its row pitch puts the next
// class row of the thread grid 8 words further modulo 16, and planes are whole
// multiples of 16 words, so the 16 lanes of an LDS pass meet 16 distinct bank
// quads and the four passes of a wave agree modulo 256 bytes.
//
// Whole sums in one workgroup cost more halo (2.1 times the tile through L2 in
// place of 1.35 with 32 x 16 class pixels and a slice of the integrands), but
// need no 64-bit atomics, which all go to memory on this part: measured on the
// int8 field at 256^2, T = 1024, r = 4, 30 us per phase, decision included,
// against 42.  Bound by the vector ALUs (14 us of v_dot2 at twice that field's
// bytes) and latency.
template <int R, int K>
struct PhaseGeom {
  static constexpr int NCLS = WinConst<R>::NCLS;
  static constexpr int V = (K == 4) ? 1 : 2;                       // class pixels per thread
  static constexpr int TPW = 64 / V;                               // threads per word
  static constexpr int RH = 7 * K + 2 * R + 1, RW = RH;            // region pixels
  static constexpr int RWK = (RW + K - 1) / K;
  static constexpr int pitch() {
    int p = RWK * K;
    while ((K * V * p) % 16 != 8) ++p;
    return p;
  }
  static constexpr int RWP = pitch();                              // words per plane row
  static constexpr int PLANE = (RH * RWP + 15) / 16 * 16;
  static constexpr int SUMS = (NCLS + 1) * 64;                     // int64 class sums and self terms
  // words in work: at most 8 (more left the
  // recount beside it no registers), within the CU's 160 KiB of LDS
  static constexpr int words_in(int bytes) {
    const int n = (bytes - 8 * SUMS) / (16 * PLANE);
    return V == 2 ? n / 2 * 2 : n;
  }
  static constexpr int FIT = words_in(163840);
  static constexpr int W = FIT < 8 ? FIT : 8;
  static constexpr int NT = W * TPW;
  static constexpr int LDS_BYTES = 8 * SUMS + 16 * PLANE * W;
  static constexpr int ITER = (RH * RW + TPW - 1) / TPW;           // words a thread copies
  static constexpr int DR = K * (V - 1) + 2 * R + 1;               // plane rows a thread reads
  // the next words are loaded ahead where their registers fit (about 80 beyond
  // those counted here, found by compiling; 256 at two waves per SIMD)
  static constexpr bool AHEAD = 6 * ITER + V * NCLS + 4 * (2 * R + 1) + (V == 2 ? 84 : 66) <= 254;
  // word of region column K tx + R + ox relative to that of column K tx
  static constexpr int dcol(int ox) { return ((R + ox) % K) * RWK + (R + ox) / K; }
  static_assert(W >= 1 && NT <= 1024 && NT % 64 == 0, "phase block geometry");
};

// Count changes of a 16-byte word (8 integrands) as four int16 pairs, and
// sum_t dc_t (c'_t + c_t) over the word.
__device__ __forceinline__ int stage_dc(const u32x4 cn, const u32x4 co, uint32_t d[4]) {
  int z = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int n0 = (int)(cn[k] & 0xFFFFu), n1 = (int)(cn[k] >> 16);
    const int o0 = (int)(co[k] & 0xFFFFu), o1 = (int)(co[k] >> 16);
    d[k] = ((uint32_t)(n0 - o0) & 0xFFFFu) | ((uint32_t)(n1 - o1) << 16);
    z += (n0 - o0) * (n0 + o0) + (n1 - o1) * (n1 + o1);
  }
  return z;
}

template <int R, int K, bool SLICED>
__device__ __forceinline__ void phase_body(const DevView& v, uint32_t kappa, uint32_t span, const SliceBlock<SLICED> sb,
                                           uint32_t bgx) {
  using G = PhaseGeom<R, K>;
  constexpr Window<R> WN = WinConst<R>::w;
  constexpr int NCLS = G::NCLS, V = G::V, WS = 2 * R + 1;
  constexpr uint32_t IPW = 8;   // integrands per word
  extern __shared__ u32x4 lds4[];
  unsigned long long* sums = (unsigned long long*)lds4;            // [NCLS + 1][64]
  const uint32_t tid = threadIdx.x, lane = tid % G::TPW, slot = tid / G::TPW;
  u32x4* reg = lds4 + G::SUMS / 2 + slot * G::PLANE;
  const uint32_t tx = lane & 7, ty = lane >> 3;
  const uint32_t a0 = sb.b / bgx * 8, b0 = sb.b % bgx * 8;
  const uint32_t ky = kappa / K, kx = kappa - ky * K;
  // top-left region pixel, made non-negative modulo the tile
  const uint32_t ys = (ky + K * a0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (kx + K * b0 + v.w * (R / v.w + 1) - R) % v.w;
  const uint32_t P = v.w * v.h;
  for (uint32_t i = tid; i < (uint32_t)G::SUMS; i += G::NT) sums[i] = 0;

  // region pixels of the thread: the same for every word.  Threads past the
  // region load pixel 0 and do not store it.
  uint32_t poff[G::ITER], wi[G::ITER];
#pragma unroll
  for (int it = 0; it < G::ITER; ++it) {
    const uint32_t i = lane + it * G::TPW;
    const uint32_t rr = i / G::RW, cc = i - rr * G::RW;
    uint32_t gy = ys + rr, gx = xs + cc;
    while (gy >= v.h) gy -= v.h;
    while (gx >= v.w) gx -= v.w;
    const bool in = i < (uint32_t)(G::RH * G::RW);
    poff[it] = in ? (gy * v.w + gx) * 16 : 0;
    wi[it] = in ? rr * G::RWP + (cc % K) * G::RWK + cc / K : 0xFFFFFFFFu;
  }
  uint32_t coff[V];
#pragma unroll
  for (int vv = 0; vv < V; ++vv) {
    const uint32_t a = a0 + ty * V + vv, b = b0 + tx;
    coff[vv] = (a < v.ch && b < v.cw) ? (a * v.cw + b) * 16 : 0;
  }
  const uint32_t top = K * ty * V * G::RWP + tx;

  int z0[V], part[V][NCLS];
  auto clear = [&]() {
#pragma unroll
    for (int vv = 0; vv < V; ++vv) {
      z0[vv] = 0;
#pragma unroll
      for (int c = 0; c < NCLS; ++c) part[vv][c] = 0;
    }
  };
  auto flush = [&]() {
#pragma unroll
    for (int vv = 0; vv < V; ++vv) {
      unsigned long long* s = sums + (ty * V + vv) * 8 + tx;
#pragma unroll
      for (int c = 0; c < NCLS; ++c) atomicAdd(s + c * 64, (unsigned long long)(long long)part[vv][c]);
      atomicAdd(s + NCLS * 64, (unsigned long long)(long long)z0[vv]);
    }
  };
  clear();

  const char* fld = (const char*)v.cnt;
  const char* nfl = (const char*)v.c_new;
  // words of the slice: up to `words`
  const uint32_t from = sb.first * (64 / IPW), words = min(sb.last * (64 / IPW), (v.t + IPW - 1) / IPW);
  u32x4 q[G::ITER], qc[V];
  // words past the last repeat it (and count nothing)
  auto issue = [&](uint32_t word) {
    const uint32_t wd = min(word, words - 1);
    const char* cs = fld + (size_t)wd * P * 16;
    const char* ns = nfl + (size_t)wd * v.pc * 16;
#pragma unroll
    for (int it = 0; it < G::ITER; ++it) q[it] = *(const u32x4*)(cs + poff[it]);
#pragma unroll
    for (int vv = 0; vv < V; ++vv) qc[vv] = *(const u32x4*)(ns + coff[vv]);
  };
  // first word of the wave: uniform, so the loop is
  const uint32_t first = __builtin_amdgcn_readfirstlane(slot);
  if (G::AHEAD) issue(from + slot);
  __syncthreads();   // the sums are cleared
  uint32_t since = 0;
  for (uint32_t wd = from + first; wd < words; wd += G::W) {
    const uint32_t word = wd + (slot - first);
    if (!G::AHEAD) issue(word);
#pragma unroll
    for (int it = 0; it < G::ITER; ++it)
      if (wi[it] != 0xFFFFFFFFu) reg[wi[it]] = q[it];
    u32x4 cn[V];
#pragma unroll
    for (int vv = 0; vv < V; ++vv) cn[vv] = qc[vv];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (G::AHEAD && wd + G::W < words) issue(word + G::W);
    uint32_t d[V][4];
#pragma unroll
    for (int vv = 0; vv < V; ++vv) {
      u32x4 co = reg[top + (R + K * vv) * G::RWP + G::dcol(0)];
      if (word >= words) co = cn[vv] = (u32x4){0, 0, 0, 0};
      z0[vv] += stage_dc(cn[vv], co, d[vv]);
    }
#pragma unroll
    for (int dr = 0; dr < G::DR; ++dr) {
      // a row's words are loaded together, so their LDS latencies overlap
      u32x4 row[WS];
#pragma unroll
      for (int ox = -R; ox <= R; ++ox) row[ox + R] = reg[top + dr * G::RWP + G::dcol(ox)];
#pragma unroll
      for (int ox = -R; ox <= R; ++ox) {
        const u32x4 f = row[ox + R];
#pragma unroll
        for (int vv = 0; vv < V; ++vv) {
          const int oy = dr - R - K * vv;
          if (oy < -R || oy > R || (ox == 0 && oy == 0)) continue;
          const int c = WN.cmap[(oy + R) * WS + ox + R];
          int x = part[vv][c];
          x = dot2(d[vv][0], f[0], x);
          x = dot2(d[vv][1], f[1], x);
          x = dot2(d[vv][2], f[2], x);
          part[vv][c] = dot2(d[vv][3], f[3], x);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (++since == span) {
      flush();
      clear();
      since = 0;
    }
  }
  flush();
  __syncthreads();

  auto pixel = [&](uint32_t px) {
    const uint32_t a = a0 + (px >> 3), b = b0 + (px & 7);
    return a < v.ch && b < v.cw ? a * v.cw + b : v.pc;
  };
  if (SLICED && v.slices > 1) {
    store_slice<NCLS, 64>(v, sb.z, sums, G::NT, pixel);
    return;
  }
  // decision, a lane of the first wave per class pixel: one FP64 weighted sum
  // of the exact class sums in increasing distance
  if (tid >= 64) return;
  const uint32_t j = pixel(tid);
  if (j == v.pc) return;
  if (v.mfma && !v.accept[j]) return;
  const long long z = (long long)sums[NCLS * 64 + tid];
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    const long long x = (long long)WN.csize[c] * z - 2 * (long long)sums[c * 64 + tid];
    acc = __dadd_rn(acc, __dmul_rn(v.wd[c], (double)x));
  }
  decide_move(v, kappa, j, (ky + K * (a0 + (tid >> 3))) * v.w + kx + K * (b0 + (tid & 7)), acc);
}

// One-dimensional grid of gx blocks a row, slice after slice, renumbered per XCD:
// an L2 then serves whole rows of blocks and their halos are read from memory once.
template <int R, int K, bool SLICED>
__global__ __launch_bounds__((PhaseGeom<R, K>::NT)) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_phase(DevView v, uint32_t kappa, uint32_t span, uint32_t gx) {
  // the colour phases' waves issue ahead of the sweep-wide recount running
  // beside them (k_commit and the BF16 form's kernels likewise), which fills
  // the remaining issue slots
  __builtin_amdgcn_s_setprio(2);
  phase_body<R, K, SLICED>(v, kappa, span, SliceBlock<SLICED>(v, xcd_block(blockIdx.x, gridDim.x), gridDim.x), gx);
}

// Batched form: member i owns blocks pre[i] .. pre[i+1]-1, laid out as its own
// grid.
template <int R, int K, bool SLICED>
__global__ __launch_bounds__((PhaseGeom<R, K>::NT)) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_phase_batch(const DevView* __restrict__ views,
                                                                     const uint32_t* __restrict__ pre, uint32_t nmem,
                                                                     uint32_t kappa) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t wk = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t i = batch_member(pre, nmem, wk);
  const DevView v = views[i];
  phase_body<R, K, SLICED>(v, kappa, v.span, SliceBlock<SLICED>(v, wk - pre[i], SLICED ? pre[i + 1] - pre[i] : 0),
                           (v.cw + 7) / 8);
}

// Raises the LDS launch limit (gfx950 has 160 KiB per CU), once per kernel.
template <class F>
hipError_t phase_lds(F kernel, int bytes) {
  return bytes > 65536 ? hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)
                       : hipSuccess;
}

template <int R, int K, bool SLICED>
hipError_t phase_rk(const DevView& v, uint32_t kappa, hipStream_t s) {
  using G = PhaseGeom<R, K>;
  static const hipError_t ready = phase_lds(k_phase<R, K, SLICED>, G::LDS_BYTES);
  if (ready != hipSuccess) return ready;
  const uint32_t gx = (v.cw + 7) / 8;
  hipLaunchKernelGGL((k_phase<R, K, SLICED>), dim3(phase_blocks_wide(v)), dim3(G::NT), (size_t)G::LDS_BYTES, s, v, kappa,
                     v.span, gx);
  return hipGetLastError();
}

template <int R, int K, bool SLICED>
hipError_t phase_batch_rk(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks, uint32_t kappa,
                          hipStream_t s) {
  using G = PhaseGeom<R, K>;
  static const hipError_t ready = phase_lds(k_phase_batch<R, K, SLICED>, G::LDS_BYTES);
  if (ready != hipSuccess) return ready;
  hipLaunchKernelGGL((k_phase_batch<R, K, SLICED>), dim3(blocks), dim3(G::NT), (size_t)G::LDS_BYTES, s, views, pre, nmem,
                     kappa);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_phase_wide(const DevView& v, uint32_t kappa, hipStream_t s) {
  const hipError_t e = by_radius_k(v.radius, v.k, [&](auto r, auto k) {
    return v.slices > 1 ? phase_rk<r(), k(), true>(v, kappa, s) : phase_rk<r(), k(), false>(v, kappa, s);
  });
  return e != hipSuccess || v.slices == 1 ? e : launch_phase_decide(v, kappa, s);
}

hipError_t launch_phase_batch_wide(uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                                   uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s) {
  return by_radius_k(radius, k, [&](auto r, auto kk) {
    return sliced ? phase_batch_rk<r(), kk(), true>(views, pre, nmem, blocks, kappa, s)
                  : phase_batch_rk<r(), kk(), false>(views, pre, nmem, blocks, kappa, s);
  });
}

uint32_t phase_blocks_wide(const DevView& v) { return ((v.cw + 7) / 8) * ((v.ch + 7) / 8) * v.slices; }

// Words of 8 integrands whose class sums fit int32: every product dc_t c_q,t is
// at most N^2 and a class has at most 12 offsets for radii up to 6.
uint32_t phase_span_wide(uint32_t n) { return (uint32_t)std::max<uint64_t>(1, 0x7FFFFFFFull / (96ull * n * n)); }

}  // namespace bnlat
