// gfx950 kernels of the screen-space lattice-offset optimiser.
//
// Data layout in HBM (P = W*H pixels, Tp = T rounded up to 128):
//   U    uint32 [P]        offset of pixel p = y*W + x, Q0.16 x | y << 16
//   cnt  uint16 [Tp/8][P][8] hit counts in 16-byte integrand tiles: the 8
//                          counts of integrands 8i..8i+7 of a pixel are
//                          contiguous and neighbouring pixels' tiles are
//                          adjacent, so a row of pixels for 8 integrands is
//                          one contiguous run
//   err  float  [P][Tp]    error vectors c/N - A_t (refreshed from the counts
//                          when read)
//   lat  uint32 [N]        rank-1 lattice points (Sec. 3.2), x | y << 16
//   ihp  int2   [Tp]       Heaviside (n packed as two int16, D' = n.(C - 2^15))
//   gest float  [P][TGp]   Gaussian estimates (TGp = Gaussian count rounded
//                          up to 64; padded rows evaluate exp(0) = 1)
// Side buffers of one colour phase (M class pixels): u_new [M],
// c_new [Tp/8][M][8] (same tiling), delta [M], accept [M].
//
// All arithmetic that decides anything is exact: sample coordinates are
// Q0.16, the Heaviside predicate n.(S - 2^15) > D' is an int16 dot product
// against an int32 threshold, and the energy change is assembled from
// integer class sums before one FP64 weighted sum in a fixed order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

// ------------------------------------------------------------ energy change
//
// Energy change of one pixel's move (Eq. (1) over the window, both pair
// orderings):  dE = (2/N^2) sum_d w(d) X_d,
//   X_d = |class d| * Z0 - 2 Z_d,  Z0 = sum_t dc_t (c'_t + c_t),
//   Z_d = sum_{o in class d} sum_t dc_t c_{p+o,t},  dc = c' - c,
// all in exact integers.  One wave per moved pixel: lane (i, q) takes the i-th
// offset of each step (WindowSteps: eight consecutive offsets of a window row,
// or of a column that those leave over) and plane q of 64 integrands, so that a
// load reads whole lines of eight planes; a word is 8 integrands, four v_dot2.
// The steps' sums meet by class in LDS.  Used for explicit pixel lists and
// colourings without a phase kernel.  Bound by the latency of a moved pixel's
// serial planes and the L2s' reads.  2000 moves at T = 1024, r = 4: 71 us; 195
// with a lane per integrand pair (a load touched 16 lines for 256 bytes), 213 to
// 265 with a lane per word (64 lines for 1 KiB).
template <int R, int MODE>
__global__ __launch_bounds__(256) void k_delta(DevView v, uint32_t kappa, uint32_t m) {
  using S = WindowSteps<R>;
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  static_assert(NCLS < 64, "a lane per class");
  __shared__ unsigned long long sums[4][NCLS + 1];
  const uint32_t lane = threadIdx.x & 63, wl = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t j = wave_id();
  if (j >= m) return;
  const uint32_t p = (MODE == MODE_CLASS) ? class_pixel(v, kappa, j) : v.pix_list[j];
  const uint32_t y = p / v.w, x = p - y * v.w, i = lane & 7, P = v.w * v.h;
  uint32_t q[S::STEPS];
  int cl[S::STEPS];
#pragma unroll
  for (int st = 0; st < S::STEPS; ++st) {
    int ox, oy;
    const bool in = S::offset(st, (int)i, ox, oy) && (ox || oy);
    cl[st] = in ? v.dcls[ox * ox + oy * oy] : -1;
    q[st] = in ? (y + v.h * (R / v.h + 1) + oy) % v.h * v.w + (x + v.w * (R / v.w + 1) + ox) % v.w : p;
  }
  if (lane <= (uint32_t)NCLS) sums[wl][lane] = 0;
  long long z0 = 0, zd[S::STEPS];
#pragma unroll
  for (int st = 0; st < S::STEPS; ++st) zd[st] = 0;
  const u32x4* nw = (const u32x4*)v.c_new + (size_t)(lane >> 3) * m + j;
  const u32x4* plane = (const u32x4*)v.cnt + (size_t)(lane >> 3) * P;
  for (uint32_t t = 0; t < v.tp; t += 64, nw += (size_t)8 * m, plane += (size_t)8 * P) {
    const u32x4 cn = *nw, co = plane[p];
    u32x4 c[S::STEPS];
#pragma unroll
    for (int st = 0; st < S::STEPS; ++st) c[st] = plane[q[st]];
    uint32_t dc[4];
    int z = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int n0 = (int)(cn[k] & 0xFFFFu), n1 = (int)(cn[k] >> 16);
      const int o0 = (int)(co[k] & 0xFFFFu), o1 = (int)(co[k] >> 16);
      const int dc0 = n0 - o0, dc1 = n1 - o1;
      dc[k] = ((uint32_t)dc0 & 0xFFFFu) | ((uint32_t)dc1 << 16);
      z += dc0 * (n0 + o0) + dc1 * (n1 + o1);
    }
    z0 += z;
#pragma unroll
    for (int st = 0; st < S::STEPS; ++st) {
      int part = 0;   // |part| <= 8 N^2
#pragma unroll
      for (int k = 0; k < 4; ++k) part = dot2(dc[k], c[st][k], part);
      zd[st] += part;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int st = 0; st < S::STEPS; ++st)
    if (cl[st] >= 0) atomicAdd(&sums[wl][cl[st]], (unsigned long long)zd[st]);
  if (i == 0) atomicAdd(&sums[wl][NCLS], (unsigned long long)z0);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const long long z = (long long)sums[wl][NCLS];
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    const long long xv = (long long)W.csize[c] * z - 2 * (long long)sums[wl][c];
    acc = __dadd_rn(acc, __dmul_rn(v.wd[c], (double)xv));
  }
  if (lane == 0) {
    double total = __dmul_rn(acc, 2.0 / ((double)v.n * (double)v.n));
    if (v.tgp) total = __dadd_rn(total, v.gdelta[j]);
    v.delta[j] = total;
    v.accept[j] = (v.objective > 0) ? (total < 0.0) : (total > 0.0);
  }
}

// Decide from the BF16 pass's class sums (one thread per pixel) and clear them.
__global__ __launch_bounds__(256) void k_delta_finish(DevView v) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= v.pc) return;
  double acc = 0.0;
  for (uint32_t c = 0; c < v.ncls; ++c) {
    const long long x = v.xpart[(size_t)c * v.pc + j];
    v.xpart[(size_t)c * v.pc + j] = 0;
    acc = __dadd_rn(acc, __dmul_rn(v.wd[c], (double)x));
  }
  double total = __dmul_rn(acc, v.xscale);
  // the approximate form's class sums already hold the Gaussian rows
  if (v.tgp && v.mfma != 2) total = __dadd_rn(total, v.gdelta[j]);
  v.delta[j] = total;
  v.delta_bf[j] = total;
  v.accept[j] = (v.objective > 0) ? (total < 0.0) : (total > 0.0);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ commit
// Accepted moves of the phase become the state (Sec. 3.4): offset and hit
// counts of the pixel (error vectors are refreshed from the counts on
// demand).
//
// A workgroup owns 64 class pixels and its waves their rows' words, a 16-byte
// word per lane, pixels fastest, so that the proposal rows are read coalesced.
// Few moves are accepted after the first sweeps: bound by the latency of the
// decision's and then the rows' loads, hence many waves with few words each
// (10 us a class at 256^2, N = 256, T = 1024 beside the recount, 19 for all four
// of a sweep in one launch; committing the class
// before inside the next phase kernel kept the recount off the CUs: 351 against
// 275 us per two sweeps).
constexpr uint32_t COMMIT_WAVES = 16;

__device__ __forceinline__ void commit_body(const DevView& v, uint32_t kappa, uint32_t blk, bool advance) {
  const uint32_t lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t j = blk * 64 + lane;
  const bool acc = j < v.pc && v.accept[j];
  const uint32_t p = class_pixel(v, kappa, j);
  if (w == 0) {
    const unsigned long long m = __ballot(acc);
    if (lane == 0 && m) atomicAdd(&v.ctr[1], (unsigned long long)__popcll(m));
    if (lane == 0 && advance && blk == 0) atomicAdd(&v.ctr[0], 1ull);
    if (acc) v.U[p] = v.u_new[j];
    if (acc && v.seen) v.seen[p] = v.u_new[j];
  }
  if (!acc) return;
  const size_t P = (size_t)v.w * v.h;
  if (v.form != FIELD_WIDE) {
    const uint32_t words = (v.t + 15) >> 4;
#pragma unroll 4
    for (uint32_t tt = w; tt < words; tt += COMMIT_WAVES) {
      const u32x4 d = *(const u32x4*)(v.n8 + ((size_t)tt * v.pc + j) * 16);
      *(u32x4*)(v.d8 + (tt * P + p) * 16) = d;
      uint4 lo, hi;
      widen8(d, v.bias8 + 8 * tt, lo, hi);
      *(uint4*)(v.cnt + (2 * tt * P + p) * 8) = lo;
      *(uint4*)(v.cnt + ((2 * tt + 1) * P + p) * 8) = hi;
    }
  } else {
    const uint32_t words = (v.t + 7) >> 3;
#pragma unroll 4
    for (uint32_t tt = w; tt < words; tt += COMMIT_WAVES) {
      const uint4 c8 = *(const uint4*)(v.c_new + ((size_t)tt * v.pc + j) * 8);
      *(uint4*)(v.cnt + (tt * P + p) * 8) = c8;
      if (v.bf) *(uint4*)(v.bf + (tt * P + p) * 8) = heaviside_field_tile(v, c8, tt * 8);
    }
  }
}

// FP32 error vectors e = c/N - A_t of every pixel from the exact counts
// (refreshed on demand; thread per (integrand tile, pixel), pixels fastest).
__global__ __launch_bounds__(256) void k_errors(DevView v) {
  const uint32_t P = v.w * v.h;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)P * (v.tp >> 3)) return;
  const uint32_t tt = (uint32_t)(i / P), p = (uint32_t)(i - (size_t)tt * P);
  const uint4 c8 = *(const uint4*)(v.cnt + i * 8);
  const uint32_t t = tt * 8;
  const float inv_n = 1.0f / (float)v.n;
  const float4 a = *(const float4*)(v.area + t), b = *(const float4*)(v.area + t + 4);
  float4 lo, hi;
  lo.x = (float)(c8.x & 0xFFFFu) * inv_n - a.x;
  lo.y = (float)(c8.x >> 16) * inv_n - a.y;
  lo.z = (float)(c8.y & 0xFFFFu) * inv_n - a.z;
  lo.w = (float)(c8.y >> 16) * inv_n - a.w;
  hi.x = (float)(c8.z & 0xFFFFu) * inv_n - b.x;
  hi.y = (float)(c8.z >> 16) * inv_n - b.y;
  hi.z = (float)(c8.w & 0xFFFFu) * inv_n - b.z;
  hi.w = (float)(c8.w >> 16) * inv_n - b.w;
  float* e = v.err + (size_t)p * v.tp + t;
  *(float4*)e = lo;
  *(float4*)(e + 4) = hi;
}

// Error rows first .. as the caller reads them, [n][t + tg]: the padding of the
// rows in memory would make the transfer to the host one copy per row (54 ms
// for 4096 rows, where one copy of the packed rows takes under 1).
__global__ __launch_bounds__(256) void k_pack_errors(DevView v, uint32_t first, uint32_t n, float* __restrict__ out) {
  const uint32_t row = v.t + v.tg;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (uint64_t)n * row) return;
  const uint32_t r = (uint32_t)(i / row), c = (uint32_t)(i - (uint64_t)r * row);
  const size_t p = (size_t)first + r;
  out[i] = c < v.t ? v.err[p * v.tp + c] : v.gerr[p * v.tgp + c - v.t];
}

__global__ __launch_bounds__(64 * COMMIT_WAVES) void k_commit(DevView v, uint32_t kappa, bool advance) {
  __builtin_amdgcn_s_setprio(2);
  commit_body(v, kappa, blockIdx.x, advance);
}

__global__ __launch_bounds__(64 * COMMIT_WAVES) void k_commit_batch(const DevView* __restrict__ views,
                                                                    const uint32_t* __restrict__ pre, uint32_t nmem,
                                                                    uint32_t kappa) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  const DevView v = views[i];
  commit_body(v, kappa, blockIdx.x - pre[i], false);
}

// All classes' moves of a sweep whose phases left them waiting.
__device__ __forceinline__ void commit_sweep_body(DevView v, uint32_t blk, bool advance) {
  const uint32_t per = (v.pc + 63) / 64, kappa = blk / per;
  v.n8 += (size_t)kappa * v.pc * v.tp;
  v.u_new += (size_t)kappa * v.pc;
  v.accept = v.accepts + (size_t)kappa * v.pc;
  commit_body(v, kappa, blk - kappa * per, advance && kappa == 0);
}

__global__ __launch_bounds__(64 * COMMIT_WAVES) void k_commit_sweep(DevView v, bool advance) {
  __builtin_amdgcn_s_setprio(2);
  commit_sweep_body(v, blockIdx.x, advance);
}

__global__ __launch_bounds__(64 * COMMIT_WAVES) void k_commit_sweep_batch(const DevView* __restrict__ views,
                                                                          const uint32_t* __restrict__ pre,
                                                                          uint32_t nmem) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  commit_sweep_body(views[i], blockIdx.x - pre[i], false);
}

// A caller that owns offsets and counts may have put another state of the problem
// there: the words of d8 of the pixels whose offset is not the one they were
// written for, from the counts.  A pixel's counts follow from its offset, so
// comparing those (8 bytes a pixel) finds the ones to read: 4 us a call of two
// sweeps where nothing was replaced (10 in a batch of 32 tiles of 64^2 and 128^2);
// reading every count would take 45 at 256^2, T = 1024.
constexpr uint32_t FOLLOW_PIXELS = 256;   // of a workgroup at a time

__device__ __forceinline__ void follow_body(const DevView& v, uint32_t blk, uint32_t nblk) {
  const uint32_t lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), P = v.w * v.h;
  constexpr int N = FOLLOW_PIXELS / 64;
  for (uint32_t p0 = blk * FOLLOW_PIXELS; p0 < P; p0 += nblk * FOLLOW_PIXELS) {
    uint32_t u[N];
    bool changed[N], any = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t p = p0 + 64 * i + lane;
      u[i] = p < P ? v.U[p] : 0;
      changed[i] = p < P && u[i] != v.seen[p];
      any = any || changed[i];
    }
    if (!__syncthreads_or(any)) continue;   // (every wave has read seen)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t p = p0 + 64 * i + lane;
      if (!changed[i]) continue;
      for (uint32_t tt = w; tt < v.tp >> 4; tt += 4)
        *(u32x4*)(v.d8 + ((size_t)tt * P + p) * 16) =
            narrow8(*(const uint4*)(v.cnt + ((size_t)(2 * tt) * P + p) * 8),
                    *(const uint4*)(v.cnt + ((size_t)(2 * tt + 1) * P + p) * 8), v.bias8 + 8 * tt);
      if (w == 0) v.seen[p] = u[i];
    }
  }
}

__global__ __launch_bounds__(256) void k_follow(DevView v) { follow_body(v, blockIdx.x, gridDim.x); }

__global__ __launch_bounds__(256) void k_follow_batch(const DevView* __restrict__ views, const uint32_t* __restrict__ pre,
                                                      uint32_t nmem) {
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  const DevView v = views[i];
  if (v.seen) follow_body(v, blockIdx.x - pre[i], pre[i + 1] - pre[i]);
}

__global__ void k_advance(unsigned long long* ctr) {
  if (threadIdx.x == 0 && blockIdx.x == 0) atomicAdd(&ctr[0], 1ull);
}

// The overlapped schedule's recount index (counter word 3) one past the sweep
// counter, and its advance by a pair of sweeps.
__global__ void k_recount_index(unsigned long long* ctr) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctr[3] = ctr[0] + 1ull;
}

__global__ void k_recount_advance_pair(unsigned long long* ctr) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctr[3] += 2ull;
}

__global__ void k_advance_batch(const DevView* __restrict__ views, uint32_t nmem) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nmem) atomicAdd(&views[i].ctr[0], 1ull);
}

__global__ __launch_bounds__(256) void k_init_offsets(DevView v) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= v.w * v.h) return;
  v.U[p] = q16_pair(philox_w01(p, 0, v.problem, S_INIT, v.seed_lo, v.seed_hi));
}

// The N samples of one pixel in van der Corput order: s^k = L(bitrev_m(k)).
__global__ void k_points(DevView v, uint32_t pixel, uint32_t* out) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= v.n) return;
  const uint32_t i = v.log2n ? (__brev(k) >> (32 - v.log2n)) : 0u;
  out[k] = wrap_add(v.lat[i], v.U[pixel]);
}

// ------------------------------------------------------------------ energy
// Y_d = sum_{o in class d} sum_p sum_t (c_p - c_{p+o})^2 over the half window
// (the other half gives the same total).  Lanes run over 64 consecutive
// pixels of a row, so every 16-byte tile load of a wave (8 integrands of 64
// neighbouring pixels) is one contiguous 1 KiB run; per tile a lane's int32
// partial sums (at most 12 offsets x 8 integrands x N^2 < 2^31) are widened
// to 64 bits.  A workgroup takes 256 pixels and a share of the tiles (64-bit
// atomics to one address follow one another, so each share has a row of sums
// of its own modulo ENERGY_ROWS).  Bound by the L1s' reads of the neighbours'
// tiles.  128^2, T = 1024, r = 3: 67 us; 498 with all tiles in one
// workgroup per 256 pixels (64 of them), differences formed from unpacked
// halves.
template <int R>
__global__ __launch_bounds__(256) void k_energy(DevView v, unsigned long long* ysum) {
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t P = v.w * v.h;
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  long long yd[NCLS];
#pragma unroll
  for (int c = 0; c < NCLS; ++c) yd[c] = 0;
  if (p < P) {
    const uint32_t y = p / v.w, x = p - y * v.w;
    uint32_t q[W.M];
#pragma unroll
    for (int mm = 0; mm < W.M; ++mm)
      q[mm] = ((y + v.h + W.oy[mm]) % v.h) * v.w + (x + v.w + W.ox[mm]) % v.w;
    for (uint32_t tt = blockIdx.y; tt < (v.tp >> 3); tt += gridDim.y) {
      const u32x4 cp = *(const u32x4*)(v.cnt + ((size_t)tt * P + p) * 8);
      int part[NCLS];
#pragma unroll
      for (int c = 0; c < NCLS; ++c) part[c] = 0;
#pragma unroll
      for (int mm = 0; mm < W.M; ++mm) {
        if (!(W.oy[mm] > 0 || (W.oy[mm] == 0 && W.ox[mm] > 0))) continue;
        const u32x4 cq = *(const u32x4*)(v.cnt + ((size_t)tt * P + q[mm]) * 8);
        int a = part[W.cls[mm]];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          uint32_t d;   // |halves| <= N (the compiler would take the halves apart)
          asm("v_pk_sub_i16 %0, %1, %2" : "=v"(d) : "v"(cp[k]), "v"(cq[k]));
          a = dot2(d, d, a);
        }
        part[W.cls[mm]] = a;
      }
#pragma unroll
      for (int c = 0; c < NCLS; ++c) yd[c] += part[c];
    }
  }
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    long long s = yd[c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0 && s) atomicAdd(&ysum[(blockIdx.y + 7 * blockIdx.x) % ENERGY_ROWS * NCLS + c], (unsigned long long)s);
  }
}

// ----------------------------------------------------- Gaussian integrands
// Low-frequency test integrands (Sec. 3.5): f_t(x) = exp(-|x - mu_t|^2 / (2 s_t^2)).
// Estimates g = (1/N) sum_k f_t(s_p^k) per pixel.  A wave owns one pixel and
// 16 Gaussians; its lanes hold the samples (8 per lane at a time, as FP64
// x, y and |x|^2, all exact: Q0.16 coordinates) and the Gaussians' exponent
// coefficients come from scalar registers, so a term costs three FP64 FMAs
// (a |x|^2 + bx x + by y + c, the base-2 exponent -log2(e) |x - mu|^2 / (2 s^2),
// accurate to FP64 rounding of terms below 600), one conversion to FP32,
// v_exp_f32 (results below 2^-126 flush to zero, far below the estimate's
// resolution) and one FP32 add.  Each lane sums its 8 terms of a Gaussian in
// FP32 and the groups in FP64; the lanes' sums are added in FP64 through LDS.
// The estimate is stored in FP32.
template <bool CHECK>
__device__ __forceinline__ void gauss_chunk(const DevView& v, uint32_t u, uint32_t c0, uint32_t lane,
                                            const double* __restrict__ gc, double acc[16]) {
  constexpr int SC = 8;
  double sx[SC], sy[SC], s2[SC];
  bool ok[SC];
#pragma unroll
  for (int k = 0; k < SC; ++k) {
    const uint32_t i = c0 + 64 * k + lane;
    ok[k] = !CHECK || i < v.n;
    const uint32_t sv = wrap_add(v.lat[ok[k] ? i : 0], u);
    sx[k] = (double)(sv & 0xFFFFu) * 0x1p-16;
    sy[k] = (double)(sv >> 16) * 0x1p-16;
    s2[k] = __fma_rn(sx[k], sx[k], sy[k] * sy[k]);
  }
  // two halves of 8 Gaussians: their 32 coefficients fit the scalar registers
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const double* gh = gc + 32 * h;
    double cf[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) cf[i] = gh[i];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const double a = cf[4 * g], bx = cf[4 * g + 1], by = cf[4 * g + 2], c = cf[4 * g + 3];
      float part = 0.0f;
#pragma unroll
      for (int k = 0; k < SC; ++k) {
        const double e = __fma_rn(a, s2[k], __fma_rn(bx, sx[k], __fma_rn(by, sy[k], c)));
        const float f = __builtin_amdgcn_exp2f((float)e);
        part = __fadd_rn(part, CHECK && !ok[k] ? 0.0f : f);
      }
      acc[8 * h + g] = __dadd_rn(acc[8 * h + g], (double)part);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Estimates of Gaussians 16 gb .. of the pixel with offset u, by one wave (red:
// its part of LDS).
__device__ __forceinline__ void gauss_estimates(const DevView& v, uint32_t u, uint32_t gb, uint32_t lane,
                                                double (*red)[65], float* out) {
  constexpr uint32_t GB = 16, CH = 512;
  const double* gc = v.gcoef + (size_t)gb * GB * 4;
  double acc[GB];
#pragma unroll
  for (uint32_t g = 0; g < GB; ++g) acc[g] = 0.0;
  uint32_t c0 = 0;
  for (; c0 + CH <= v.n; c0 += CH) gauss_chunk<false>(v, u, c0, lane, gc, acc);
  if (c0 < v.n) gauss_chunk<true>(v, u, c0, lane, gc, acc);
  // lane sums -> per-Gaussian totals, eight Gaussians at a time: lane l adds
  // 8 of Gaussian l % 8's lane sums, then the eight groups are added across
  // lanes
#pragma unroll
  for (uint32_t h = 0; h < 2; ++h) {
#pragma unroll
    for (uint32_t g = 0; g < GB / 2; ++g) red[g][lane] = acc[8 * h + g];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t g = lane & 7, q = lane >> 3;
    double t = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) t = __dadd_rn(t, red[g][8 * q + k]);
    t = __dadd_rn(t, __shfl_xor(t, 8));
    t = __dadd_rn(t, __shfl_xor(t, 16));
    t = __dadd_rn(t, __shfl_xor(t, 32));
    if (lane < GB / 2) out[8 * h + g] = (float)(t / (double)v.n);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int MODE>
__global__ __launch_bounds__(256) void k_gauss_est(DevView v, uint32_t kappa, uint32_t m) {
  __shared__ double red[4][8][65];
  const uint32_t lane = threadIdx.x & 63, wl = threadIdx.x >> 6;
  const uint32_t wave = wave_id();
  const uint32_t ngb = v.tgp / 16;
  const uint32_t j = wave / ngb, gb = wave - j * ngb;
  if (j >= m) return;
  uint32_t u;
  float* out;
  if (MODE == MODE_ALL) {
    u = v.U[j];
    out = v.gest + (size_t)j * v.tgp;
  } else {
    u = v.u_new[j];
    out = v.g_new + (size_t)j * v.tgp;
  }
  if (MODE == MODE_LIST) {
    // a move to the offset that its pixel has changes nothing, whichever form the
    // tile's estimates took
    const uint32_t p = v.pix_list[j];
    if (u == v.U[p]) {
      if (lane < 16) out[gb * 16 + lane] = v.gest[(size_t)p * v.tgp + gb * 16 + lane];
      return;
    }
  }
  gauss_estimates(v, u, gb, lane, red[wl], out + gb * 16);
}

// Sweeps whose estimates come from the lattice lines (gauss_lines.hip) decide as
// the sample by sample estimates would.  Those are off the exact mean g by at most
// 2^-24 (0.37 + 10 g): the exponent's rounding to FP32 (2^-24 max y 2^-y ln 2),
// v_exp_f32 and seven FP32 additions per lane, and the result's rounding; the
// lines' are exact but for that.  The two differ by less than
// eta(g) = 2^-24 (0.37 + 11 g), and a Gaussian's part of the energy change,
//   2 sum_m w_m d x_m,  d = g' - g,  x_m = g' + g - 2 g_m,
// by less than 2 sum_m w_m (|x_m| + |d|) (eta(g') + eta(g) + 2 eta(g_m)), where
// g_m <= (g' + g + |x_m|) / 2.  A move whose energy change is within that bound of
// 0 is listed and its Gaussian part evaluated again from estimates sample by
// sample (of its window: k_gauss_again), then decided.
// 512^2, N = 1024, 1024 Gaussians: about one move in 5000, 0.33 ms a phase (its cost
// is the exponentials of 122 pixels a move), where estimating every proposal so
// would take 14.  With eta(1) for every g four times as many (1.39 ms).  (Where
// nearly all moves are close it costs more than it spares: one Heaviside beside 64
// Gaussians of s = 5, 128^2, N = 1024, 2.3 ms a sweep against 0.5 sample by sample;
// with eight Heavisides or s up to 1 it is faster.)
//
// The bound from W = sum w, b = sum w x^2 (sum w |x| <= sqrt(W b)), s = g' + g.
__device__ __forceinline__ double gauss_margin(double W, double b, double s, double d) {
  const double r = sqrt(W * b) * (1.0 + 1e-12);
  return 2.0 * 0x1p-24 * 1.01 * ((W * d + r) * (1.48 + 22.0 * s) + 11.0 * (b + d * r));
}

// One workgroup per listed move and 16 Gaussians (striding over them).
template <int R>
__global__ __launch_bounds__(256) void k_gauss_again(DevView v, uint32_t kappa) {
  constexpr int S = 2 * R + 1, SQ = S * S;
  __shared__ double red[4][8][65];
  __shared__ float est[SQ + 1][16];   // the window's estimates, raster order, then the move's
  __shared__ double sums[4];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wl = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t ngb = v.tgp / 16, items = v.gunsure[0] * ngb;
  for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
    const uint32_t e = it / ngb, gb = it - e * ngb;
    const uint32_t j = __builtin_amdgcn_readfirstlane(v.gunsure[1 + e]);
    const uint32_t p = class_pixel(v, kappa, j), y = p / v.w, x = p - y * v.w;
    for (uint32_t i = wl; i <= (uint32_t)SQ; i += 4) {
      const uint32_t oy = i / S, ox = i - oy * S;
      const uint32_t q = (y + oy + v.h * (R / v.h + 1) - R) % v.h * v.w + (x + ox + v.w * (R / v.w + 1) - R) % v.w;
      gauss_estimates(v, i == (uint32_t)SQ ? v.u_new[j] : v.U[q], gb, lane, red[wl], est[i]);
    }
    __syncthreads();
    const uint32_t t = tid & 15;
    const double gn = est[SQ][t], go = est[SQ / 2][t], d = gn - go, sm = gn + go;
    double acc = 0.0;
    for (uint32_t i = tid >> 4; i < (uint32_t)SQ; i += 16) {
      const int oy = (int)(i / S) - R, ox = (int)(i % S) - R;
      if (oy || ox) acc += v.wd[v.dcls[ox * ox + oy * oy]] * (d * (sm - 2.0 * (double)est[i][t]));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) sums[wl] = acc;
    __syncthreads();
    if (tid == 0) v.gpart[it] = (sums[0] + sums[1]) + (sums[2] + sums[3]);
  }
}

// The listed moves' decisions (one workgroup); empties the list.
__global__ __launch_bounds__(256) void k_gauss_decide_again(DevView v) {
  const uint32_t n = v.gunsure[0], ngb = v.tgp / 16;
  for (uint32_t e = threadIdx.x; e < n; e += 256) {
    const uint32_t j = v.gunsure[1 + e];
    double acc = 0.0;
    for (uint32_t gb = 0; gb < ngb; ++gb) acc += v.gpart[(size_t)e * ngb + gb];
    const double total = __dadd_rn(v.hpart[j], 2.0 * acc);
    v.gdelta[j] = 2.0 * acc;
    v.delta[j] = total;
    v.accept[j] = (v.objective > 0) ? (total < 0.0) : (total > 0.0);
  }
  __syncthreads();
  if (threadIdx.x == 0) v.gunsure[0] = 0;
}

// Gaussian rows' part of a move's energy change (plain form of Eq. (1) over
// the window, FP64 arithmetic on the FP32 estimates); one wave per moved
// pixel, lanes over integrands, workgroups renumbered per XCD so that moved
// pixels whose windows overlap read the shared rows through one L2.  Written
// to gdelta[j]; the decision adds it to the exact Heaviside part.
template <int R, int MODE>
__global__ __launch_bounds__(256) void k_delta_gauss(DevView v, uint32_t kappa, uint32_t m) {
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t j = __builtin_amdgcn_readfirstlane(xcd_block(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6));
  if (j >= m) return;
  const uint32_t p = (MODE == MODE_CLASS) ? class_pixel(v, kappa, j) : v.pix_list[j];
  const uint32_t y = p / v.w, x = p - y * v.w;
  double cs[NCLS];
#pragma unroll
  for (int c = 0; c < NCLS; ++c) cs[c] = 0.0;
  double margin = 0.0;
  for (uint32_t base = 0; base < v.tgp; base += 64) {
    const uint32_t t = base + lane;
    const double gn = v.g_new[(size_t)j * v.tgp + t], go = v.gest[(size_t)p * v.tgp + t];
    const double d = gn - go, sm = gn + go;
    double b = 0.0, wsum = 0.0;
#pragma unroll
    for (int mm = 0; mm < W.M; ++mm) {
      const uint32_t q = ((y + v.h + W.oy[mm]) % v.h) * v.w + (x + v.w + W.ox[mm]) % v.w;
      const double e = sm - 2.0 * (double)v.gest[(size_t)q * v.tgp + t];
      cs[W.cls[mm]] += d * e;
      if (MODE == MODE_CLASS) {
        b += v.wd[W.cls[mm]] * e * e;
        wsum += v.wd[W.cls[mm]];
      }
    }
    if (MODE == MODE_CLASS) margin += gauss_margin(wsum, b, sm, fabs(d));
  }
  if (MODE == MODE_CLASS && v.gmargin) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) margin += __shfl_xor(margin, off);
    if (lane == 0) v.gmargin[j] = margin;
  }
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    double xv = cs[c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) xv += __shfl_xor(xv, off);
    acc += v.wd[c] * xv;
  }
  if (lane == 0) v.gdelta[j] = 2.0 * acc;
}

// hi + lo += x, with the rounding of hi kept in lo.
__device__ __forceinline__ void add_exact(double& hi, double& lo, double x) {
  const double s = __dadd_rn(hi, x), b = __dsub_rn(s, hi);
  lo = __dadd_rn(lo, __dadd_rn(__dsub_rn(hi, __dsub_rn(s, b)), __dsub_rn(x, b)));
  hi = s;
}

// One Gaussian's window sums of PX class pixels K apart in a row,
//   t = sum_m w_m x_m (rounding of its rows' sums in tl),  s2 = sum_m w_m g_m^2,
// x_m = sm - 2 g_m, from estimates in LDS (corner: the first pixel's window corner;
// column and row strides CS, RS).  The two or four offsets (+-ox, +-oy) share
// their weight: their estimates are added first, without rounding (FP32 values),
// the rows +-oy for all pixels at once.
template <int R, int K, int PX, int CS, int RS, bool MARGIN>
__device__ __forceinline__ void gauss_window(const float* corner, const double* wd, const double (&sm)[PX],
                                             double (&t)[PX], double (&tl)[PX], double (&s2)[PX]) {
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int S = 2 * R + 1, COLS = K * (PX - 1) + S;
#pragma unroll
  for (int i = 0; i < PX; ++i) t[i] = tl[i] = s2[i] = 0.0;
#pragma unroll
  for (int oy = R; oy >= 0; --oy) {
    double h[COLS], q[COLS];
#pragma unroll
    for (int x = 0; x < COLS; ++x) {
      const double a = (double)corner[(R + oy) * RS + x * CS];
      h[x] = a;
      q[x] = a * a;
      if (oy) {
        const double b = (double)corner[(R - oy) * RS + x * CS];
        h[x] += b;
        q[x] = __fma_rn(b, b, q[x]);
      }
    }
#pragma unroll
    for (int i = 0; i < PX; ++i) {
      double row = 0.0;
#pragma unroll
      for (int ox = R; ox >= 0; --ox) {
        if (!ox && !oy) continue;
        const int c = K * i + R;
        const double u = ox ? h[c + ox] + h[c - ox] : h[c], uu = ox ? q[c + ox] + q[c - ox] : q[c];
        const double w = wd[W.cmap[(R + oy) * S + R + ox]];
        const double x = __fma_rn(-2.0, u, (double)((oy ? 2 : 1) * (ox ? 2 : 1)) * sm[i]);
        if (MARGIN) s2[i] = __fma_rn(w, uu, s2[i]);
        row = ox == R ? __dmul_rn(w, x) : __fma_rn(w, x, row);
      }
      add_exact(t[i], tl[i], row);
    }
    // (rows apart: their values for several pixels in flight together would halve
    // the waves)
    if (PX > 1) __builtin_amdgcn_sched_barrier(0);
  }
}

// A Gaussian's part d sum w x of a move into acc + lo, and (MARGIN) its share of the
// margin.
// sum w x^2 = 4 s2 + sm (2 t - W sm), with room for its rounding.
template <bool MARGIN>
__device__ __forceinline__ void gauss_part(double W, double d, double sm, double t, double tl, double s2, double& acc,
                                           double& lo, double& margin) {
  const double p = __dmul_rn(d, t);
  add_exact(acc, lo, p);
  lo += __fma_rn(d, tl, __fma_rn(d, t, -p));
  if (!MARGIN) return;
  const double b = __fma_rn(4.0, s2, sm * __fma_rn(-W, sm, 2.0 * t));
  margin += gauss_margin(W, fmax(b, 0.0) + 1e-13 * W, sm, fabs(d));
}

// Colour-phase form of the same sum: a workgroup owns 4 x 2 class pixels (one
// wave each) and, for 64 Gaussians at a time, stages the estimate rows of
// their window region ((K + 2r + 1) x (3K + 2r + 1) pixels) in LDS, so that
// each row is read from memory once per workgroup rather than once per moved
// pixel.
//
// Rounding: k_delta_gauss adds d x_m per class.  Here a Gaussian's weighted sum of
// x_m is formed first: at most R + 1 roundings in a row of the window, those of
// everything after it kept.  Against 80-bit sums (radii 1 to 5, 64 to 1024
// Gaussians, estimates spread by 0.1 and by 0.01) its mean error is 0.3 to 0.95 of
// k_delta_gauss's; W sm - 2 sum w g, which cancels after the sums, had 5 to 90
// times that.  It also takes fewer FP64 operations (at r = 5 28 a pixel and pair of
// rows with the margin's, 44 before).
template <int R, int K>
struct GaussStage {
  static constexpr int BCX = 4, BCY = 2, NW = BCX * BCY;
  static constexpr int RH = K * (BCY - 1) + 2 * R + 1;
  static constexpr int RW = K * (BCX - 1) + 2 * R + 1;
  static constexpr int RA = RH * RW;
  static constexpr int LDS_BYTES = RA * 64 * 4;
};

template <int R, int K, bool MARGIN>
__global__ __launch_bounds__(512) void k_delta_gauss_stage(DevView v, uint32_t kappa) {
  using G = GaussStage<R, K>;
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  constexpr int NT = 64 * G::NW;
  constexpr int ITER = (G::RA * 16 + NT - 1) / NT;
  extern __shared__ float gl[];                  // [RA][64] estimates of the region
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t a0 = blockIdx.y * G::BCY, b0 = blockIdx.x * G::BCX;
  const uint32_t cy = w / G::BCX, cx = w - cy * G::BCX;
  const uint32_t a = a0 + cy, b = b0 + cx;
  const bool act = (a < v.ch) && (b < v.cw);
  const uint32_t j = act ? a * v.cw + b : 0;
  const uint32_t ky = kappa / K, kx = kappa - ky * K;
  const uint32_t ys = (ky + K * a0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (kx + K * b0 + v.w * (R / v.w + 1) - R) % v.w;
  // staging: float4 it of a thread is quad (idx & 15) of region pixel idx >> 4
  // (threads past the region reload its last pixel and do not store it)
  uint32_t goff[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const uint32_t idx = threadIdx.x + it * NT;
    const uint32_t r = min(idx >> 4, (uint32_t)G::RA - 1);
    const uint32_t rr = r / G::RW, cc = r - rr * G::RW;
    uint32_t gy = ys + rr, gx = xs + cc;
    while (gy >= v.h) gy -= v.h;
    while (gx >= v.w) gx -= v.w;
    goff[it] = gy * v.w + gx;
  }
  const int own = (K * cy + R) * G::RW + K * cx + R;
  const float* corner = gl + ((K * cy) * G::RW + K * cx) * 64 + lane;
  double wd[NCLS], wsum = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    wd[c] = v.wd[c];
    wsum += (double)W.csize[c] * wd[c];
  }
  double acc = 0.0, lo = 0.0, margin = 0.0;
  for (uint32_t base = 0; base < v.tgp; base += 64) {
    f32x4 q[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it)
      q[it] = *(const f32x4*)(v.gest + (size_t)goff[it] * v.tgp + base + 4 * ((threadIdx.x + it * NT) & 15));
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const uint32_t idx = threadIdx.x + it * NT;
      if (idx < (uint32_t)G::RA * 16) *(f32x4*)&gl[idx * 4] = q[it];
    }
    __syncthreads();
    if (act) {
      const double gn = v.g_new[(size_t)j * v.tgp + base + lane], go = gl[own * 64 + lane];
      const double sm[1] = {gn + go};
      double t[1], tl[1], s2[1];
      gauss_window<R, K, 1, 64, 64 * G::RW, MARGIN>(corner, wd, sm, t, tl, s2);
      gauss_part<MARGIN>(wsum, gn - go, sm[0], t[0], tl[0], s2[0], acc, lo, margin);
    }
  }
  if (!act) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double a = __shfl_xor(acc, off);
    lo += __shfl_xor(lo, off);
    add_exact(acc, lo, a);
    if (MARGIN) margin += __shfl_xor(margin, off);
  }
  if (lane != 0) return;
  v.gdelta[j] = 2.0 * (acc + lo);
  if (MARGIN) v.gmargin[j] = margin;
}

// The same for launches with many blocks: a workgroup owns 8 x BCY class pixels
// and 16 Gaussians at a time, a thread four neighbouring pixels of a row and one
// Gaussian, so that a window row's values are read from LDS, converted and
// paired once for four pixels (12 against 30 a pixel at r = 5, K = 2), and the
// region from memory once for 64 (10 pixels of it a pixel against 28).  Bound by
// the FP64 operations.  512^2, 1024 Gaussians, r = 5: 0.72 ms a phase without the
// margin, 1.04 with it; 1.8 and, with it, 1.5 with k_delta_gauss_stage's layout and
// one sum per window offset.
template <int R, int K>
struct GaussTile {
  static constexpr int BCX = 8, BCY = K == 4 ? 4 : 8, PX = 4, NT = BCX / PX * BCY * 16;
  static constexpr int RH = K * (BCY - 1) + 2 * R + 1, RW = K * (BCX - 1) + 2 * R + 1, RA = RH * RW;
  static constexpr int LDS_BYTES = RA * 16 * 4;
};

template <int R, int K, bool MARGIN>
__global__ __launch_bounds__((GaussTile<R, K>::NT)) void k_delta_gauss_tile(DevView v, uint32_t kappa, uint32_t gx) {
  using G = GaussTile<R, K>;
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  constexpr int ITER = (G::RA * 4 + G::NT - 1) / G::NT;
  extern __shared__ float gl[];                  // [RA][16] estimates of the region
  const uint32_t tid = threadIdx.x, t = tid & 15, grp = tid >> 4;
  // (four consecutive rows a wave: their words meet different banks)
  const uint32_t cy = grp % G::BCY, half = grp / G::BCY;
  const uint32_t wk = xcd_block(blockIdx.x, gridDim.x), a0 = wk / gx * G::BCY, b0 = wk % gx * G::BCX;
  const uint32_t ky = kappa / K, kx = kappa - ky * K;
  const uint32_t ys = (ky + K * a0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (kx + K * b0 + v.w * (R / v.w + 1) - R) % v.w;
  uint32_t goff[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const uint32_t r = min((tid + it * G::NT) >> 2, (uint32_t)G::RA - 1);
    const uint32_t rr = r / G::RW, cc = r - rr * G::RW;
    uint32_t y = ys + rr, x = xs + cc;
    while (y >= v.h) y -= v.h;
    while (x >= v.w) x -= v.w;
    goff[it] = y * v.w + x;
  }
  bool act[G::PX];
  uint32_t j[G::PX];
#pragma unroll
  for (int i = 0; i < G::PX; ++i) {
    const uint32_t a = a0 + cy, b = b0 + G::PX * half + i;
    act[i] = a < v.ch && b < v.cw;
    j[i] = act[i] ? a * v.cw + b : 0;
  }
  double wd[NCLS], wsum = 0.0;
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    wd[c] = v.wd[c];
    wsum += (double)W.csize[c] * wd[c];
  }
  const float* col0 = gl + (K * cy * G::RW + K * G::PX * half) * 16 + t;   // window corner of the first pixel
  double acc[G::PX], lo[G::PX], margin[G::PX];
#pragma unroll
  for (int i = 0; i < G::PX; ++i) acc[i] = lo[i] = margin[i] = 0.0;
  for (uint32_t base = 0; base < v.tgp; base += 16) {
    f32x4 q[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it)
      q[it] = *(const f32x4*)(v.gest + (size_t)goff[it] * v.tgp + base + 4 * ((tid + it * G::NT) & 3));
    float gn[G::PX];
#pragma unroll
    for (int i = 0; i < G::PX; ++i) gn[i] = v.g_new[(size_t)j[i] * v.tgp + base + t];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const uint32_t idx = tid + it * G::NT;
      if (idx < (uint32_t)G::RA * 4) *(f32x4*)&gl[idx * 4] = q[it];
    }
    __syncthreads();
    double d[G::PX], sm[G::PX], ts[G::PX], tl[G::PX], s2[G::PX];
#pragma unroll
    for (int i = 0; i < G::PX; ++i) {
      const double go = (double)col0[(R * G::RW + K * i + R) * 16];
      d[i] = (double)gn[i] - go;
      sm[i] = (double)gn[i] + go;
    }
    gauss_window<R, K, G::PX, 16, 16 * G::RW, MARGIN>(col0, wd, sm, ts, tl, s2);
#pragma unroll
    for (int i = 0; i < G::PX; ++i) gauss_part<MARGIN>(wsum, d[i], sm[i], ts[i], tl[i], s2[i], acc[i], lo[i], margin[i]);
  }
#pragma unroll
  for (int i = 0; i < G::PX; ++i) {
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      const double a = __shfl_xor(acc[i], off);
      lo[i] += __shfl_xor(lo[i], off);
      add_exact(acc[i], lo[i], a);
      if (MARGIN) margin[i] += __shfl_xor(margin[i], off);
    }
    if (t == 0 && act[i]) {
      v.gdelta[j[i]] = 2.0 * (acc[i] + lo[i]);
      if (MARGIN) v.gmargin[j[i]] = margin[i];
    }
  }
}

// Gaussian rows' part of the energy: per distance class, sum over the half
// window of |g_p - g_q|^2 (FP64 atomics; doubled by the host).
template <int R>
__global__ __launch_bounds__(256) void k_energy_gauss(DevView v, double* gsum) {
  constexpr Window<R> W = WinConst<R>::w;
  constexpr int NCLS = WinConst<R>::NCLS;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t p = wave_id();
  if (p >= v.w * v.h) return;
  const uint32_t y = p / v.w, x = p - y * v.w;
  double cs[NCLS];
#pragma unroll
  for (int c = 0; c < NCLS; ++c) cs[c] = 0.0;
  for (uint32_t base = 0; base < v.tgp; base += 64) {
    const uint32_t t = base + lane;
    const double gp = v.gest[(size_t)p * v.tgp + t];
#pragma unroll
    for (int mm = 0; mm < W.M; ++mm) {
      if (W.oy[mm] > 0 || (W.oy[mm] == 0 && W.ox[mm] > 0)) {
        const uint32_t q = ((y + v.h + W.oy[mm]) % v.h) * v.w + (x + v.w + W.ox[mm]) % v.w;
        const double d = gp - (double)v.gest[(size_t)q * v.tgp + t];
        cs[W.cls[mm]] += d * d;
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NCLS; ++c) {
    double xv = cs[c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) xv += __shfl_xor(xv, off);
    if (lane == 0 && xv != 0.0) atomicAdd(&gsum[c], xv);
  }
}

// Commit of accepted moves' Gaussian estimate rows.
__global__ __launch_bounds__(256) void k_commit_gauss(DevView v, uint32_t kappa) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t j = wave_id();
  if (j >= v.pc || !v.accept[j]) return;
  const uint32_t p = class_pixel(v, kappa, j);
  const uint32_t P = v.w * v.h;
  for (uint32_t t = lane; t < v.tgp; t += 64) {
    const float g = v.g_new[(size_t)j * v.tgp + t];
    v.gest[(size_t)p * v.tgp + t] = g;
    if (v.bf)
      v.bf[tix(p, v.tp + t, P)] = __builtin_bit_cast(uint16_t, (__bf16)gaussian_error(v, g, t));
  }
}

// Gaussian error rows g - I (refreshed on demand).
__global__ __launch_bounds__(256) void k_gauss_errors(DevView v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)v.w * v.h * v.tgp) return;
  const uint32_t t = (uint32_t)(i % v.tgp);
  v.gerr[i] = (float)((double)v.gest[i] - v.gint[t]);
}


template <int MODE>
hipError_t delta_dispatch(const DevView& v, uint32_t kappa, uint32_t m, hipStream_t s) {
  if (m == 0) return hipSuccess;
  const dim3 grid((m + 3) / 4), block(256);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL((k_delta<1, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 2: hipLaunchKernelGGL((k_delta<2, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 3: hipLaunchKernelGGL((k_delta<3, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 4: hipLaunchKernelGGL((k_delta<4, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 5: hipLaunchKernelGGL((k_delta<5, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 6: hipLaunchKernelGGL((k_delta<6, MODE>), grid, block, 0, s, v, kappa, m); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_init_offsets(const DevView& v, hipStream_t s) {
  const uint32_t P = v.w * v.h;
  hipLaunchKernelGGL(k_init_offsets, dim3((P + 255) / 256), dim3(256), 0, s, v);
  return hipGetLastError();
}


bool staged_phases(const DevView& v) { return !v.mfma && (v.k == 1 || v.k == 2 || v.k == 4); }

uint32_t phase_blocks(const DevView& v) {
  switch (v.form) {
    case FIELD_NARROW: return phase_blocks_narrow(v);
    case FIELD_SPLIT: return phase_blocks_split(v);
    default: return phase_blocks_wide(v);
  }
}

hipError_t launch_phase(const DevView& v, uint32_t kappa, hipStream_t s) {
  switch (v.form) {
    case FIELD_NARROW: return launch_phase_narrow(v, kappa, s);
    case FIELD_SPLIT: return launch_phase_split(v, kappa, s);
    default: return launch_phase_wide(v, kappa, s);
  }
}

hipError_t launch_delta(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s) {
  if (mode != MODE_CLASS) return delta_dispatch<MODE_LIST>(v, kappa, m, s);
  // BF16 precision form: matrix-core Gram pass, decision, exact re-evaluation
  if (v.mfma) return launch_delta_bf16(v, kappa, s);
  if (!staged_phases(v)) return delta_dispatch<MODE_CLASS>(v, kappa, m, s);
  hipError_t e = launch_phase(v, kappa, s);
  return e != hipSuccess || !v.gmargin ? e : launch_gauss_again(v, kappa, s);
}

hipError_t launch_finish(const DevView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_delta_finish, dim3((v.pc + 255) / 256), dim3(256), 0, s, v);
  return hipGetLastError();
}

uint32_t commit_blocks(const DevView& v) { return (v.pc + 63) / 64; }

hipError_t launch_commit(const DevView& v, uint32_t kappa, hipStream_t s, bool advance) {
  hipLaunchKernelGGL(k_commit, dim3(commit_blocks(v)), dim3(64 * COMMIT_WAVES), 0, s, v, kappa, advance);
  return hipGetLastError();
}

// Phases on narrow forms read an accepted move of an earlier class from its
// proposal, so that a sweep has one commit launch: three of the eight launches
// of a sweep's chain at K = 2 less, and the rows of all classes in flight
// together (two sweeps of 256^2, N = 256, T = 1024: 312 -> 248 us, of 32^2, N = 16,
// T = 64: 113 -> 95).  (Gaussian rows are read
// from the estimates, which their commit updates class by class.)
bool moves_wait(const DevView& v) { return v.form != FIELD_WIDE && !v.tgp; }

uint32_t commit_sweep_blocks(const DevView& v) { return v.k * v.k * commit_blocks(v); }

hipError_t launch_commit_sweep(const DevView& v, hipStream_t s, bool advance) {
  hipLaunchKernelGGL(k_commit_sweep, dim3(commit_sweep_blocks(v)), dim3(64 * COMMIT_WAVES), 0, s, v, advance);
  return hipGetLastError();
}

hipError_t launch_commit_sweep_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks,
                                     hipStream_t s) {
  hipLaunchKernelGGL(k_commit_sweep_batch, dim3(blocks), dim3(64 * COMMIT_WAVES), 0, s, views, pre, nmem);
  return hipGetLastError();
}

hipError_t launch_follow(const DevView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_follow, dim3((v.w * v.h + FOLLOW_PIXELS - 1) / FOLLOW_PIXELS), dim3(256), 0, s, v);
  return hipGetLastError();
}

hipError_t launch_follow_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_follow_batch, dim3(blocks), dim3(256), 0, s, views, pre, nmem);
  return hipGetLastError();
}

hipError_t launch_errors(const DevView& v, hipStream_t s) {
  const size_t n = (size_t)v.w * v.h * (v.tp >> 3);
  hipLaunchKernelGGL(k_errors, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, v);
  return hipGetLastError();
}

hipError_t launch_pack_errors(const DevView& v, uint32_t first, uint32_t n, float* out, hipStream_t s) {
  const uint64_t items = (uint64_t)n * (v.t + v.tg);
  hipLaunchKernelGGL(k_pack_errors, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, v, first, n, out);
  return hipGetLastError();
}

hipError_t launch_advance(const DevView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, v.ctr);
  return hipGetLastError();
}

hipError_t launch_recount_index(const DevView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_recount_index, dim3(1), dim3(64), 0, s, v.ctr);
  return hipGetLastError();
}

hipError_t launch_recount_advance_pair(const DevView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_recount_advance_pair, dim3(1), dim3(64), 0, s, v.ctr);
  return hipGetLastError();
}

hipError_t launch_points(const DevView& v, uint32_t pixel, uint32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_points, dim3((v.n + 255) / 256), dim3(256), 0, s, v, pixel, out);
  return hipGetLastError();
}

hipError_t launch_energy(const DevView& v, unsigned long long* y, hipStream_t s) {
  const uint32_t P = v.w * v.h;
  // about eight workgroups per CU
  const uint32_t gx = (P + 255) / 256, gy = std::max(1u, std::min(v.tp >> 3, 2048 / gx));
  const dim3 grid(gx, gy), block(256);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL(k_energy<1>, grid, block, 0, s, v, y); break;
    case 2: hipLaunchKernelGGL(k_energy<2>, grid, block, 0, s, v, y); break;
    case 3: hipLaunchKernelGGL(k_energy<3>, grid, block, 0, s, v, y); break;
    case 4: hipLaunchKernelGGL(k_energy<4>, grid, block, 0, s, v, y); break;
    case 5: hipLaunchKernelGGL(k_energy<5>, grid, block, 0, s, v, y); break;
    case 6: hipLaunchKernelGGL(k_energy<6>, grid, block, 0, s, v, y); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gauss_again(const DevView& v, uint32_t kappa, hipStream_t s) {
  const dim3 grid(2048), block(256);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL(k_gauss_again<1>, grid, block, 0, s, v, kappa); break;
    case 2: hipLaunchKernelGGL(k_gauss_again<2>, grid, block, 0, s, v, kappa); break;
    case 3: hipLaunchKernelGGL(k_gauss_again<3>, grid, block, 0, s, v, kappa); break;
    case 4: hipLaunchKernelGGL(k_gauss_again<4>, grid, block, 0, s, v, kappa); break;
    case 5: hipLaunchKernelGGL(k_gauss_again<5>, grid, block, 0, s, v, kappa); break;
    case 6: hipLaunchKernelGGL(k_gauss_again<6>, grid, block, 0, s, v, kappa); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gauss_decide_again, dim3(1), dim3(256), 0, s, v);
  return hipGetLastError();
}

// Tiles whose estimates come from the lines: the line form gives a wave 64 pixels
// and 4 Gaussians, the sample form one pixel and 16 Gaussians: below about 1024
// waves, one a SIMD, the former leaves most of the chip idle (at N = 1024 a wave
// takes about 50 us, where the sample form is done in 5 us for 144 pixels and 128
// Gaussians).
bool gauss_lines_pay(const DevView& v, uint32_t m) { return (uint64_t)((m + 63) / 64) * (v.tgp / 16) >= 256; }

hipError_t launch_gauss_est(const DevView& v, int mode, uint32_t m, hipStream_t s) {
  if (!v.tgp || m == 0) return hipSuccess;
  // a problem's sweeps, phases and whole tile use one form; pixel lists the one
  // that is faster at their size
  // (from 16384 of its waves on the sample form fills the chip several times over;
  // N = 1024, 1024 Gaussians: 85 us the call against 133 at 64 moves, 131 against 141 at
  // 256, 188 against 144 at 512; N = 256: 89 against 91 at 128, 107 against 93 at 256)
  const uint64_t waves = (uint64_t)m * (v.tgp >> 4);
  if (v.glines && (mode != MODE_LIST || waves >= 16384)) return launch_gauss_lines(v, mode == MODE_ALL, m, s);
  const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
  if (mode == MODE_ALL) hipLaunchKernelGGL(k_gauss_est<MODE_ALL>, grid, block, 0, s, v, 0u, m);
  else if (mode == MODE_LIST) hipLaunchKernelGGL(k_gauss_est<MODE_LIST>, grid, block, 0, s, v, 0u, m);
  else hipLaunchKernelGGL(k_gauss_est<MODE_CLASS>, grid, block, 0, s, v, 0u, m);
  return hipGetLastError();
}

namespace {
template <int MODE>
hipError_t gauss_delta_dispatch(const DevView& v, uint32_t kappa, uint32_t m, hipStream_t s) {
  const dim3 grid((m + 3) / 4), block(256);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL((k_delta_gauss<1, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 2: hipLaunchKernelGGL((k_delta_gauss<2, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 3: hipLaunchKernelGGL((k_delta_gauss<3, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 4: hipLaunchKernelGGL((k_delta_gauss<4, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 5: hipLaunchKernelGGL((k_delta_gauss<5, MODE>), grid, block, 0, s, v, kappa, m); break;
    case 6: hipLaunchKernelGGL((k_delta_gauss<6, MODE>), grid, block, 0, s, v, kappa, m); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int R, int K>
hipError_t gauss_stage_launch(const DevView& v, uint32_t kappa, hipStream_t s) {
  using T = GaussTile<R, K>;
  if constexpr (T::LDS_BYTES <= 65536) {
    // tiles from 256 blocks on, a workgroup per CU; smaller blocks below
    const uint32_t gx = (v.cw + T::BCX - 1) / T::BCX, blocks = gx * ((v.ch + T::BCY - 1) / T::BCY);
    if (blocks >= 256) {
      hipLaunchKernelGGL((v.gmargin ? k_delta_gauss_tile<R, K, true> : k_delta_gauss_tile<R, K, false>), dim3(blocks), dim3(T::NT), (size_t)T::LDS_BYTES, s, v, kappa, gx);
      return hipGetLastError();
    }
  }
  using G = GaussStage<R, K>;
  if constexpr (G::LDS_BYTES > 65536) {
    return gauss_delta_dispatch<MODE_CLASS>(v, kappa, v.pc, s);
  } else {
    const dim3 grid((v.cw + G::BCX - 1) / G::BCX, (v.ch + G::BCY - 1) / G::BCY);
    hipLaunchKernelGGL((v.gmargin ? k_delta_gauss_stage<R, K, true> : k_delta_gauss_stage<R, K, false>), grid, dim3(64 * G::NW), (size_t)G::LDS_BYTES, s, v, kappa);
    return hipGetLastError();
  }
}

template <int R>
hipError_t gauss_stage_by_k(const DevView& v, uint32_t kappa, hipStream_t s) {
  switch (v.k) {
    case 1: return gauss_stage_launch<R, 1>(v, kappa, s);
    case 2: return gauss_stage_launch<R, 2>(v, kappa, s);
    case 4: return gauss_stage_launch<R, 4>(v, kappa, s);
    default: return gauss_delta_dispatch<MODE_CLASS>(v, kappa, v.pc, s);
  }
}
}  // namespace

hipError_t launch_gauss_delta(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s) {
  if (!v.tgp || m == 0) return hipSuccess;
  // the approximate BF16 form evaluates the Gaussian rows in its Gram pass
  // and re-evaluates accepted moves exactly
  if (mode == MODE_CLASS && v.mfma == 2) return hipSuccess;
  if (mode == MODE_CLASS) {
    switch (v.radius) {
      case 1: return gauss_stage_by_k<1>(v, kappa, s);
      case 2: return gauss_stage_by_k<2>(v, kappa, s);
      case 3: return gauss_stage_by_k<3>(v, kappa, s);
      case 4: return gauss_stage_by_k<4>(v, kappa, s);
      case 5: return gauss_stage_by_k<5>(v, kappa, s);
      case 6: return gauss_stage_by_k<6>(v, kappa, s);
      default: return hipErrorInvalidValue;
    }
  }
  return gauss_delta_dispatch<MODE_LIST>(v, kappa, m, s);
}

hipError_t launch_gauss_delta_exact(const DevView& v, uint32_t kappa, hipStream_t s) {
  if (!v.tgp) return hipSuccess;
  switch (v.radius) {
    case 1: return gauss_stage_by_k<1>(v, kappa, s);
    case 2: return gauss_stage_by_k<2>(v, kappa, s);
    case 3: return gauss_stage_by_k<3>(v, kappa, s);
    case 4: return gauss_stage_by_k<4>(v, kappa, s);
    case 5: return gauss_stage_by_k<5>(v, kappa, s);
    case 6: return gauss_stage_by_k<6>(v, kappa, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gauss_commit(const DevView& v, uint32_t kappa, hipStream_t s) {
  if (!v.tgp) return hipSuccess;
  hipLaunchKernelGGL(k_commit_gauss, dim3((v.pc + 3) / 4), dim3(256), 0, s, v, kappa);
  return hipGetLastError();
}

hipError_t launch_gauss_errors(const DevView& v, hipStream_t s) {
  if (!v.tgp) return hipSuccess;
  const size_t n = (size_t)v.w * v.h * v.tgp;
  hipLaunchKernelGGL(k_gauss_errors, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, v);
  return hipGetLastError();
}

hipError_t launch_gauss_energy(const DevView& v, double* gsum, hipStream_t s) {
  if (!v.tgp) return hipSuccess;
  const uint32_t P = v.w * v.h;
  const dim3 grid((P + 3) / 4), block(256);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL(k_energy_gauss<1>, grid, block, 0, s, v, gsum); break;
    case 2: hipLaunchKernelGGL(k_energy_gauss<2>, grid, block, 0, s, v, gsum); break;
    case 3: hipLaunchKernelGGL(k_energy_gauss<3>, grid, block, 0, s, v, gsum); break;
    case 4: hipLaunchKernelGGL(k_energy_gauss<4>, grid, block, 0, s, v, gsum); break;
    case 5: hipLaunchKernelGGL(k_energy_gauss<5>, grid, block, 0, s, v, gsum); break;
    case 6: hipLaunchKernelGGL(k_energy_gauss<6>, grid, block, 0, s, v, gsum); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}


// ------------------------------------------------------------------ batches

hipError_t launch_phase_batch(uint32_t form, uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                              uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s) {
  switch (form) {
    case FIELD_NARROW: return launch_phase_batch_narrow(radius, k, sliced, views, pre, nmem, blocks, kappa, s);
    case FIELD_SPLIT: return launch_phase_batch_split(radius, k, sliced, views, pre, nmem, blocks, kappa, s);
    default: return launch_phase_batch_wide(radius, k, sliced, views, pre, nmem, blocks, kappa, s);
  }
}

hipError_t launch_commit_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks,
                               uint32_t kappa, hipStream_t s) {
  hipLaunchKernelGGL(k_commit_batch, dim3(blocks), dim3(64 * COMMIT_WAVES), 0, s, views, pre, nmem, kappa);
  return hipGetLastError();
}

hipError_t launch_advance_batch(const DevView* views, uint32_t nmem, hipStream_t s) {
  hipLaunchKernelGGL(k_advance_batch, dim3((nmem + 63) / 64), dim3(64), 0, s, views, nmem);
  return hipGetLastError();
}
}  // namespace bnlat
