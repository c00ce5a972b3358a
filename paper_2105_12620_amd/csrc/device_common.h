// Device helpers shared by the gfx950 kernel sources: Philox, Q0.16
// arithmetic, tiled count indexing, the int16 dot product, colour-class
// pixel order, proposals and the window offset tables.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bnlat_dev.h"

// v_writelane_b32: write a wave-uniform value into one lane of a register.
extern "C" __device__ int bnlat_writelane_i32(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace bnlat {
namespace {

typedef short v2i16 __attribute__((ext_vector_type(2)));
// Native 4 x u32 vector: kept in registers where HIP's uint4 struct is not.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));


// Philox4x32-10 (Salmon et al., SC 2011): two 32x32->64 products per round,
// key advanced by the Weyl constants between rounds.  Returns words 0 and 1.
__device__ inline uint2 philox_w01(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                   uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  return make_uint2(c0, c1);
}

// Q0.16 pair from the top halves of words 0 and 1.
__device__ inline uint32_t q16_pair(uint2 w) { return (w.x >> 16) | (w.y & 0xFFFF0000u); }

// Componentwise (a + b) mod 2^16 of two packed Q0.16 pairs: the toroidal
// shift mod(s + u, 1) of Sec. 3.2.
__device__ inline uint32_t wrap_add(uint32_t a, uint32_t b) {
  return ((a + b) & 0xFFFFu) | (((a >> 16) + (b >> 16)) << 16);
}

// S - 2^15 per component, as two int16.
__device__ inline uint32_t centre(uint32_t s) { return s ^ 0x80008000u; }

// 16 int8 deviations (bias: the bias8 words of their integrands) back as 16-bit
// counts.
__device__ __forceinline__ void widen8(const u32x4 d, const uint32_t* __restrict__ bias, uint4& lo, uint4& hi) {
  uint32_t o[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t x = d[k] ^ 0x80808080u;   // byte = count - base + 128
    o[2 * k] = __builtin_amdgcn_perm(0u, x, 0x0C010C00u) - bias[2 * k];
    o[2 * k + 1] = __builtin_amdgcn_perm(0u, x, 0x0C030C02u) - bias[2 * k + 1];
  }
  lo = make_uint4(o[0], o[1], o[2], o[3]);
  hi = make_uint4(o[4], o[5], o[6], o[7]);
}

// 16 counts of two tiles as int8 deviations: per half count - base + 128 (no
// borrow between the halves), then the low bytes, less 128.
__device__ __forceinline__ u32x4 narrow8(const uint4 lo, const uint4 hi, const uint32_t* __restrict__ bias) {
  const uint32_t c[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  u32x4 o;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    o[k] = __builtin_amdgcn_perm(c[2 * k + 1] + bias[2 * k + 1], c[2 * k] + bias[2 * k], 0x06040200u) ^ 0x80808080u;
  return o;
}

// Element (row, t) of a tiled count buffer with `rows` rows.
__device__ inline size_t tix(uint32_t row, uint32_t t, uint32_t rows) {
  return ((size_t)(t >> 3) * rows + row) * 8 + (t & 7);
}

// Signed int16x2 dot product plus accumulator (v_dot2_i32_i16).  The clamp
// bit keeps the three-operand encoding; it never engages because every
// product sum here stays below 2^31 in magnitude.
__device__ inline int dot2(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot2(__builtin_bit_cast(v2i16, a), __builtin_bit_cast(v2i16, b), c, true);
}

// Signed int8x4 dot product plus accumulator (v_dot4_i32_i8; the clamp as above).
__device__ inline int dot4(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot4((int)a, (int)b, c, true);
}

// Bytewise a - b mod 2^8.
__device__ inline uint32_t sub_bytes(uint32_t a, uint32_t b) {
  return ((a | 0x80808080u) - (b & 0x7F7F7F7Fu)) ^ ((a ^ ~b) & 0x80808080u);
}

__device__ inline uint32_t wave_id() {
  return __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
}

// Workgroup barrier of the kernels that fill LDS with global_load_lds: waits
// until at most N of this wave's vector-memory loads are in flight (they
// complete in order, so every earlier one has landed) and its LDS accesses
// are done, then meets the other waves (a __syncthreads would also wait for
// the loads still meant to be in flight).  The empty asm statements keep the
// compiler from moving memory accesses across.  s_waitcnt immediate in the
// gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt (bits 6:4) left open,
// lgkmcnt (bits 11:8) zero.
template <int N>
__device__ inline void barrier_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Workgroups go to the eight XCDs in turn (workgroup b to XCD b mod 8), each
// with its own L2.  This renumbers them so that every XCD's workgroups form one
// contiguous range of logical indices: neighbouring work then shares an L2.
__device__ inline uint32_t xcd_block(uint32_t b, uint32_t g) {
  const uint32_t x = b & 7, i = b >> 3, q = g >> 3, r = g & 7;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + i;
}

__device__ inline uint32_t class_pixel(const DevView& v, uint32_t kappa, uint32_t j) {
  const uint32_t ky = kappa / v.k, kx = kappa - ky * v.k;
  const uint32_t a = j / v.cw, b = j - a * v.cw;
  return (ky + v.k * a) * v.w + (kx + v.k * b);
}

__device__ inline uint32_t proposal(const DevView& v, uint32_t p, uint32_t sweep) {
  return q16_pair(philox_w01(p, sweep, v.problem, S_PROP, v.seed_lo, v.seed_hi));
}

// Energy change of class pixel j (pixel p) from its Heaviside part; a move too close
// to be decided from the line form's estimates is listed (launch_gauss_again), but
// for one to the offset that the pixel has: it changes nothing in either form.
__device__ __forceinline__ double with_gaussian_part(const DevView& v, uint32_t j, uint32_t p, double heaviside) {
  if (!v.tgp) return heaviside;
  const double total = __dadd_rn(heaviside, v.gdelta[j]);
  if (v.gmargin && fabs(total) <= v.gmargin[j] && v.u_new[j] != v.U[p]) {
    v.gunsure[1 + atomicAdd(v.gunsure, 1u)] = j;
    v.hpart[j] = heaviside;
  }
  return total;
}

// Decision of class pixel j (pixel p) from its weighted class sums; in the BF16
// form's re-evaluation of a move that its own value accepted, a move that the exact
// value rejects is a veto.
__device__ __forceinline__ void decide_move(const DevView& v, uint32_t kappa, uint32_t j, uint32_t p, double sum) {
  const double total = with_gaussian_part(v, j, p, __dmul_rn(sum, 2.0 / ((double)v.n * (double)v.n)));
  const bool ok = (v.objective > 0) ? (total < 0.0) : (total > 0.0);
  v.delta[j] = total;
  v.accept[j] = ok;
  if (v.accepts) v.accepts[(size_t)kappa * v.pc + j] = ok;
  if (v.mfma && !ok) atomicAdd(&v.ctr[2], 1ull);
}

// A phase launch's blocks, slice after slice: b of the launch's (or member's) n is
// block b of slice z, with stages (64 integrands) [first, last).  SLICED: launches
// of problems with several slices (the others' kernels are compiled without; their
// prologue was 1 to 2 us longer with).
template <bool SLICED>
struct SliceBlock {
  uint32_t b, z, first, last;
  __device__ __forceinline__ SliceBlock(const DevView& v, uint32_t b_, uint32_t n)
      : b(b_), z(0), first(0), last((v.t + 63) / 64) {
    if (!SLICED) return;
    const uint32_t blocks = n / v.slices, per = (last + v.slices - 1) / v.slices;
    z = b / blocks;
    b -= z * blocks;
    first = z * per;
    last = min(first + per, last);
  }
};

// A workgroup's class sums of one slice (LDS, [NCLS + 1][PX], the self terms last)
// into xsum; pixel(px) is the class pixel's index, or v.pc past the tile.
template <int NCLS, uint32_t PX, class F>
__device__ __forceinline__ void store_slice(const DevView& v, uint32_t z, const unsigned long long* sums, uint32_t threads,
                                            F pixel) {
  constexpr uint32_t ROW = NCLS + 1;
  for (uint32_t e = threadIdx.x; e < PX * ROW; e += threads) {
    const uint32_t px = e / ROW, c = e - px * ROW, j = pixel(px);
    if (j < v.pc) v.xsum[((size_t)z * v.pc + j) * ROW + c] = (long long)sums[c * PX + px];
  }
}

// The window's offsets in steps of up to eight: row steps of consecutive offsets
// of a window row, then column steps of eight rows of the columns they leave
// over.  offset: slot i of step st, and whether the slot holds one.
template <int R>
struct WindowSteps {
  static constexpr int WS = 2 * R + 1;
  static constexpr int RC = WS < 8 ? WS : 8;             // offsets of a row step
  static constexpr int LC = WS - RC;                     // columns left to column steps
  static constexpr int CH = (WS + 7) / 8;                // column steps per such column
  static constexpr int LASTROWS = WS - 8 * (CH - 1);     // rows of a column's last step
  static constexpr int STEPS = WS + LC * CH;
  __device__ static inline bool offset(int st, int i, int& ox, int& oy) {
    if (st < WS) {
      oy = st - R;
      ox = -R + i;
      return i < RC;
    }
    const int t = st - WS, col = t / CH, part = t % CH;
    ox = -R + RC + col;
    oy = -R + 8 * part + i;
    return oy <= R;
  }
};

// ------------------------------------------------- BF16 error field values

// Round to the nearest BF16 (ties to even); bits of two values packed.
__device__ inline uint32_t bf16x2_bits(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}

// Field value of 8 Heaviside counts (one 16-byte count tile) in either mode.
__device__ inline uint4 heaviside_field_tile(const DevView& v, const uint4 c8, uint32_t t) {
  const uint32_t w[4] = {c8.x, c8.y, c8.z, c8.w};
  uint32_t o[4];
  const float inv_n = 1.0f / (float)v.n;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float c0 = (float)(w[k] & 0xFFFFu), c1 = (float)(w[k] >> 16);
    if (v.mfma == 1) {
      o[k] = bf16x2_bits(c0, c1);
    } else {
      o[k] = bf16x2_bits(__fsub_rn(__fmul_rn(c0, inv_n), v.area[t + 2 * k]),
                         __fsub_rn(__fmul_rn(c1, inv_n), v.area[t + 2 * k + 1]));
    }
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// Field value of Gaussian row t (FP32 estimate g): g - I rounded to FP32,
// then to BF16 by the caller; padded rows are 0.
__device__ inline float gaussian_error(const DevView& v, float g, uint32_t t) {
  return t < v.tg ? (float)((double)g - v.gint[t]) : 0.0f;
}

// --------------------------------------------------------- window tables

// Offsets of the (2R+1)^2 - 1 window grouped by squared distance d in
// increasing d (row-major inside a group), with their group index.
template <int R>
struct Window {
  static constexpr int M = (2 * R + 1) * (2 * R + 1) - 1;
  static constexpr int DMAX = 2 * R * R;
  int ox[M], oy[M], cls[M];
  int ncls;
  int d[DMAX + 1], csize[DMAX + 1];
  int cmap[(2 * R + 1) * (2 * R + 1)];   // group of offset (x, y) at (y + R)(2R + 1) + x + R; -1 at (0, 0)
  constexpr Window() : ox(), oy(), cls(), ncls(0), d(), csize(), cmap() {
    int idx = 0;
    for (int dd = 1; dd <= DMAX; ++dd) {
      int found = 0;
      for (int y = -R; y <= R; ++y)
        for (int x = -R; x <= R; ++x)
          if (x * x + y * y == dd) {
            ox[idx] = x;
            oy[idx] = y;
            cls[idx] = ncls;
            cmap[(y + R) * (2 * R + 1) + x + R] = ncls;
            ++idx;
            ++found;
          }
      if (found) {
        d[ncls] = dd;
        csize[ncls] = found;
        ++ncls;
      }
    }
    cmap[R * (2 * R + 1) + R] = -1;
  }
};

template <int R>
struct WinConst {
  static constexpr Window<R> w{};
  static constexpr int NCLS = w.ncls;
};

// Member of a batch that owns launch block blk (prefix sums of blocks per
// member): the lanes compare 64 members at once, one round of loads where a
// serial search took one per member (3 us of every workgroup at 32 members).
__device__ inline uint32_t batch_member(const uint32_t* __restrict__ pre, uint32_t nmem, uint32_t blk) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t i = 0;
  for (uint32_t m = 1; m < nmem; m += 64) {
    const bool past = m + lane < nmem && pre[m + lane] <= blk;
    i += (uint32_t)__popcll(__ballot(past));
  }
  return __builtin_amdgcn_readfirstlane(i);
}

// Calls f with the radius and colour modulus as constants.
template <int R, class F>
hipError_t by_radius_k1(uint32_t k, F f) {
  switch (k) {
    case 1: return f(std::integral_constant<int, R>(), std::integral_constant<int, 1>());
    case 2: return f(std::integral_constant<int, R>(), std::integral_constant<int, 2>());
    case 4: return f(std::integral_constant<int, R>(), std::integral_constant<int, 4>());
    default: return hipErrorInvalidValue;
  }
}

template <class F>
hipError_t by_radius_k(uint32_t radius, uint32_t k, F f) {
  switch (radius) {
    case 1: return by_radius_k1<1>(k, f);
    case 2: return by_radius_k1<2>(k, f);
    case 3: return by_radius_k1<3>(k, f);
    case 4: return by_radius_k1<4>(k, f);
    case 5: return by_radius_k1<5>(k, f);
    case 6: return by_radius_k1<6>(k, f);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace bnlat
