// gfx950 hit-counting kernels: the estimator of the test-integrand map
// (Sec. 2) for every pixel (bn_compute_errors), for the proposals of one
// colour class, of a pixel list, or of a whole sweep (the overlapped
// schedule), plus their batched form.
//
// Counts land in the tiled layout uint16 [Tp/8][rows][8]; the Heaviside
// predicate n.(S - 2^15) > D' is an exact int16 dot product against an int32
// threshold on Q0.16 sample coordinates.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

// Resolve the pixel, offset and output buffers (row index, row count) of work
// item j of a count launch: counts as uint16 [Tp/8][rows][8] in wide, as int8
// [Tp/16][rows][16] less their integrand's base in narrow (either null).
template <int MODE>
__device__ inline void count_target(const DevView& v, uint32_t kappa, uint32_t j, uint32_t m,
                                    uint32_t& p, uint32_t& u, uint16_t*& wide, int8_t*& narrow, uint32_t& row,
                                    uint32_t& rows) {
  if (MODE == MODE_ALL) {
    p = j;
    u = v.U[p];
    wide = v.cnt;
    narrow = v.d8;
    row = p;
    rows = v.w * v.h;
  } else if (MODE == MODE_CLASS) {
    p = class_pixel(v, kappa, j);
    u = proposal(v, p, (uint32_t)v.ctr[0]);
    wide = v.c_new;
    narrow = v.n8;
    row = j;
    rows = v.pc;
  } else if (MODE == MODE_SWEEP) {
    const uint32_t cls = j / v.pc, jj = j - cls * v.pc;
    p = class_pixel(v, cls, jj);
    u = proposal(v, p, (uint32_t)v.ctr[0] + kappa);
    const size_t first = (size_t)cls * v.pc * v.tp;
    wide = v.c_new ? v.c_new + first : nullptr;
    narrow = v.n8 ? v.n8 + first : nullptr;
    row = jj;
    rows = v.pc;
  } else {
    p = v.pix_list[j];
    u = v.u_new[j];
    wide = v.c_new;
    narrow = nullptr;
    row = j;
    rows = m;
  }
}

// ----------------------------------------------------------- hit counting
//
// Estimator of the test-integrand map (Sec. 2): c[p][t] = number of the N
// scrambled samples on the hit side of Heaviside t.  Every lane owns one work
// item (a pixel, or a proposal); a wave walks a chunk of integrands with
// wave-uniform parameters from scalar loads.  Two counters give the same
// integers:
//
// LineCounter (N >= 16).  The samples are the points of a shifted plane
// lattice in the unit square, so they lie on parallel lines: with b1 the
// lattice vector of smallest |x| + |y| (in units of 1/N), at most
// |x| + |y| <= sqrt(2 N) lines meet the square, and a line's samples are
// A + l b2 + j b1 for consecutive j in [lo_l, hi_l).  A Heaviside's edge
// crosses line l at one place, which moves by the same amount from each line
// to the next, so per (line, integrand) the work is one 64-bit add (the
// crossing in units of b1, 32 fraction bits), one clamp of its integer part
// to [lo_l, hi_l] and half a three-operand add: 2.5 lane-operations per line
// in place of 1.75 per sample (at N = 256: 16 lines, 45 against 466 with the
// set-up of an integrand).  lo and hi depend only on which of N classes the
// pixel's shift falls in (shifts that differ by a lattice vector give the
// same lines) and come from a table; A is a sample of the pixel.  Bound by
// the vector ALU; measured at 256^2, N = 256, T = 1000 with the error vectors
// written: 105 us per bn_compute_errors against 877 us sample by sample
// (470 MB written, padded rows and the int8 field among them: 4.5 TB/s).
//   Exactness: with D' + 1/2 in place of D', the crossings are odd multiples
// of 1 / (2 |m|), m = n . b1, hence at least that far from an integer.  The
// fixed-point value is off by at most 2^-33 per rounding: the first crossing
// (one FP64 fma onto 1.5 2^20, whose last bit is 2^-32), the uniform offset
// and the slope of each further line, (R + 1) 2^-33 in all for R lines;
// |m| <= 2^30 R / N and R^2 <= 2 N keep that below 1 / (2 |m|).  Integrands
// with |m| < LINE_MIN_M (edges nearly along the lines: about one drawn in 10^4, and
// short normals that a caller gives), whose crossings leave the fma's range, take
// FP64 throughout, six operations a line (128^2, N = 4096, 256 normals (0, 1): 35 us
// per bn_compute_errors; sample by sample, in a loop of dependent loads, 6.3 ms, and one
// such integrand among ordinary ones made 512 of them take 272 us in place of 33).
//
// SampleCounter (N <= 8, where it costs less: 14 lane-operations at N = 8
// against 17): per (sample, integrand) one v_dot2 with the threshold folded in
// (n.s > D' exactly when r = n.s - D' - 1 >= 0; |n.s|, |D'| <= 2^30, so r
// never overflows); per sample one v_perm_b32 turns the sign bits of two
// integrands' residues into 0x00/0xFF bytes in the two 16-bit halves of a
// word, and per two such words one v_add3_u32 sums them: 255 x the misses of
// integrands i and i + 1, which become N - misses, already packed as the tile
// layout stores them.

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// The integrand tables never change while a kernel runs: read through the
// constant address space, wave-uniform elements come by scalar loads although
// the kernel stores counts (which the compiler must take to alias).
#define BN_UNIFORM __attribute__((address_space(4)))
template <class T>
__device__ inline const BN_UNIFORM T* uniform(const T* p) {
  return (const BN_UNIFORM T*)p;
}

// Sign bytes of a sample's residues for two integrands: byte 0 is 0xFF when
// lo < 0 and byte 2 is 0xFF when hi < 0 (v_perm_b32 selectors 9 and 11 repeat
// bit 31 of the second and of the first operand; selector 12 is a zero byte).
__device__ inline uint32_t sign_bytes(int lo, int hi) {
  return __builtin_amdgcn_perm((uint32_t)hi, (uint32_t)lo, 0x0C0B0C09u);
}

// Per 16-bit half, x = 255 m with 0 <= m <= 255 becomes m:
// floor(255 (m + 1) / 256) = m, so m = (x + 255) >> 8.
__device__ inline uint32_t halves_div255(uint32_t x) {
  const u16x2 h = __builtin_bit_cast(u16x2, x);
  return __builtin_bit_cast(uint32_t, (u16x2)((h + (u16x2){255, 255}) >> (u16x2){8, 8}));
}

// Packed hit counts of integrands t .. t + 7 at offset u (t wave-uniform).
template <int NS>
struct SampleCounter {
  uint32_t sp[NS];
  __device__ __forceinline__ SampleCounter(const DevView& v, uint32_t u) {
#pragma unroll
    for (int k = 0; k < NS; ++k) sp[k] = centre(wrap_add(uniform(v.lat)[k], u));
  }
  __device__ __forceinline__ void count8(const DevView& v, uint32_t t, uint32_t c[4]) const {
    const BN_UNIFORM int* ip = uniform((const int*)(v.ihp + t));
    int nn[8], dd[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) nn[i] = ip[2 * i], dd[i] = ip[2 * i + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t n0 = (uint32_t)nn[2 * i], n1 = (uint32_t)nn[2 * i + 1];
      const int thr0 = -dd[2 * i] - 1, thr1 = -dd[2 * i + 1] - 1;
      uint32_t a = 0;
      // four samples' residues first, then their sign words: a v_perm then
      // reads a v_dot2 result several instructions after it
      constexpr int G = NS < 4 ? NS : 4;
#pragma unroll
      for (int k = 0; k < NS; k += G) {
        int r0[4], r1[4];
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < G; ++e) r0[e] = dot2(n0, sp[k + e], thr0), r1[e] = dot2(n1, sp[k + e], thr1);
#pragma unroll
        for (int e = 0; e < G; ++e) w[e] = sign_bytes(r0[e], r1[e]);
        if (G == 4) a = a + w[0] + w[1], a = a + w[2] + w[3];
        else if (G == 2) a = a + w[0] + w[1];
        else a += w[0];
      }
      c[i] = (NS | (NS << 16)) - halves_div255(a);
    }
  }
};

// v_med3_i32 (x clamped to [lo, hi] for lo <= hi).
__device__ inline int med3(int x, int lo, int hi) { return max(min(x, lo), min(max(x, lo), hi)); }

// One LineRec out of the 16 words of a pair.
typedef int i32x16 __attribute__((ext_vector_type(16)));
struct LineTerms {
  uint32_t n;
  int d, inv_hi;
  double inv;
  unsigned long long off, slope;
  __device__ __forceinline__ LineTerms(const i32x16 q, int k) : n((uint32_t)q[k]), d(q[k + 1]), inv_hi(q[k + 3]) {
    auto two = [&](int i) { return (unsigned long long)(uint32_t)q[i] | ((unsigned long long)(uint32_t)q[i + 1] << 32); };
    inv = __builtin_bit_cast(double, two(k + 2));
    off = two(k + 4);
    slope = two(k + 6);
  }
};
static_assert(sizeof(LineRec) == 32, "LineTerms reads 8 words per integrand");

template <int R>
struct LineCounter {
  static constexpr double MAGIC = 0x1.8p20;      // a sum with it has 32 fraction bits in the low word
  static constexpr int BIAS = 0x41380000;        // its high word
  uint32_t u, a;                                 // offset; centred sample A
  int start;                                     // -(sum of lo, all lines, with their bias)
  int lo[R], hi[R];
  __device__ __forceinline__ LineCounter(const DevView& v, uint32_t u_) : u(u_) {
    const uint32_t sh = 16 - v.log2n;
    const uint32_t ux = u & 0xFFFFu, uy = u >> 16;
    const uint32_t cls = ((uy >> sh) * v.gx - (ux >> sh) * v.gy) & (v.n - 1);
    constexpr uint32_t W = line_row_words(R);
    uint32_t w[W];
    const u32x4* row = (const u32x4*)(v.lrow + (size_t)cls * W);
#pragma unroll
    for (uint32_t i = 0; i < W / 4; ++i) {
      const u32x4 q = row[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * i + e] = q[e];
    }
    const uint32_t fm = (1u << sh) - 1;
    const uint32_t ax = ((w[0] & 0xFFFFu) << sh) + (ux & fm), ay = ((w[0] >> 16) << sh) + (uy & fm);
    a = centre(ax | (ay << 16));
    start = -(int)w[1] - (int)((uint32_t)R * (uint32_t)BIAS);
#pragma unroll
    for (int l = 0; l < R; ++l) {
      lo[l] = (int)(int16_t)(w[2 + l] & 0xFFFFu) + BIAS;
      hi[l] = ((int)w[2 + l] >> 16) + BIAS;
    }
  }
  // Hits of an integrand whose edge is nearly along the lines.
  __device__ __forceinline__ uint32_t flat(const DevView& v, const BN_UNIFORM int* w) const {
    const double inv = *(const BN_UNIFORM double*)(w + 4), m2 = *(const BN_UNIFORM double*)(w + 6);
    double x = (double)w[1] + 0.5 - (double)dot2((uint32_t)w[0], a, 0);
    uint32_t s = (uint32_t)start;
#pragma unroll
    for (int l = 0; l < R; ++l) {
      int k;
      asm("v_cvt_i32_f64 %0, %1" : "=v"(k) : "v"(floor(x * inv)));   // saturates, as the addition does
      s += (uint32_t)med3(__builtin_elementwise_add_sat(k, BIAS + 1), lo[l], hi[l]);
      x -= m2;
    }
    return inv > 0.0 ? v.n - s : s;
  }
  __device__ __forceinline__ void count8(const DevView& v, uint32_t t, uint32_t c[4]) const {
    const BN_UNIFORM i32x16* rec = uniform((const i32x16*)(v.lrec + t));
    // all pairs' terms load while the first is counted
    i32x16 pair[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) pair[i] = rec[i];
    uint32_t plain = 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const LineTerms q0(pair[i], 0), q1(pair[i], 8);
      unsigned long long x0 = __builtin_bit_cast(unsigned long long,
                                                 __fma_rn((double)dot2(q0.n, a, 0), q0.inv, MAGIC));
      unsigned long long x1 = __builtin_bit_cast(unsigned long long,
                                                 __fma_rn((double)dot2(q1.n, a, 0), q1.inv, MAGIC));
      uint32_t s0 = (uint32_t)start, s1 = (uint32_t)start;
      x0 += q0.off;
      x1 += q1.off;
#pragma unroll
      for (int l = 0; l < R; l += 2) {
        const int k00 = med3((int)(x0 >> 32), lo[l], hi[l]), k10 = med3((int)(x1 >> 32), lo[l], hi[l]);
        x0 += q0.slope;
        x1 += q1.slope;
        const int k01 = med3((int)(x0 >> 32), lo[l + 1], hi[l + 1]), k11 = med3((int)(x1 >> 32), lo[l + 1], hi[l + 1]);
        s0 = s0 + (uint32_t)k00 + (uint32_t)k01;
        s1 = s1 + (uint32_t)k10 + (uint32_t)k11;
        if (l + 2 < R) {
          x0 += q0.slope;
          x1 += q1.slope;
        }
      }
      // s counts the samples before the crossing: the misses where m > 0
      // (inv < 0), the hits where m < 0; per half N - s = (s ^ 0xFFFF) + N + 1
      // less the carry out of the half
      const bool g0 = q0.inv_hi < 0, g1 = q1.inv_hi < 0;
      const uint32_t flip = (g0 ? 0xFFFFu : 0u) | (g1 ? 0xFFFF0000u : 0u);
      const uint32_t add = (g0 ? v.n + 1u - 0x10000u : 0u) + (g1 ? (v.n + 1u) << 16 : 0u);
      c[i] = ((s0 | (s1 << 16)) ^ flip) + add;
      plain = min(plain, min((uint32_t)q0.inv_hi, (uint32_t)q1.inv_hi));
    }
    if (plain == 0) {
#pragma unroll 1
      for (int i = 0; i < 8; ++i) {
        const BN_UNIFORM int* w = (const BN_UNIFORM int*)rec + 8 * i;
        if (w[3] != 0) continue;
        const uint32_t h = flat(v, w) << (16 * (i & 1)), keep = i & 1 ? 0xFFFFu : 0xFFFF0000u;
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = k == i >> 1 ? (c[k] & keep) | h : c[k];
      }
    }
  }
};

// Counts of one chunk of tch integrands (a multiple of 32) for 64 work items.
// MODE_ALL also writes the FP32 error vectors [P][Tp]: 32 integrands' counts
// of the wave's pixels change hands through LDS, so that eight lanes write one
// pixel's whole 128-byte line.
constexpr uint32_t ERR_PITCH = 17;   // words of a pixel's 32 counts in LDS

template <class Counter, int MODE>
__device__ __forceinline__ void count_body(const DevView& v, uint32_t kappa, uint32_t m, uint32_t tch, uint32_t blk,
                                           uint32_t* lds) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(blk * 4 + (threadIdx.x >> 6));
  const uint32_t nch = (v.tp + tch - 1) / tch;
  const uint32_t jg = wave / nch, ch = wave - jg * nch;
  if (jg * 64 >= m) return;
  // lanes past the last item repeat it and store nothing
  const uint32_t j0 = jg * 64 + lane;
  const bool live = j0 < m;
  const uint32_t j = live ? j0 : m - 1;
  uint32_t p, u, row, rows;
  uint16_t* wide;
  int8_t* narrow;
  count_target<MODE>(v, kappa, j, m, p, u, wide, narrow, row, rows);
  const bool to_wide = MODE == MODE_ALL || MODE == MODE_LIST || v.form == FIELD_WIDE;
  const bool to_narrow = MODE != MODE_LIST && v.form != FIELD_WIDE;
  if ((MODE == MODE_CLASS || MODE == MODE_SWEEP) && ch == 0 && live) v.u_new[j] = u;
  if (MODE == MODE_ALL && v.seen && ch == 0 && live) v.seen[p] = u;
  const Counter counter(v, u);
  const float inv_n = 1.0f / (float)v.n;
  const uint32_t t0 = ch * tch, t1 = min(t0 + tch, v.tp), tz = min(t1, (v.t + 7) & ~7u);
  uint32_t* el = lds + (MODE == MODE_ALL ? (threadIdx.x >> 6) * 64 * ERR_PITCH : 0);
  uint32_t b0 = 0, b1 = 0;   // narrow counts of the first half of a 16-integrand word
#pragma unroll 1
  for (uint32_t t = t0; t < t1; t += 8) {
    uint32_t c[4] = {0, 0, 0, 0};   // padded integrands count 0
    if (t < tz) counter.count8(v, t, c);
    // computed in every lane (an empty asm consumes them): otherwise the
    // counting would move under the store's branch
    asm volatile("" : : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
    if (to_wide && live) *(uint4*)(wide + tix(row, t, rows)) = make_uint4(c[0], c[1], c[2], c[3]);
    if (to_narrow) {
      // per half count - base + 128 (no borrow between the halves), then
      // the low bytes, less 128
      const BN_UNIFORM uint32_t* bias = uniform(v.bias8) + t / 2;
      const uint32_t w0 = __builtin_amdgcn_perm(c[1] + bias[1], c[0] + bias[0], 0x06040200u) ^ 0x80808080u;
      const uint32_t w1 = __builtin_amdgcn_perm(c[3] + bias[3], c[2] + bias[2], 0x06040200u) ^ 0x80808080u;
      if (!(t & 8)) {
        b0 = w0;
        b1 = w1;
      } else if (live) {
        *(uint4*)(narrow + ((size_t)(t >> 4) * rows + row) * 16) = make_uint4(b0, b1, w0, w1);
      }
    }
    if (MODE == MODE_ALL) {
      const uint32_t e = (t - t0) & 31;
#pragma unroll
      for (int i = 0; i < 4; ++i) el[lane * ERR_PITCH + e / 2 + i] = c[i];
      if (e == 24) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t tb = t - 24 + 4 * (lane & 7);
        const float4 ar = *(const float4*)(v.area + tb);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t q = 8 * i + (lane >> 3), jq = jg * 64 + q;
          const uint32_t w0 = el[q * ERR_PITCH + 2 * (lane & 7)], w1 = el[q * ERR_PITCH + 2 * (lane & 7) + 1];
          float4 o;
          o.x = (float)(w0 & 0xFFFFu) * inv_n - ar.x;
          o.y = (float)(w0 >> 16) * inv_n - ar.y;
          o.z = (float)(w1 & 0xFFFFu) * inv_n - ar.z;
          o.w = (float)(w1 >> 16) * inv_n - ar.w;
          if (jq < m) *(float4*)(v.err + (size_t)jq * v.tp + tb) = o;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

// The launch may have fewer workgroups than the vblocks its work needs (the
// sweep-wide recount of the overlapped schedule is capped so that it leaves
// room on every CU for the colour phases running beside it): workgroups then
// stride over the virtual blocks.
template <class Counter, int MODE>
__global__ __launch_bounds__(256) void k_count(DevView v, uint32_t kappa, uint32_t m, uint32_t tch,
                                               uint32_t vblocks) {
  __shared__ uint32_t lds[MODE == MODE_ALL ? 4 * 64 * ERR_PITCH : 1];
  for (uint32_t b = blockIdx.x; b < vblocks; b += gridDim.x) count_body<Counter, MODE>(v, kappa, m, tch, b, lds);
}

// Batched form: member i owns blocks pre[i] .. pre[i+1]-1; the proposals of
// every pixel of the sweep kappa steps ahead of the member's sweep counter
// (the overlapped schedule's sweep-wide recount).
template <class Counter>
__global__ __launch_bounds__(256) void k_count_batch(const DevView* __restrict__ views,
                                                     const uint32_t* __restrict__ pre, uint32_t nmem,
                                                     uint32_t kappa) {
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  const DevView v = views[i];
  count_body<Counter, MODE_SWEEP>(v, kappa, v.w * v.h, v.tch, blockIdx.x - pre[i], nullptr);
}

// The integrand chunk of a wave: v.tch, halved while a launch over m items
// would hold under 8192 waves.
inline uint32_t count_chunk(const DevView& v, uint32_t m, uint32_t tch) {
  const uint64_t groups = (m + 63) / 64;
  while (tch > 32 && groups * ((v.tp + tch - 1) / tch) < 8192) tch = ((tch >> 1) + 31) & ~31u;
  return tch;
}

inline uint32_t count_vblocks(const DevView& v, uint32_t m, uint32_t tch) {
  return (uint32_t)(((uint64_t)((m + 63) / 64) * ((v.tp + tch - 1) / tch) + 3) / 4);
}

// Calls f with the counter of launch kind `kind` (N up to 8, else 16 + the
// line counter's template size).
template <class F>
hipError_t with_counter(int kind, F f) {
#define BN_LINES(R) case 16 + R: return f((LineCounter<R>*)nullptr);
  switch (kind) {
    case 1: return f((SampleCounter<1>*)nullptr);
    case 2: return f((SampleCounter<2>*)nullptr);
    case 4: return f((SampleCounter<4>*)nullptr);
    case 8: return f((SampleCounter<8>*)nullptr);
    BN_LINE_TEMPLATES(BN_LINES)
    default: return hipErrorInvalidValue;
  }
#undef BN_LINES
}

template <int MODE>
hipError_t count_dispatch(const DevView& v, uint32_t kappa, uint32_t m, hipStream_t s) {
  if (m == 0) return hipSuccess;
  const uint32_t tch = count_chunk(v, m, v.tch);
  const uint32_t vb = count_vblocks(v, m, tch);
  // a capped launch gets the fewest rounds the cap allows and as few
  // workgroups as those rounds need, so that every workgroup strides over the
  // same number of blocks
  uint32_t nb = vb;
  if (MODE == MODE_SWEEP && v.count_cap && vb > v.count_cap) {
    const uint32_t rounds = (vb + v.count_cap - 1) / v.count_cap;
    nb = (vb + rounds - 1) / rounds;
  }
  return with_counter(count_kind(v), [&](auto* c) {
    using Counter = std::remove_pointer_t<decltype(c)>;
    hipLaunchKernelGGL((k_count<Counter, MODE>), dim3(nb), dim3(256), 0, s, v, kappa, m, tch, vb);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_count(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s) {
  switch (mode) {
    case MODE_ALL: return count_dispatch<MODE_ALL>(v, kappa, m, s);
    case MODE_CLASS: return count_dispatch<MODE_CLASS>(v, kappa, m, s);
    case MODE_SWEEP: return count_dispatch<MODE_SWEEP>(v, kappa, m, s);
    default: return count_dispatch<MODE_LIST>(v, kappa, m, s);
  }
}

// Launch kind of a problem's counting kernel: N up to 8, else 16 + the line
// counter's template size.
int count_kind(const DevView& v) { return v.lines ? 16 + (int)v.lines : (int)v.n; }

uint32_t count_blocks(const DevView& v) { return count_vblocks(v, v.w * v.h, v.tch); }

hipError_t launch_count_batch(int kind, const DevView* views, const uint32_t* pre, uint32_t nmem,
                              uint32_t blocks, uint32_t kappa, hipStream_t s) {
  return with_counter(kind, [&](auto* c) {
    using Counter = std::remove_pointer_t<decltype(c)>;
    hipLaunchKernelGGL(k_count_batch<Counter>, dim3(blocks), dim3(256), 0, s, views, pre, nmem, kappa);
    return hipGetLastError();
  });
}

}  // namespace bnlat
