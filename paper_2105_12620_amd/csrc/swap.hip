// gfx950 kernels of the swap mutation (Sec. 3.4, with the pixel permutation
// of Sec. 2): the tile is optimised by exchanging the offsets of couples of
// pixels.  A couple's hit-count vectors move with its offsets, so a pass is a
// pure neighbourhood evaluation with no recount.
//
// The couple (a, b) changes the windowed energy of Eq. (1) by the two single
// moves c_a -> c_b and c_b -> c_a evaluated on the unmodified state plus a
// pair correction.  With dc = c_b - c_a, in exact integers per distance class d:
//   X_d = -2 sum_{o in d} sum_t dc_t (c_{a+o,t} - c_{b+o,t})  +  2 m_d sum_t dc_t^2,
// where m_d counts the offsets o of class d with a + o = b on the torus (the
// terms |d| (c_b^2 - c_a^2) of the two single moves cancel).  Then
//   dE = (2 / N^2) sum_d w(d) X_d,
// summed in FP64 in increasing d exactly as for the redraw mutation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "bnlat_dev.h"
#include "device_common.h"
#include "swap_dev.h"

namespace bnlat {
namespace {

// XOR mask of pass kappa of the sweep in the device counter.
__device__ inline uint32_t swap_mask(const DevView& v, uint32_t kappa) {
  const uint32_t sweep = (uint32_t)v.ctr[0];
  return philox_w01(kappa, sweep, v.problem, S_SWAP, v.seed_lo, v.seed_hi).x & (v.w * v.h - 1);
}

// LDS-staged member evaluation.  A workgroup owns a BW x BH block of tile
// pixels; its pass members (pixels whose scrambled list position falls in the
// pass) are listed in LDS.  For one stage at a time, two planes of 16-byte words
// (8 integrands' counts, or 16 int8 deviations where every |count - base| is at
// most 63: half the words, and v_dot4 in place of v_dot2), the counts of the block plus its window halo (region
// RH x RW, row pitch RWP = RW + 1) and the two partner words of every member
// are staged in LDS, and every member is served by a group of 16 lanes: lane
// (i, p) forms dc = c_partner - c_own of plane p and, per step, reads one
// 16-byte word of plane p at window offset i of the step.  A row step covers
// eight consecutive offsets of a window row, a column step eight consecutive
// rows of one of the columns the row steps leave over.  gfx950's LDS serves a
// ds_read_b128 in passes of 16 lanes over 64 four-byte banks: with the plane
// stride 8 words of 16 bytes past a multiple of 16 and RWP odd, the 16 words
// a group reads fall in 16 distinct bank quads wherever the member lies, so
// every pass is conflict-free.
//
// Staging is a ring of three stage buffers filled straight from HBM by
// global_load_lds_dwordx4 (lane l of a load writes 16 bytes at the wave's LDS
// base + 16 l): the loads of stage s + 2 are issued while stage s is
// evaluated.  Every wave issues the same number D of loads per stage (slots
// past the stage's loads repeat one of them), so waiting for stage s is
// s_waitcnt vmcnt(D) while stage s + 1 is in flight (loads return in order),
// followed by a barrier without a memory fence (a fence would wait for every
// load in flight).  A stage buffer is refilled only after the barrier that
// follows the last reads of it.
//
// A lane accumulates its product of each step separately (int32 per step);
// when the member's integrand slice is done, the steps' sums are added into
// distance classes (the lane's offset of a step fixes the class) by 64-bit
// atomics in LDS and stored, a row of classes per member and slice; the
// decision adds the slices.  (Gathering the classes in registers took 2200
// instructions a round, more than half of the narrow form's stages, and 64-bit
// atomics of the slices into one row go to memory on this part.)  The workgroups are renumbered
// per XCD (xcd_block), so that the blocks one L2 serves at a time are whole
// rows of blocks of one integrand slice and their halos are read from HBM
// once.
//
// Integrand slices of the tile run in separate workgroups; per-lane int32
// step sums stay below 2^31 because the host bounds a slice to S stages with
// S * 8 N^2 < 2^31 (eight products of at most N^2 per lane and stage; sixteen of
// at most 126^2 in the int8 form).
//
// 256^2, N = 256, T = 1024, r = 4, K = 2: 47 us per pass (86 on counts with the
// classes gathered in registers), bound by the region's reads through the L2s
// (2.5 times the tile); blocks of 32 x 16 pixels leave one workgroup per CU and
// took 1.15 (1024 threads) to 1.7 times as long per sweep.

// integrands of a stage
constexpr uint32_t SWAP_STAGE(bool narrow) { return narrow ? 32 : 16; }

template <int R>
struct SwapGeom {
  static constexpr int BW = 32, BH = (R <= 4) ? 8 : 4;   // tile pixels per workgroup
  static constexpr int WS = 2 * R + 1;                   // window side
  static constexpr int RW = BW + 2 * R, RH = BH + 2 * R;
  static constexpr int RWP = RW + 1;                     // odd row pitch (16-byte words)
  static constexpr int RA = RH * RWP;                    // words of one plane's region
  static constexpr int RA_PAD = (RA + 63) / 64 * 64;     // whole 64-lane loads
  static constexpr int PLANE = RA_PAD + 8;               // plane stride: 8 past a multiple of 16
  static constexpr int NT = 512;                         // threads
  static constexpr int NWAVE = NT / 64;
  static constexpr int GL = 16;                          // lanes per member group
  static constexpr int GROUPS = NT / GL;
  static constexpr int SLOTS = (R <= 4) ? 3 : 2;         // members per group and round
  static constexpr int CAP = GROUPS * SLOTS;             // members per round
  static constexpr int PART = 2 * CAP;                   // partner words per stage
  static constexpr int SBUF = 2 * PLANE + PART;          // words of one stage buffer
  static constexpr int NBUF = 3;                         // ring depth
  static constexpr int PD = NBUF - 1;                    // stages loaded ahead
  static constexpr int NRL = 2 * RA_PAD / 64;            // region loads per stage
  static constexpr int NLD = NRL + PART / 64;            // loads per stage
  static constexpr int D = (NLD + NWAVE - 1) / NWAVE;    // loads per wave and stage
  static constexpr int RC = WindowSteps<R>::RC, CH = WindowSteps<R>::CH, STEPS = WindowSteps<R>::STEPS;
  static constexpr int LASTROWS = WindowSteps<R>::LASTROWS;
  static constexpr int NPIX = BW * BH;
  static constexpr int NWV = NPIX / 64;                  // waves that test membership
  static constexpr int LDS_BYTES = NBUF * SBUF * 16 + (3 * NPIX + NWV + 8 * STEPS) * 4;
  static_assert(NPIX % 64 == 0 && RWP % 2 == 1 && PLANE % 16 == 8 && PART % 64 == 0, "swap block geometry");
  static_assert(D * NWAVE < 2 * NLD, "repeated load slots");
  static_assert(PD >= 1 && PD <= 3 && (PD - 1) * D < 64, "ring depth and vmcnt");
};

template <int R, bool NARROW>
__global__ __launch_bounds__(SwapGeom<R>::NT, (R <= 4) ? 4 : 2) void k_swap_stage(DevView v, SwapView sv, uint32_t kappa,
                                                                    uint32_t slen, uint32_t gx, uint32_t gy) {
  using G = SwapGeom<R>;
  constexpr int NCLS = WinConst<R>::NCLS;
  extern __shared__ u32x4 lds4[];
  uint32_t* mpos = (uint32_t*)(lds4 + G::NBUF * G::SBUF);   // [NPIX] region word of each member
  uint32_t* mj = mpos + G::NPIX;                   // [NPIX] list slot
  uint32_t* mb = mj + G::NPIX;                     // [NPIX] partner pixel
  uint32_t* wcnt = mb + G::NPIX;                   // [NWV] members per wave
  int* ctab = (int*)(wcnt + G::NWV);               // [STEPS][8] class of each step's slot (-1: none)
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t P = v.w * v.h;
  const uint32_t mask = swap_mask(v, kappa);
  const uint32_t wk = xcd_block(blockIdx.x, gridDim.x);
  const uint32_t bxy = wk % (gx * gy), bz = wk / (gx * gy);
  const uint32_t x0 = (bxy % gx) * G::BW, y0 = (bxy / gx) * G::BH;

  // members of the block, in raster order
  bool in = false;
  uint32_t j = 0, b = 0, pos = 0;
  if (tid < (uint32_t)G::NPIX) {
    const uint32_t ly = tid / G::BW, lx = tid % G::BW;
    if (y0 + ly < v.h && x0 + lx < v.w) {
      const uint32_t L = sv.pinv[((y0 + ly) * v.w + x0 + lx) ^ mask];
      in = L / sv.m == kappa;
      j = L - kappa * sv.m;
      b = sv.perm[L ^ 1u] ^ mask;
      pos = (ly + R) * G::RWP + lx + R;
    }
  }
  const unsigned long long bal = __ballot(in);
  if (lane == 0 && wv < (uint32_t)G::NWV) wcnt[wv] = (uint32_t)__popcll(bal);
  if (tid < 8u * G::STEPS) {
    int ox, oy;
    ctab[tid] = WindowSteps<R>::offset((int)tid / 8, (int)tid % 8, ox, oy) ? sv.dcls[ox * ox + oy * oy] : -1;
  }
  __syncthreads();
  uint32_t before = 0, nm = 0;
#pragma unroll
  for (int q = 0; q < G::NWV; ++q) {
    if ((uint32_t)q < wv) before += wcnt[q];
    nm += wcnt[q];
  }
  if (in) {
    const uint32_t idx = before + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
    mpos[idx] = pos;
    mj[idx] = j;
    mb[idx] = b;
  }

  // load slot k of this wave issues load d = wv + NWAVE k of a stage (slots
  // past the stage's loads repeat load d - NLD).  Region load d < NRL covers
  // plane d / (RA_PAD / 64), region words 64 (d mod RA_PAD/64) + lane (the
  // padding column and words past the region load pixel 0); partner load d
  // covers partner words 64 (d - NRL) + lane = 2 m + plane of round member m,
  // read from the pixel-major copy (lsrc holds the partner pixel and plane).
  // W and H are powers of two.
  const uint32_t ys = (y0 + v.h * (R / v.h + 1) - R) % v.h;
  const uint32_t xs = (x0 + v.w * (R / v.w + 1) - R) % v.w;
  const uint32_t wm = v.w - 1, hm = v.h - 1;
  uint32_t ldst[G::D], lsrc[G::D];
#pragma unroll
  for (int k = 0; k < G::D; ++k) {
    uint32_t d = wv + G::NWAVE * k;
    if (d >= (uint32_t)G::NLD) d -= G::NLD;
    if (d < (uint32_t)G::NRL) {
      const uint32_t pl = d / (G::RA_PAD / 64), u0 = (d % (G::RA_PAD / 64)) * 64, u = u0 + lane;
      const uint32_t rr = u / G::RWP, cc = u - rr * G::RWP;
      const uint32_t gq = (u < (uint32_t)G::RA && cc < (uint32_t)G::RW) ? ((ys + rr) & hm) * v.w + ((xs + cc) & wm) : 0;
      ldst[k] = pl * G::PLANE + u0;
      lsrc[k] = pl * P + gq;
    } else {
      ldst[k] = 2 * G::PLANE + 64 * (d - G::NRL);
      lsrc[k] = 0;
    }
  }
  // words of a pixel's row; a stage is two planes of words in either form
  const uint32_t rowq = v.tp >> (NARROW ? 4 : 3);
  const u32x4* field = NARROW ? (const u32x4*)sv.field8 : (const u32x4*)v.cnt;
  const u32x4* rowsq = NARROW ? (const u32x4*)sv.row8 : (const u32x4*)sv.row;
  auto issue = [&](uint32_t st, uint32_t buf) {
    const u32x4* cs = field + (size_t)(2 * st) * P;
    const u32x4* rs = rowsq + 2 * st;
#pragma unroll
    for (int k = 0; k < G::D; ++k) {
      const u32x4* src = ldst[k] < 2u * G::PLANE ? cs + lsrc[k] : rs + (size_t)(lsrc[k] >> 1) * rowq + (lsrc[k] & 1);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)(lds4 + buf * G::SBUF + ldst[k]),
                                       16, 0, 0);
    }
  };

  auto dot = [](uint32_t a, uint32_t b, int c) { return NARROW ? dot4(a, b, c) : dot2(a, b, c); };
  const uint32_t grp = tid / G::GL, li = tid & 7, lp = (tid >> 3) & 1;
  // word of the lane's slot relative to the member's own word of plane lp:
  // row steps, column steps, a column's last step (lanes past the window
  // repeat its last offset)
  const uint32_t lr = min(li, (uint32_t)G::RC - 1), lc = li * G::RWP,
                 lcl = min(li, (uint32_t)G::LASTROWS - 1) * G::RWP;
  // the same shifted so that every step reads at a non-negative constant
  // offset, and the partner word of the group's first slot
  const uint32_t rof = lr - (R * G::RWP + R), cof = lc - (R * G::RWP + R - G::RC),
                 clof = lcl - (R * G::RWP + R - G::RC), pe0 = 2 * G::PLANE + 2 * grp + lp;
  const uint32_t st0 = bz * slen, st1 = min(st0 + slen, v.tp / SWAP_STAGE(NARROW));
  const uint32_t nst = st1 > st0 ? st1 - st0 : 0;
  __syncthreads();
  for (uint32_t base = 0; base < nm; base += G::CAP) {
    // this round's partner pixels
#pragma unroll
    for (int k = 0; k < G::D; ++k) {
      if (ldst[k] >= 2u * G::PLANE) {
        // partner word 2 base + e of the round (its member and plane), with
        // the wave-uniform part summed first: kept per load across rounds,
        // the lane parts spilled at radius 4
        const uint32_t e2 = __builtin_amdgcn_readfirstlane(2 * base + ldst[k] - 2 * G::PLANE) + lane,
                       m = e2 >> 1;
        lsrc[k] = (m < nm ? mb[m] : 0) * 2 + (e2 & 1);
      }
    }
    int acc[G::SLOTS][G::STEPS];
    int dd[G::SLOTS];
    // per slot: the member's own word of plane lp; the lane's reads are at
    // fixed offsets from it (one register per slot rather than one per step
    // kind: fewer spills at radius 4)
    uint32_t sp[G::SLOTS];
    bool ok[G::SLOTS];
#pragma unroll
    for (int s = 0; s < G::SLOTS; ++s) {
      const uint32_t mi = grp + G::GROUPS * s;
      ok[s] = base + mi < nm;
      sp[s] = lp * G::PLANE + (ok[s] ? mpos[base + mi] : (uint32_t)(R * G::RWP + R));
      dd[s] = 0;
#pragma unroll
      for (int st = 0; st < G::STEPS; ++st) acc[s][st] = 0;
    }
    // the previous round's reads of the ring are done
    barrier_vm<0>();
#pragma unroll
    for (int k = 0; k < G::PD; ++k)
      if ((uint32_t)k < nst) issue(st0 + k, k);
    for (uint32_t si = 0; si < nst; ++si) {
      // stage si has landed once at most the loads of the stages issued
      // after it (up to PD - 1 of them) are in flight
      const uint32_t ahead = min((uint32_t)G::PD - 1, nst - 1 - si);
      if (G::PD >= 3 && ahead == 2) barrier_vm<2 * G::D>();
      else if (G::PD >= 2 && ahead == 1) barrier_vm<G::D>();
      else barrier_vm<0>();
      if (si + G::PD < nst) issue(st0 + si + G::PD, (si + G::PD) % G::NBUF);
      const u32x4* bf = lds4 + (si % G::NBUF) * G::SBUF;
#pragma unroll
      for (int s = 0; s < G::SLOTS; ++s) {
        if (ok[s]) {
          const u32x4 own = bf[sp[s]], pc = bf[pe0 + 2 * G::GROUPS * s];
          uint32_t dl[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            // partner minus own, per int16 half (|dc| <= N, no wrap) or per
            // byte (|dc| <= 126); the words go through scalars (a bit cast
            // straight from the vector element read only the first word)
            const uint32_t pw_h = pc[h], ow_h = own[h];
            dl[h] = NARROW ? sub_bytes(pw_h, ow_h)
                           : __builtin_bit_cast(uint32_t, (v2i16)(__builtin_bit_cast(v2i16, pw_h) -
                                                                  __builtin_bit_cast(v2i16, ow_h)));
            dd[s] = dot(dl[h], dl[h], dd[s]);
          }
          const u32x4* rp = bf + (sp[s] + rof);
          const u32x4* cp = bf + (sp[s] + cof);
          const u32x4* clp = bf + (sp[s] + clof);
#pragma unroll
          for (int st = 0; st < G::STEPS; ++st) {
            u32x4 c;
            if (st < G::WS) {
              c = rp[st * G::RWP];
            } else {
              const int t = st - G::WS, col = t / G::CH, part = t % G::CH;
              c = (part < G::CH - 1 ? cp : clp)[col + 8 * part * G::RWP];
            }
            int a = acc[s][st];
            a = dot(dl[0], c[0], a);
            a = dot(dl[1], c[1], a);
            a = dot(dl[2], c[2], a);
            acc[s][st] = dot(dl[3], c[3], a);
          }
        }
      }
    }
    // the members' step sums, by class, in the ring's LDS; d2 last
    barrier_vm<0>();
    unsigned long long* sums = (unsigned long long*)lds4;
    constexpr uint32_t ROW = NCLS + 1;
    static_assert(8 * G::CAP * ROW <= 16 * G::NBUF * G::SBUF, "class sums exceed the ring");
    for (uint32_t e = tid; e < G::CAP * ROW; e += G::NT) sums[e] = 0;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < G::SLOTS; ++s) {
      if (!ok[s]) continue;
      unsigned long long* to = sums + (grp + G::GROUPS * s) * ROW;
#pragma unroll
      for (int st = 0; st < G::STEPS; ++st) {
        const int c = ctab[st * 8 + li];
        if (c >= 0) atomicAdd(&to[c], (unsigned long long)(long long)acc[s][st]);
      }
      // dc^2 of plane lp is the same in the group's eight slots
      if (li == 0) atomicAdd(&to[NCLS], (unsigned long long)(long long)dd[s]);
    }
    __syncthreads();
    const uint32_t mr = min(nm - base, (uint32_t)G::CAP);
    for (uint32_t e = tid; e < mr * ROW; e += G::NT) {
      const uint32_t m = e / ROW, c = e - m * ROW, js = mj[base + m];
      const long long x = (long long)sums[e];
      if (c < (uint32_t)NCLS) sv.xs[((size_t)bz * sv.m + js) * NCLS + c] = -2 * x;
      else if (!(js & 1u)) sv.d2[(size_t)bz * (sv.m >> 1) + (js >> 1)] = x;
    }
  }
}

// Decision of couple i by one wave: add the slices' class sums of the two
// members (lane c + 32 m: class c of member m) and the pair correction, take the
// FP64 weighted sum in increasing d and decide.  Writes delta, accept and the
// couple's pixels (u_new); returns the decision and the pixels.
template <int R>
__device__ __forceinline__ bool swap_decide(const DevView& v, const SwapView& sv, uint32_t kappa, uint32_t i,
                                            uint32_t lane, uint32_t& a, uint32_t& b) {
  constexpr int NCLS = WinConst<R>::NCLS;
  static_assert(NCLS < 32, "a lane per class and member, and one for d2");
  const uint32_t mask = swap_mask(v, kappa);
  const uint32_t L = kappa * sv.m + 2 * i;
  a = __builtin_amdgcn_readfirstlane(sv.perm[L] ^ mask);
  b = __builtin_amdgcn_readfirstlane(sv.perm[L + 1] ^ mask);
  const int c = (int)(lane & 31);
  // lane NCLS: the slices' d2
  long long x = 0;
  const bool sq = lane == (uint32_t)NCLS;
  const long long* q = sq ? sv.d2 + i : sv.xs + ((size_t)2 * i + (lane >> 5)) * NCLS + c;
  const size_t step = sq ? sv.m >> 1 : (size_t)sv.m * NCLS;
  if (sq || c < NCLS) {
#pragma unroll 8
    for (uint32_t z = 0; z < sv.slices; ++z) x += q[z * step];
  }
  const long long d2 = __shfl(x, NCLS);
  x += __shfl_xor(x, 32);
  // offsets o with a + o = b on the torus: o = d or d - W per axis with
  // d = (b - a) mod W (two per axis at most because r < min(W, H)); W and H
  // are powers of two
  const uint32_t lw = __builtin_ctz(v.w), wm = v.w - 1, hm = v.h - 1;
  const int dx = (int)(((b & wm) - (a & wm)) & wm), dy = (int)(((b >> lw) - (a >> lw)) & hm);
  const int cx[2] = {dx, dx - (int)v.w}, cy[2] = {dy, dy - (int)v.h};
#pragma unroll
  for (int ky = 0; ky < 2; ++ky) {
#pragma unroll
    for (int kx = 0; kx < 2; ++kx) {
      const int ox = cx[kx], oy = cy[ky];
      if (ox < -R || ox > R || oy < -R || oy > R || (ox == 0 && oy == 0)) continue;
      if (c == sv.dcls[ox * ox + oy * oy]) x += 2 * d2;
    }
  }
  const double term = c < NCLS ? __dmul_rn(v.wd[c], (double)x) : 0.0;
  const uint2 t = __builtin_bit_cast(uint2, term);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < NCLS; ++k)
    acc = __dadd_rn(acc, __builtin_bit_cast(double, make_uint2(__builtin_amdgcn_readlane(t.x, k),
                                                              __builtin_amdgcn_readlane(t.y, k))));
  const double total = __dmul_rn(acc, 2.0 / ((double)v.n * (double)v.n));
  const bool ok = (v.objective > 0) ? (total < 0.0) : (total > 0.0);
  if (lane == 0) {
    v.delta[i] = total;
    v.accept[i] = ok;
    v.u_new[2 * i] = a;
    v.u_new[2 * i + 1] = b;
  }
  return __builtin_amdgcn_readfirstlane(ok ? 1u : 0u) != 0;
}

// Exchange of an accepted couple's offsets and count tiles by one wave: the
// counts are read from the pixel-major copy (whole lines), written to both
// layouts.
__device__ __forceinline__ void swap_exchange(const DevView& v, const SwapView& sv, uint32_t a, uint32_t b,
                                              uint32_t lane) {
  if (lane == 0) {
    const uint32_t ua = v.U[a], ub = v.U[b];
    v.U[a] = ub;
    v.U[b] = ua;
  }
  const uint32_t P = v.w * v.h;
  if (sv.row8) {
    u32x4* wa = (u32x4*)(sv.row8 + (size_t)a * v.tp);
    u32x4* wb = (u32x4*)(sv.row8 + (size_t)b * v.tp);
    for (uint32_t tt = lane; tt < (v.tp >> 4); tt += 64) {
      const u32x4 qa = wa[tt], qb = wb[tt];
      wa[tt] = qb;
      wb[tt] = qa;
      *(u32x4*)(sv.field8 + ((size_t)tt * P + a) * 16) = qb;
      *(u32x4*)(sv.field8 + ((size_t)tt * P + b) * 16) = qa;
      uint4 lo, hi;
      widen8(qb, v.bias8 + 8 * tt, lo, hi);
      *(uint4*)(v.cnt + ((size_t)(2 * tt) * P + a) * 8) = lo;
      *(uint4*)(v.cnt + ((size_t)(2 * tt + 1) * P + a) * 8) = hi;
      widen8(qa, v.bias8 + 8 * tt, lo, hi);
      *(uint4*)(v.cnt + ((size_t)(2 * tt) * P + b) * 8) = lo;
      *(uint4*)(v.cnt + ((size_t)(2 * tt + 1) * P + b) * 8) = hi;
    }
    return;
  }
  uint4* wa = (uint4*)(sv.row + (size_t)a * v.tp);
  uint4* wb = (uint4*)(sv.row + (size_t)b * v.tp);
  for (uint32_t tt = lane; tt < (v.tp >> 3); tt += 64) {
    const uint4 qa = wa[tt], qb = wb[tt];
    wa[tt] = qb;
    wb[tt] = qa;
    *(uint4*)(v.cnt + ((size_t)tt * P + a) * 8) = qb;
    *(uint4*)(v.cnt + ((size_t)tt * P + b) * 8) = qa;
  }
}

// One wave per couple: the decision alone (the phase-stepping calls).
template <int R>
__global__ __launch_bounds__(256) void k_swap_finish(DevView v, SwapView sv, uint32_t kappa) {
  const uint32_t i = wave_id();
  if (i >= (sv.m >> 1)) return;
  uint32_t a, b;
  (void)swap_decide<R>(v, sv, kappa, i, threadIdx.x & 63, a, b);
}

// One wave per couple: decision and, if accepted, the exchange (the sweeps:
// one launch less per pass, and no round trip of the decision through HBM).
// The accepted couples are counted by workgroup: a 64-bit atomic goes to memory,
// and one per couple took 4 of the launch's 17 us at 256^2 (13 now, bound by the
// latency of its dependent loads).
constexpr uint32_t EXCHANGE_WAVES = 16;

__device__ __forceinline__ void count_accept(const DevView& v, uint32_t* n, bool ok, uint32_t lane) {
  if (ok && lane == 0) atomicAdd(n, 1u);
  __syncthreads();
  if (threadIdx.x == 0 && *n) atomicAdd(&v.ctr[1], (unsigned long long)*n);
}

template <int R>
__global__ __launch_bounds__(64 * EXCHANGE_WAVES) void k_swap_decide_exchange(DevView v, SwapView sv, uint32_t kappa) {
  __shared__ uint32_t n;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i = wave_id();
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  uint32_t a = 0, b = 0;
  const bool ok = i < (sv.m >> 1) && swap_decide<R>(v, sv, kappa, i, lane, a, b);
  if (ok) swap_exchange(v, sv, a, b, lane);
  count_accept(v, &n, ok, lane);
}

// One wave per accepted couple: exchange offsets and count tiles.
__global__ __launch_bounds__(64 * EXCHANGE_WAVES) void k_swap_commit(DevView v, SwapView sv) {
  __shared__ uint32_t n;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i = wave_id();
  if (threadIdx.x == 0) n = 0;
  __syncthreads();
  const bool ok = i < (sv.m >> 1) && v.accept[i];
  if (ok) swap_exchange(v, sv, v.u_new[2 * i], v.u_new[2 * i + 1], lane);
  count_accept(v, &n, ok, lane);
}

// int8 deviations from the tiled counts, tiled and pixel-major: thread per
// (pixel, 16-integrand tile), pixels fastest, so that the tiled accesses are
// coalesced.
__global__ __launch_bounds__(256) void k_swap_rows8(DevView v, SwapView sv) {
  const uint32_t P = v.w * v.h;
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (uint64_t)P * (v.tp >> 4)) return;
  const uint32_t tt = (uint32_t)(i / P), p = (uint32_t)(i - (uint64_t)tt * P);
  const u32x4 d = narrow8(*(const uint4*)(v.cnt + ((size_t)(2 * tt) * P + p) * 8),
                          *(const uint4*)(v.cnt + ((size_t)(2 * tt + 1) * P + p) * 8), v.bias8 + 8 * tt);
  *(u32x4*)(sv.field8 + ((size_t)tt * P + p) * 16) = d;
  *((u32x4*)(sv.row8 + (size_t)p * v.tp) + tt) = d;
}

// Pixel-major copy of the tiled counts: thread per (pixel, 8-integrand tile),
// pixels fastest, so that the tiled reads are coalesced.
__global__ __launch_bounds__(256) void k_swap_rows(DevView v, SwapView sv) {
  const uint32_t P = v.w * v.h;
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (uint64_t)P * (v.tp >> 3)) return;
  const uint32_t tt = (uint32_t)(i / P), p = (uint32_t)(i - (uint64_t)tt * P);
  *((uint4*)(sv.row + (size_t)p * v.tp) + tt) = *(const uint4*)(v.cnt + ((size_t)tt * P + p) * 8);
}

}  // namespace

// The staged kernels use more than 64 KiB of LDS per workgroup (gfx950 has
// 160 KiB per CU); the launch limit is raised once per process.
hipError_t prepare_swap_kernels() {
  static hipError_t status = [] {
    hipError_t e = hipSuccess;
#define BN_SWAP_ATTR(RR)                                                                               \
  if (e == hipSuccess)                                                                                 \
    e = hipFuncSetAttribute((const void*)k_swap_stage<RR, false>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                            (int)SwapGeom<RR>::LDS_BYTES);                                             \
  if (e == hipSuccess)                                                                                 \
    e = hipFuncSetAttribute((const void*)k_swap_stage<RR, true>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                            (int)SwapGeom<RR>::LDS_BYTES);
    BN_SWAP_ATTR(1)
    BN_SWAP_ATTR(2)
    BN_SWAP_ATTR(3)
    BN_SWAP_ATTR(4)
    BN_SWAP_ATTR(5)
    BN_SWAP_ATTR(6)
#undef BN_SWAP_ATTR
    return e;
  }();
  return status;
}

// Integrand slices: enough workgroups for about 1024 threads on each of the
// 256 CUs; at least sqrt(stages / 8) stages a slice, for the decision reads every
// slice's sums; and few enough that every per-lane int32 step sum stays below 2^31.
// Sweeps on int8 at r = 4 by least stages a slice: 32^2 (four blocks) T = 256
// 1: 65 us, 2: 72; T = 1024 1: 77, 2: 74, 4: 81; T = 4096 1: 149, 2: 108, 4: 102,
// 8: 115; 8^2 T = 16384 1: 170, 4: 85, 8: 80.
template <int R>
uint32_t stages_per_slice(const DevView& v, const SwapView& sv) {
  using G = SwapGeom<R>;
  const uint32_t blocks = ((v.w + G::BW - 1) / G::BW) * ((v.h + G::BH - 1) / G::BH);
  const uint32_t stages = v.tp / SWAP_STAGE(sv.row8 != nullptr);
  // products per lane and stage, and their bound
  const double per_stage = sv.row8 ? 16.0 * 126.0 * 126.0 : 8.0 * (double)v.n * v.n;
  const uint32_t smax = (uint32_t)std::max(1.0, std::floor(2147483647.0 / per_stage));
  const uint32_t target = 262144 / G::NT;
  const uint32_t least = std::max(1u, (uint32_t)std::sqrt(stages / 8.0));
  const uint32_t nz = std::max<uint32_t>(1, std::min<uint32_t>(stages / least, (target + blocks - 1) / blocks));
  return std::min((stages + nz - 1) / nz, smax);
}

template <int R>
uint32_t slices(const DevView& v, const SwapView& sv) {
  const uint32_t stages = v.tp / SWAP_STAGE(sv.row8 != nullptr), per = stages_per_slice<R>(v, sv);
  return (stages + per - 1) / per;
}

uint32_t swap_slices(const DevView& v, const SwapView& sv) {
  switch (v.radius) {
    case 1: return slices<1>(v, sv);
    case 2: return slices<2>(v, sv);
    case 3: return slices<3>(v, sv);
    case 4: return slices<4>(v, sv);
    case 5: return slices<5>(v, sv);
    default: return slices<6>(v, sv);
  }
}

template <int R>
hipError_t swap_stage_launch(const DevView& v, const SwapView& sv, uint32_t kappa, hipStream_t s, bool decide) {
  using G = SwapGeom<R>;
  const uint32_t gx = (v.w + G::BW - 1) / G::BW, gy = (v.h + G::BH - 1) / G::BH, per = stages_per_slice<R>(v, sv);
  const dim3 grid(gx * gy * sv.slices), block(G::NT);
  if (sv.row8)
    hipLaunchKernelGGL((k_swap_stage<R, true>), grid, block, (size_t)G::LDS_BYTES, s, v, sv, kappa, per, gx, gy);
  else
    hipLaunchKernelGGL((k_swap_stage<R, false>), grid, block, (size_t)G::LDS_BYTES, s, v, sv, kappa, per, gx, gy);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !decide) return e;
  hipLaunchKernelGGL(k_swap_finish<R>, dim3(((sv.m >> 1) + 3) / 4), dim3(256), 0, s, v, sv, kappa);
  return hipGetLastError();
}

hipError_t launch_swap_evaluate(const DevView& v, const SwapView& sv, uint32_t kappa, hipStream_t s, bool decide) {
  switch (v.radius) {
    case 1: return swap_stage_launch<1>(v, sv, kappa, s, decide);
    case 2: return swap_stage_launch<2>(v, sv, kappa, s, decide);
    case 3: return swap_stage_launch<3>(v, sv, kappa, s, decide);
    case 4: return swap_stage_launch<4>(v, sv, kappa, s, decide);
    case 5: return swap_stage_launch<5>(v, sv, kappa, s, decide);
    case 6: return swap_stage_launch<6>(v, sv, kappa, s, decide);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_swap_decide_exchange(const DevView& v, const SwapView& sv, uint32_t kappa, hipStream_t s) {
  const dim3 g(((sv.m >> 1) + EXCHANGE_WAVES - 1) / EXCHANGE_WAVES), b(64 * EXCHANGE_WAVES);
  switch (v.radius) {
    case 1: hipLaunchKernelGGL(k_swap_decide_exchange<1>, g, b, 0, s, v, sv, kappa); break;
    case 2: hipLaunchKernelGGL(k_swap_decide_exchange<2>, g, b, 0, s, v, sv, kappa); break;
    case 3: hipLaunchKernelGGL(k_swap_decide_exchange<3>, g, b, 0, s, v, sv, kappa); break;
    case 4: hipLaunchKernelGGL(k_swap_decide_exchange<4>, g, b, 0, s, v, sv, kappa); break;
    case 5: hipLaunchKernelGGL(k_swap_decide_exchange<5>, g, b, 0, s, v, sv, kappa); break;
    case 6: hipLaunchKernelGGL(k_swap_decide_exchange<6>, g, b, 0, s, v, sv, kappa); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_swap_rows(const DevView& v, const SwapView& sv, hipStream_t s) {
  const uint64_t n = (uint64_t)v.w * v.h * (v.tp >> (sv.row8 ? 4 : 3));
  if (sv.row8) hipLaunchKernelGGL(k_swap_rows8, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, v, sv);
  else hipLaunchKernelGGL(k_swap_rows, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, v, sv);
  return hipGetLastError();
}

hipError_t launch_swap_commit(const DevView& v, const SwapView& sv, hipStream_t s) {
  const uint32_t half = sv.m >> 1;
  hipLaunchKernelGGL(k_swap_commit, dim3((half + EXCHANGE_WAVES - 1) / EXCHANGE_WAVES), dim3(64 * EXCHANGE_WAVES), 0, s, v,
                     sv);
  return hipGetLastError();
}

}  // namespace bnlat
