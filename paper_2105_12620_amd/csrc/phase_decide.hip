// gfx950 decisions of a colour phase whose integrands are split over workgroups.
//
// The phase kernels (phase_gram.h, phase_wide.hip) give a workgroup its class pixels
// and, where those fill the chip, every integrand.  Where they do not, each
// workgroup takes a slice of the integrands and stores its class sums, and a wave
// per class pixel adds the slices here (lane c + 32 m: class c of every second
// slice), takes the FP64 weighted sum in increasing distance and decides: the same
// integers, the same sum.  Bound by the latency of its loads (4 us at 32 slices of
// 256 class pixels).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "bnlat_dev.h"
#include "device_common.h"

namespace bnlat {
namespace {

template <int R>
__device__ __forceinline__ void decide_body(const DevView& v, uint32_t kappa, uint32_t j) {
  constexpr int NCLS = WinConst<R>::NCLS;
  constexpr uint32_t ROW = NCLS + 1;
  static_assert(ROW <= 32, "a lane per class and the self term");
  if (j >= v.pc || (v.mfma && !v.accept[j])) return;
  const uint32_t lane = threadIdx.x & 63, c = lane & 31;
  long long x = 0;
  if (c < ROW) {
    const long long* q = v.xsum + (size_t)j * ROW + c;
#pragma unroll 8
    for (uint32_t z = lane >> 5; z < v.slices; z += 2) x += q[(size_t)z * v.pc * ROW];
  }
  x += __shfl_xor(x, 32);
  const long long self = __shfl(x, NCLS);
  const double term = c < (uint32_t)NCLS ? __dmul_rn(v.wd[c], (double)((long long)WinConst<R>::w.csize[c] * self - 2 * x)) : 0.0;
  const uint2 t = __builtin_bit_cast(uint2, term);
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < NCLS; ++k)
    sum = __dadd_rn(sum, __builtin_bit_cast(double, make_uint2(__builtin_amdgcn_readlane(t.x, k),
                                                              __builtin_amdgcn_readlane(t.y, k))));
  if (lane != 0) return;
  const uint32_t a = j / v.cw, b = j - a * v.cw, ky = kappa / v.k, kx = kappa - ky * v.k;
  decide_move(v, kappa, j, (ky + v.k * a) * v.w + kx + v.k * b, sum);
}

template <int R>
__global__ __launch_bounds__(256) void k_phase_decide(DevView v, uint32_t kappa) {
  __builtin_amdgcn_s_setprio(2);
  decide_body<R>(v, kappa, wave_id());
}

template <int R>
__global__ __launch_bounds__(256) void k_phase_decide_batch(const DevView* __restrict__ views,
                                                            const uint32_t* __restrict__ pre, uint32_t nmem,
                                                            uint32_t kappa) {
  __builtin_amdgcn_s_setprio(2);
  const uint32_t i = batch_member(pre, nmem, blockIdx.x);
  const DevView v = views[i];
  decide_body<R>(v, kappa, __builtin_amdgcn_readfirstlane((blockIdx.x - pre[i]) * 4 + (threadIdx.x >> 6)));
}

template <class F>
hipError_t by_radius(uint32_t radius, F f) {
  switch (radius) {
    case 1: return f(std::integral_constant<int, 1>());
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    case 5: return f(std::integral_constant<int, 5>());
    case 6: return f(std::integral_constant<int, 6>());
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Slices of at least two stages of 64 integrands, as many as give a workgroup per CU,
// from twelve stages on: a stage takes about a microsecond, the decisions' launch
// 4 to 5.  Per sweep of four phases, int8 operands, 32^2 and 64^2, whole and split:
// T = 256 60 and 73 us, 512 77 and 76 (one colour class: 34 and 38), 1024 108 and 80,
// 4096 290 and 90 (by 4 stages 94, by 8 112), 16384 1023 and 137; 128^2 (64
// workgroups) T = 4096 311 and 156 (128 workgroups: 212, 512: 179); uint16 operands,
// 32^2, T = 4096 814 and 260, where the recount takes the rest.
uint32_t phase_slices(const DevView& v, uint32_t blocks) {
  constexpr uint32_t CUS = 256;
  const uint32_t stages = (v.t + 63) / 64;
  if (stages < 12) return 1;
  const uint32_t most = std::max(1u, std::min(CUS / blocks, stages / 2)), per = (stages + most - 1) / most;
  return (stages + per - 1) / per;
}

hipError_t launch_phase_decide(const DevView& v, uint32_t kappa, hipStream_t s) {
  return by_radius(v.radius, [&](auto r) {
    hipLaunchKernelGGL(k_phase_decide<r()>, dim3((v.pc + 3) / 4), dim3(256), 0, s, v, kappa);
    return hipGetLastError();
  });
}

uint32_t decide_blocks(const DevView& v) { return v.slices > 1 ? (v.pc + 3) / 4 : 0; }

hipError_t launch_phase_decide_batch(uint32_t radius, const DevView* views, const uint32_t* pre, uint32_t nmem,
                                     uint32_t blocks, uint32_t kappa, hipStream_t s) {
  return by_radius(radius, [&](auto r) {
    hipLaunchKernelGGL(k_phase_decide_batch<r()>, dim3(blocks), dim3(256), 0, s, views, pre, nmem, kappa);
    return hipGetLastError();
  });
}

}  // namespace bnlat
