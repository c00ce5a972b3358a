// gfx950 sampler query: sample k of screen pixel p for every dimension pair of
// a padded screen-space sampler (Sec. 3.1: dimensions are consumed in pairs,
// each pair with its own tile; Sec. 3.2: s^k_p = mod(Phi(k) d + u_p, 1) with
// the rank-1 lattice in van der Corput order).  Values are exact: Q0.16
// coordinates converted to float.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sampler_dev.h"

namespace bnlat {
namespace {

// A workgroup takes 256 queries and walks the pairs, a thread per query, so that
// a pair's fields and the query's parts are loaded once; the samples change
// hands in LDS, eight pairs at a time, so that whole runs of a query's row are
// written.  Bound by the offsets' and lattice points' gathers.  260 000 queries of
// six pairs: 13.1 us; 18 with a thread per (query, pair), each dividing 64-bit
// indexes.
constexpr uint32_t QUERIES = 256, RUN = 8;

__global__ __launch_bounds__(QUERIES) void k_sample(SamplerPairs pairs, uint32_t first, uint32_t count, uint32_t npairs,
                                                    const uint32_t* __restrict__ x, const uint32_t* __restrict__ y,
                                                    const uint32_t* __restrict__ k, uint32_t m,
                                                    float* __restrict__ out) {
  __shared__ uint32_t sample[QUERIES * (RUN + 1)];
  const uint32_t tid = threadIdx.x, j0 = blockIdx.x * QUERIES, j = min(j0 + tid, m - 1);
  const uint32_t qx = x[j], qy = y[j], qk = k[j];
  const float inv = 1.0f / 65536.0f;
  for (uint32_t d0 = 0; d0 < count; d0 += RUN) {
    const uint32_t run = min(RUN, count - d0);
    for (uint32_t d = 0; d < run; ++d) {
      const SamplerPair& pr = pairs.pair[d0 + d];
      const uint32_t kk = qk & (pr.n - 1);
      const uint32_t li = pr.log2n ? (__brev(kk) >> (32 - pr.log2n)) : 0u;
      const uint32_t l = pr.lat[li], u = pr.U[qy % pr.h * pr.w + qx % pr.w];
      sample[tid * (RUN + 1) + d] = ((l + u) & 0xFFFFu) | (((l >> 16) + (u >> 16)) << 16);
    }
    __syncthreads();
    // (out may lie on any float: a component per store)
    const uint32_t n = min(QUERIES, m - j0) * run * 2;
    for (uint32_t i = tid; i < n; i += QUERIES) {
      const uint32_t q = (i >> 1) / run, d = (i >> 1) - q * run, s = sample[q * (RUN + 1) + d];
      out[((size_t)(j0 + q) * npairs + first + d0 + d) * 2 + (i & 1)] = (float)(i & 1 ? s >> 16 : s & 0xFFFFu) * inv;
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_sample(const SamplerPairs& pairs, uint32_t first, uint32_t count, uint32_t npairs, const uint32_t* x,
                         const uint32_t* y, const uint32_t* k, uint32_t m, float* out, hipStream_t s) {
  if (!m || !count) return hipSuccess;
  hipLaunchKernelGGL(k_sample, dim3((m - 1) / QUERIES + 1), dim3(QUERIES), 0, s, pairs, first, count, npairs, x, y, k, m,
                     out);
  return hipGetLastError();
}

}  // namespace bnlat
