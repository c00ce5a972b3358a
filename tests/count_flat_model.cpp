// CPU model of the line counter's flat edges (csrc/count.hip, LineCounter::flat)
// on the library's own tables, and the direct count of the samples.
#include <climits>
#include <cmath>
#include <cstring>

#include "../paper_2105_12620_amd/csrc/lattice_lines.h"

using namespace bnlat;

namespace {

// v_cvt_i32_f64 and a saturating addition
int to_int(double x) { return x <= INT_MIN ? INT_MIN : x >= INT_MAX ? INT_MAX : (int)x; }
int add_sat(int a, int b) {
  const long long s = (long long)a + b;
  return s < INT_MIN ? INT_MIN : s > INT_MAX ? INT_MAX : (int)s;
}

}  // namespace

// Flat edges among k (normal, edge point, offset) rows: counts in got (want's
// value for the others), the direct counts in want; returns how many are flat.
extern "C" int count_flat_model(uint32_t n, uint32_t gx, uint32_t gy, uint32_t k, const int16_t* nx, const int16_t* ny,
                                const uint16_t* cx, const uint16_t* cy, const uint16_t* ux, const uint16_t* uy,
                                uint32_t* got, uint32_t* want) {
  const uint32_t step = 65536 / n;
  uint32_t sh = 0;
  while ((1u << sh) < step) ++sh;
  const LatticeLines g = lattice_lines(n, gx, gy);
  const uint32_t R = line_template(g.lines), W = line_row_words(R);
  std::vector<uint32_t> rows;
  if (!g.lines || !R || !lattice_rows(n, gx, gy, g, R, W, rows)) return -1;
  const int BIAS = 0x41380000;
  int flat = 0;
  for (uint32_t i = 0; i < k; ++i) {
    const LineRec q = line_record(g, step, nx[i], ny[i], cx[i], cy[i]);
    uint32_t direct = 0;
    for (uint32_t s = 0; s < n; ++s) {
      const int x = (int)((((uint64_t)s * gx % n) * step + ux[i]) & 0xFFFF) - 32768;
      const int y = (int)((((uint64_t)s * gy % n) * step + uy[i]) & 0xFFFF) - 32768;
      direct += (int64_t)nx[i] * x + (int64_t)ny[i] * y > q.d;
    }
    got[i] = want[i] = direct;
    if (q.inv != 0.0) continue;
    ++flat;
    const uint32_t cls = ((uint32_t)(uy[i] >> sh) * gx - (uint32_t)(ux[i] >> sh) * gy) & (n - 1);
    const uint32_t* w = &rows[(size_t)cls * W];
    const uint32_t fm = (1u << sh) - 1;
    const int ax = (int)(((w[0] & 0xFFFF) << sh) + (ux[i] & fm)) - 32768;
    const int ay = (int)(((w[0] >> 16) << sh) + (uy[i] & fm)) - 32768;
    double inv, m2;
    std::memcpy(&inv, &q.off, 8);
    std::memcpy(&m2, &q.slope, 8);
    double x = (double)q.d + 0.5 - (double)((int)nx[i] * ax + (int)ny[i] * ay);
    uint32_t s = (uint32_t)(-(int)w[1]) - R * (uint32_t)BIAS;
    for (uint32_t l = 0; l < R; ++l) {
      const int lo = (int)(int16_t)(w[2 + l] & 0xFFFF) + BIAS, hi = ((int)w[2 + l] >> 16) + BIAS;
      const int c = add_sat(to_int(std::floor(x * inv)), BIAS + 1);
      s += (uint32_t)std::max(std::min(c, hi), lo);
      x -= m2;
    }
    got[i] = inv > 0.0 ? n - s : s;
  }
  return flat;
}
