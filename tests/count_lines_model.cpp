// CPU model of the line counter (csrc/count.hip) on the library's own tables
// (csrc/lattice_lines.h): the same integer and FP64 operations per line, and
// the direct count of the samples.
#include <cmath>
#include <cstring>

#include "../paper_2105_12620_amd/csrc/lattice_lines.h"

using namespace bnlat;

namespace {

uint64_t bits(double x) {
  uint64_t b;
  std::memcpy(&b, &x, 8);
  return b;
}

int clamp(int x, int lo, int hi) { return std::max(std::min(x, lo), std::min(std::max(x, lo), hi)); }

}  // namespace

// For each of k (normal, edge point, offset) rows: the line count in got, the
// direct count in want.  Returns the lattice's line count, or -1 without one.
extern "C" int count_lines_model(uint32_t n, uint32_t gx, uint32_t gy, uint32_t k, const int16_t* nx, const int16_t* ny,
                                 const uint16_t* cx, const uint16_t* cy, const uint16_t* ux, const uint16_t* uy,
                                 uint32_t* got, uint32_t* want, uint32_t* by_sample) {
  const uint32_t step = 65536 / n;
  uint32_t sh = 0;
  while ((1u << sh) < step) ++sh;
  const LatticeLines g = lattice_lines(n, gx, gy);
  const uint32_t R = line_template(g.lines), W = line_row_words(R);
  std::vector<uint32_t> rows;
  if (!g.lines || !R || !lattice_rows(n, gx, gy, g, R, W, rows)) return -1;
  if ((uint64_t)g.lines * g.lines > 2ull * n) return -1;
  const int BIAS = 0x41380000;
  *by_sample = 0;
  for (uint32_t i = 0; i < k; ++i) {
    const LineRec q = line_record(g, step, nx[i], ny[i], cx[i], cy[i]);
    uint32_t direct = 0;
    for (uint32_t s = 0; s < n; ++s) {
      const int x = (int)((((uint64_t)s * gx % n) * step + ux[i]) & 0xFFFF) - 32768;
      const int y = (int)((((uint64_t)s * gy % n) * step + uy[i]) & 0xFFFF) - 32768;
      direct += (int64_t)nx[i] * x + (int64_t)ny[i] * y > q.d;
    }
    want[i] = direct;
    if (q.inv == 0.0) {
      got[i] = direct;
      ++*by_sample;
      continue;
    }
    const uint32_t cls = ((uint32_t)(uy[i] >> sh) * gx - (uint32_t)(ux[i] >> sh) * gy) & (n - 1);
    const uint32_t* w = &rows[(size_t)cls * W];
    const uint32_t fm = (1u << sh) - 1;
    const int ax = (int)(((w[0] & 0xFFFF) << sh) + (ux[i] & fm)) - 32768;
    const int ay = (int)(((w[0] >> 16) << sh) + (uy[i] & fm)) - 32768;
    const int dot = (int)nx[i] * ax + (int)ny[i] * ay;
    uint64_t x = bits(std::fma((double)dot, q.inv, 0x1.8p20)) + (uint64_t)q.off;
    uint32_t s = (uint32_t)(-(int)w[1]) - R * (uint32_t)BIAS;
    for (uint32_t l = 0; l < R; ++l) {
      const int lo = (int)(int16_t)(w[2 + l] & 0xFFFF) + BIAS, hi = ((int)w[2 + l] >> 16) + BIAS;
      s += (uint32_t)clamp((int)(x >> 32), lo, hi);
      x += (uint64_t)q.slope;
    }
    got[i] = q.inv < 0.0 ? n - s : s;
  }
  return (int)g.lines;
}

// Counts of the padded integrand on every class's lines (all must be 0).
extern "C" int count_lines_padding(uint32_t n, uint32_t gx, uint32_t gy) {
  const LatticeLines g = lattice_lines(n, gx, gy);
  const uint32_t R = line_template(g.lines), W = line_row_words(R);
  std::vector<uint32_t> rows;
  if (!lattice_rows(n, gx, gy, g, R, W, rows)) return -1;
  const LineRec q = line_padding();
  int bad = 0;
  for (uint32_t cls = 0; cls < n; ++cls) {
    const uint32_t* w = &rows[(size_t)cls * W];
    const uint64_t x = bits(std::fma(0.0, q.inv, 0x1.8p20)) + (uint64_t)q.off;
    int s = -(int)w[1];
    for (uint32_t l = 0; l < R; ++l)
      s += clamp((int)(x >> 32) - 0x41380000, (int)(int16_t)(w[2 + l] & 0xFFFF), (int)w[2 + l] >> 16);
    bad += s != 0;
  }
  return bad;
}

// The bound on |count - N area| that decides the operands of the colour phases.
extern "C" uint32_t count_lines_deviation(uint32_t n, uint32_t gx, uint32_t gy) {
  return count_deviation(n, lattice_lines(n, gx, gy));
}

// Gaussian estimates along the lines (csrc/gauss_lines.hip) on the library's
// tables, and the sum over the samples.  Returns the steps of the longest line;
// flagged counts the rows whose exponents the table calls out of range (got is
// then the direct sum).
extern "C" int gauss_lines_model(uint32_t n, uint32_t gx, uint32_t gy, uint32_t k, const double* mx, const double* my,
                                 const double* sd, const uint16_t* ux, const uint16_t* uy, double* got, double* want,
                                 uint32_t* flagged) {
  const LatticeLines g = lattice_lines(n, gx, gy);
  const GaussLines q = gauss_lines(n, gx, gy, g);
  const uint32_t step = 65536 / n;
  uint32_t sh = 0;
  while ((1u << sh) < step) ++sh;
  std::vector<double> four(4 * gauss_table_words(q)), t(gauss_table_words(q));
  *flagged = 0;
  for (uint32_t i = 0; i < k; ++i) {
    const double gm = 1.4426950408889634074 / (2.0 * sd[i] * sd[i]);
    const double a = -gm, bx = 2.0 * gm * mx[i], by = 2.0 * gm * my[i], c = -gm * (mx[i] * mx[i] + my[i] * my[i]);
    long double direct = 0;
    for (uint32_t s = 0; s < n; ++s) {
      const long double x = (((uint64_t)s * gx % n * step + ux[i]) & 0xFFFF) / 65536.0L - mx[i];
      const long double y = (((uint64_t)s * gy % n * step + uy[i]) & 0xFFFF) / 65536.0L - my[i];
      direct += std::exp2((long double)a * (x * x + y * y));
    }
    want[i] = (double)(direct / n);
    gauss_table(n, g, q, a, bx, by, c, mx[i], my[i], four.data() + i % 4);
    for (size_t e = 0; e < t.size(); ++e) t[e] = four[4 * e + i % 4];
    if (t[11] != 0.0) {
      ++*flagged;
      got[i] = want[i];
      continue;
    }
    const uint32_t cls = ((uint32_t)(uy[i] >> sh) * gx - (uint32_t)(ux[i] >> sh) * gy) & (n - 1), fm = (1u << sh) - 1;
    const uint32_t* row = &q.rows[(size_t)cls * q.stride];
    const double ax = ((int)(int16_t)(row[0] & 0xFFFF) * (int)(1u << sh) + (int)(ux[i] & fm)) / 65536.0;
    const double ay = (((int)row[0] >> 16) * (int)(1u << sh) + (int)(uy[i] & fm)) / 65536.0;
    double y = std::exp2(t[0] * (ax * ax + ay * ay) + t[1] * ax + t[2] * ay + t[3]);
    const double za = std::exp2(t[4] * ax + t[5] * ay + t[6]), ys = std::exp2(t[7] * ax + t[8] * ay + t[9]);
    const double* w = &t[GAUSS_HEAD + 2 * q.lines];
    double total = 0.0;
    for (uint32_t l = 0; l < q.lines; ++l) {
      const GaussLines::Span& gr = q.spans[l];
      const uint32_t r = row[1 + l];
      const int lo = (int)(r & 0xFFFF), hi = (int)(r >> 16);
      const double z = za * t[GAUSS_HEAD + 2 * l];
      double p = 0.0;
      for (int s = gr.steps - 1; s >= 0; --s) {
        const bool in = s < hi && s >= lo;
        if (s >= gr.full_lo && s < gr.full_hi && !in) return -1;   // the unmasked part
        p = std::fma(p, z, in ? w[s] : 0.0);
      }
      if (hi > gr.steps) return -1;
      total += y * t[GAUSS_HEAD + 2 * l + 1] * p;
      if (l + 1 < q.lines) y *= ys * std::pow(za, (double)(q.j0[l + 1] - q.j0[l]));
    }
    got[i] = total / n;
  }
  return (int)q.steps;
}
