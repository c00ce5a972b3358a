// The rank-1 lattice of Sec. 3.2 as parallel lines: host tables of the line
// counter (count.hip).  Host code without HIP types.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cstdlib>
#include <utility>
#include <vector>

namespace bnlat {

// One Heaviside's terms of the line counter (count.hip).  With the lattice's
// line vectors b1 (along a line) and b2 (to the next one) in Q0.16 units,
// m = n . b1 and m2 = n . b2: the crossing of line l is
// -dot * inv + off + l * slope in units of b1, as int64 with 32 fraction bits.
struct LineRec {
  uint32_t n;        // nx | ny << 16
  int32_t d;         // D' = n . (C - 2^15)
  double inv;        // -1 / m; 0: counted sample by sample (|m| < LINE_MIN_M)
  long long off;     // ((D' + 1/2) / m + 1) 2^32, rounded
  long long slope;   // -(m2 / m) 2^32, rounded
};
constexpr int LINE_MIN_M = 1 << 12;

// Template sizes of the line counter: the smallest that holds `lines` lines,
// or 0 when there is none; words of one shift class's row at a template size.
#define BN_LINE_TEMPLATES(X) X(2) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(44) X(64) X(90)
inline uint32_t line_template(uint32_t lines) {
#define BN_LINE_FITS(R) if (lines <= R) return R;
  BN_LINE_TEMPLATES(BN_LINE_FITS)
#undef BN_LINE_FITS
  return 0;
}
constexpr uint32_t line_row_words(uint32_t lines) { return (lines + 2 + 3) / 4 * 4; }

// The lattice (gx, gy) / N seen as parallel lines: b1 its vector of smallest
// |x| + |y| (in units of 1 / N; at most that many lines meet the unit
// square), b2 a shortest vector to the next line (det(b1, b2) = N).
struct LatticeLines {
  int64_t b1[2], b2[2];
  uint32_t lines;
};

inline LatticeLines lattice_lines(int64_t n, int64_t gx, int64_t gy) {
  std::vector<std::pair<int64_t, int64_t>> vec;   // lattice vectors in (-N, N)^2, and N along each axis
  for (int64_t k = 1; k < n; ++k) {
    const int64_t x = k * gx % n, y = k * gy % n;
    for (int64_t a : {x, x - n})
      for (int64_t b : {y, y - n}) vec.emplace_back(a, b);
  }
  for (int64_t s : {n, -n}) {
    vec.emplace_back(s, 0);
    vec.emplace_back((int64_t)0, s);
  }
  auto size = [](const std::pair<int64_t, int64_t>& v) { return std::llabs(v.first) + std::llabs(v.second); };
  const auto b1 = *std::min_element(vec.begin(), vec.end(), [&](const auto& a, const auto& b) { return size(a) < size(b); });
  LatticeLines out{{b1.first, b1.second}, {0, 0}, (uint32_t)size(b1)};
  int64_t best = -1;
  for (const auto& v : vec) {
    const int64_t det = b1.first * v.second - b1.second * v.first;
    if (det != n && det != -n) continue;
    const int64_t s = det > 0 ? 1 : -1, x = s * v.first, y = s * v.second, len = x * x + y * y;
    if (best >= 0 && len >= best) continue;
    best = len;
    out.b2[0] = x;
    out.b2[1] = y;
  }
  if (best < 0) out.lines = 0;
  return out;
}

inline int64_t floor_div(int64_t a, int64_t b) { return a / b - ((a % b != 0) && ((a < 0) != (b < 0))); }

// The lines of every shift class, rows of `stride` words: sample A of the
// first line (x | y << 16, lattice units), sum of lo over the lines, then
// lo | hi << 16 (int16) per line, j counted from A + l b2.  Class k holds the
// shifts (x, y) with y gx - x gy = k mod N.  False if a row does not fit.
inline bool lattice_rows(int64_t n, int64_t gx, int64_t gy, const LatticeLines& g, uint32_t max_lines, uint32_t stride,
                  std::vector<uint32_t>& rows) {
  rows.assign((size_t)n * stride, 0u);
  int64_t inv = 1;   // gx^-1 mod N (N a power of two: Newton)
  for (int i = 0; i < 6; ++i) inv = ((inv * (2 - gx * inv)) % n + n) % n;
  if (n == 1) inv = 0;
  const int64_t bx = g.b1[0], by = g.b1[1], top = n - 1;
  for (int64_t k = 0; k < n; ++k) {
    const int64_t py = k * inv % n;   // the class's sample with x = 0
    // line index of the square's corners relative to the sample's line
    int64_t l0 = 0, l1 = 0;
    for (int64_t cx : {(int64_t)0, top})
      for (int64_t cy : {(int64_t)0, top}) {
        const int64_t d = bx * (cy - py) - by * cx;
        l0 = std::min(l0, floor_div(d, n));
        l1 = std::max(l1, floor_div(d, n) + 1);
      }
    uint32_t* row = &rows[(size_t)k * stride];
    bool first = true;
    int64_t base = 0, j0 = 0, sum = 0, total = 0;
    for (int64_t l = l0; l <= l1; ++l) {
      const int64_t x = l * g.b2[0], y = py + l * g.b2[1];
      int64_t a = -4 * n, b = 4 * n;   // j range with the line's points in [0, N)^2
      for (int axis = 0; axis < 2; ++axis) {
        const int64_t c = axis ? y : x, s = axis ? by : bx;
        if (s > 0) {
          a = std::max(a, floor_div(-c + s - 1, s));
          b = std::min(b, floor_div(top - c, s));
        } else if (s < 0) {
          a = std::max(a, floor_div(c - top - s - 1, -s));
          b = std::min(b, floor_div(c, -s));
        } else if (c < 0 || c > top) {
          b = a - 1;
        }
      }
      if (b < a) continue;
      if (first) {
        first = false;
        base = l;
        j0 = a;
        row[0] = (uint32_t)(x + a * bx) | ((uint32_t)(y + a * by) << 16);
      }
      const int64_t lo = a - j0, hi = b + 1 - j0;
      if (l - base >= max_lines || lo < -32768 || hi > 32767) return false;
      row[2 + (l - base)] = ((uint32_t)lo & 0xFFFFu) | ((uint32_t)hi << 16);
      sum += lo;
      total += hi - lo;
    }
    if (total != n) return false;
    row[1] = (uint32_t)(int32_t)sum;
  }
  return true;
}

// a / b rounded to the nearest integer (b != 0).
inline __int128 round_div(__int128 a, __int128 b) {
  if (b < 0) a = -a, b = -b;
  const __int128 q = (2 * a + b) / (2 * b);
  return q - (((2 * a + b) % (2 * b)) < 0);
}

// The line counter's terms of one Heaviside; step = 65536 / N.
inline LineRec line_record(const LatticeLines& g, int64_t step, int64_t nx, int64_t ny, int64_t cx, int64_t cy) {
  LineRec r;
  r.n = ((uint32_t)(uint16_t)nx) | ((uint32_t)(uint16_t)ny << 16);
  r.d = (int32_t)(nx * (cx - 32768) + ny * (cy - 32768));
  r.inv = 0.0;
  r.off = r.slope = 0;
  const int64_t m = (nx * g.b1[0] + ny * g.b1[1]) * step, m2 = (nx * g.b2[0] + ny * g.b2[1]) * step;
  if (std::llabs(m) < LINE_MIN_M) return r;
  r.inv = -1.0 / (double)m;
  r.off = (long long)round_div((__int128)(2 * (int64_t)r.d + 1) << 31, m) + (1ll << 32);
  r.slope = (long long)round_div((__int128)(-m2) << 32, m);
  return r;
}

// How far a hit count can be from N times the integrand's area, for every
// shift (0: no useful bound).  A line's samples on one side of the edge are
// the integers in an interval, off its length by at most one; the lengths are
// a concave function of the line's place (chords of a convex polygon), so
// their sum over the lines is off its integral, N times the area, by at most
// the longest chord, N / max(|x|, |y|) for b1 = (x, y) / N; at most lines + 1
// lines meet the square.
inline uint32_t count_deviation(int64_t n, const LatticeLines& g) {
  const int64_t m = std::max(std::llabs(g.b1[0]), std::llabs(g.b1[1]));
  return g.lines && m ? (uint32_t)(g.lines + 1 + (n + m - 1) / m) : 0;
}

// A padded integrand: a crossing far before every line, counted on the m < 0
// side, so that it never counts a sample.
inline LineRec line_padding() { return LineRec{0u, 0, 1e-300, -(1ll << 52), 0}; }

}  // namespace bnlat
