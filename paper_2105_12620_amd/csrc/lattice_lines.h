// The rank-1 lattice of Sec. 3.2 as parallel lines: host tables of the line
// counter (count.hip).  Host code without HIP types.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

namespace bnlat {

// One Heaviside's terms of the line counter (count.hip).  With the lattice's
// line vectors b1 (along a line) and b2 (to the next one) in Q0.16 units,
// m = n . b1 and m2 = n . b2: the crossing of line l is
// -dot * inv + off + l * slope in units of b1, as int64 with 32 fraction bits.
// Edges nearly along the lines (|m| < LINE_MIN_M), whose crossings leave that
// format, have inv = 0 and, in off and slope, the doubles 1 / m (2^40 for m = 0)
// and m2: the crossing of line l is floor((D' + 1/2 - dot - l m2) / m) + 1, exactly
// (the numerator is a half integer under 2^34, so 1 / (2 |m|) away from the next
// crossing, and the quotient's rounding is below 2^-18).
struct LineRec {
  uint32_t n;        // nx | ny << 16
  int32_t d;         // D' = n . (C - 2^15)
  double inv;        // -1 / m, or 0
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
  // f(x, y) for the lattice vectors in (-N, N)^2, and N along each axis
  auto each = [&](auto f) {
    for (int64_t k = 1, x = gx % n, y = gy % n; k < n; ++k) {
      f(x, y), f(x, y - n), f(x - n, y), f(x - n, y - n);
      if ((x += gx) >= n) x %= n;
      if ((y += gy) >= n) y %= n;
    }
    for (int64_t s : {n, -n}) f(s, (int64_t)0), f((int64_t)0, s);
  };
  LatticeLines out{{0, 0}, {0, 0}, 0};
  int64_t best = -1;
  each([&](int64_t x, int64_t y) {
    const int64_t size = std::llabs(x) + std::llabs(y);
    if (best >= 0 && size >= best) return;
    best = size;
    out.b1[0] = x;
    out.b1[1] = y;
  });
  out.lines = (uint32_t)best;
  best = -1;
  each([&](int64_t x, int64_t y) {
    const int64_t det = out.b1[0] * y - out.b1[1] * x;
    if (det != n && det != -n) return;
    const int64_t s = det > 0 ? 1 : -1, len = x * x + y * y;
    if (best >= 0 && len >= best) return;
    best = len;
    out.b2[0] = s * x;
    out.b2[1] = s * y;
  });
  if (best < 0) out.lines = 0;
  return out;
}

inline int64_t floor_div(int64_t a, int64_t b) { return a / b - ((a % b != 0) && ((a < 0) != (b < 0))); }

// floor(c / s) for |c| < 2^22 (s > 0), by the reciprocal: (c + 1/2) / s is 1 / (2 s)
// away from the next integer.
struct FloorDiv {
  double inv;
  int64_t up, whole;   // whole multiples of s that make the quotient positive
  explicit FloorDiv(int64_t s) : inv(1.0 / (double)s), up(((int64_t)1 << 22) / s + 1), whole(up * s) {}
  int64_t operator()(int64_t c) const { return (int64_t)(((double)(c + whole) + 0.5) * inv) - up; }
};

// Steps j in [lo, hi) with the points (x, y) + j (bx, by) inside [0, N)^2.
struct LineInterval {
  int64_t n, step[2];
  FloorDiv div[2];
  LineInterval(int64_t n_, int64_t bx, int64_t by)
      : n(n_), step{bx, by}, div{FloorDiv(std::max<int64_t>(1, std::llabs(bx))), FloorDiv(std::max<int64_t>(1, std::llabs(by)))} {}
  void operator()(int64_t x, int64_t y, int64_t& lo, int64_t& hi) const {
    const int64_t top = n - 1;
    int64_t a = -4 * n, b = 4 * n;
    for (int axis = 0; axis < 2; ++axis) {
      const int64_t c = axis ? y : x, s = step[axis];
      if (s > 0) {
        a = std::max(a, div[axis](-c + s - 1));
        b = std::min(b, div[axis](top - c));
      } else if (s < 0) {
        a = std::max(a, div[axis](c - top - s - 1));
        b = std::min(b, div[axis](c));
      } else if (c < 0 || c > top) {
        b = a - 1;
      }
    }
    lo = a;
    hi = std::max(a, b + 1);
  }
};

// gx^-1 mod N (N a power of two, gx odd: Newton).
inline int64_t generator_inverse(int64_t n, int64_t gx) {
  int64_t inv = 1;
  for (int i = 0; i < 6; ++i) inv = ((inv * (2 - gx * inv)) % n + n) % n;
  return n == 1 ? 0 : inv;
}

// The lines that meet the square in every shift class: class k holds the shifts
// (x, y) with y gx - x gy = k mod N.  Line l of class k is that of the points
// (0, py) + l b2 + j b1, (0, py) its sample with x = 0; the steps j in [lo, hi).
struct ClassLines {
  struct Span {
    int32_t l, lo, hi;
  };
  std::vector<uint32_t> start;   // [N + 1] spans of each class, by l; none is empty
  std::vector<Span> spans;
  std::vector<int32_t> py;       // [N]
};

inline ClassLines class_lines(int64_t n, int64_t gx, int64_t gy, const LatticeLines& g) {
  ClassLines out;
  const int64_t inv = generator_inverse(n, gx), bx = g.b1[0], by = g.b1[1], top = n - 1;
  const LineInterval interval(n, bx, by);
  out.spans.reserve((size_t)n * (g.lines + 1));
  for (int64_t k = 0; k < n; ++k) {
    const int64_t py = k * inv % n;
    out.py.push_back((int32_t)py);
    out.start.push_back((uint32_t)out.spans.size());
    // line index of the square's corners relative to the sample's line
    int64_t l0 = 0, l1 = 0;
    for (int64_t cx : {(int64_t)0, top})
      for (int64_t cy : {(int64_t)0, top}) {
        const int64_t d = floor_div(bx * (cy - py) - by * cx, n);
        l0 = std::min(l0, d);
        l1 = std::max(l1, d + 1);
      }
    for (int64_t l = l0; l <= l1; ++l) {
      int64_t a, b;
      interval(l * g.b2[0], py + l * g.b2[1], a, b);
      if (b > a) out.spans.push_back({(int32_t)l, (int32_t)a, (int32_t)b});
    }
  }
  out.start.push_back((uint32_t)out.spans.size());
  return out;
}

// The lines of every shift class, rows of `stride` words: sample A of the
// first line (x | y << 16, lattice units), sum of lo over the lines, then
// lo | hi << 16 (int16) per line, j counted from A + l b2.  False if a row does
// not fit.
inline bool lattice_rows(int64_t n, const ClassLines& c, const LatticeLines& g, uint32_t max_lines, uint32_t stride,
                         std::vector<uint32_t>& rows) {
  rows.assign((size_t)n * stride, 0u);
  for (int64_t k = 0; k < n; ++k) {
    uint32_t* row = &rows[(size_t)k * stride];
    if (c.start[k] == c.start[k + 1]) return false;
    const ClassLines::Span first = c.spans[c.start[k]];
    const int64_t x = first.l * g.b2[0] + first.lo * g.b1[0], y = c.py[k] + first.l * g.b2[1] + first.lo * g.b1[1];
    row[0] = (uint32_t)x | ((uint32_t)y << 16);
    int64_t sum = 0, total = 0;
    for (uint32_t i = c.start[k]; i < c.start[k + 1]; ++i) {
      const ClassLines::Span q = c.spans[i];
      const int64_t lo = q.lo - first.lo, hi = q.hi - first.lo;
      if (q.l - first.l >= (int64_t)max_lines || lo < -32768 || hi > 32767) return false;
      row[2 + (q.l - first.l)] = ((uint32_t)lo & 0xFFFFu) | ((uint32_t)hi << 16);
      sum += lo;
      total += hi - lo;
    }
    if (total != n) return false;
    row[1] = (uint32_t)(int32_t)sum;
  }
  return true;
}

inline bool lattice_rows(int64_t n, int64_t gx, int64_t gy, const LatticeLines& g, uint32_t max_lines, uint32_t stride,
                         std::vector<uint32_t>& rows) {
  return lattice_rows(n, class_lines(n, gx, gy, g), g, max_lines, stride, rows);
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
  if (std::llabs(m) < LINE_MIN_M) {
    const double flat[2] = {m ? 1.0 / (double)m : 0x1p40, (double)m2};
    std::memcpy(&r.off, &flat[0], 8);
    std::memcpy(&r.slope, &flat[1], 8);
    return r;
  }
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

// The same lines for the Gaussian estimates (gauss_lines.hip): class rows
// anchored at the lattice point A nearest the square's centre, line l at
// A + l b2 for l = first .. first + lines - 1, steps counted from the line's
// origin O_l = A + l b2 + j0_l b1, j0_l the smallest step any class has on it.
struct GaussLines {
  uint32_t lines = 0, stride = 0, steps = 0;   // steps: longest line
  int64_t first = 0;
  std::vector<int64_t> j0;                     // [lines]
  // per line: steps to take, and the part [full_lo, full_hi) of them that
  // every class has (without one: [steps, steps), so that a step above full_hi
  // is above every class's first)
  struct Span {
    int32_t steps, full_lo, full_hi;
  };
  std::vector<Span> spans;
  // [N][stride]: A (int16 x | y << 16), then lo | hi << 16 per line
  std::vector<uint32_t> rows;
};

inline GaussLines gauss_lines(int64_t n, const ClassLines& c, const LatticeLines& g) {
  GaussLines out;
  const int64_t bx = g.b1[0], by = g.b1[1], cx = g.b2[0], cy = g.b2[1];
  // nearest integer to a / (2 n)
  auto near = [&](int64_t a) { return floor_div(a + n, 2 * n); };
  // A = (0, py) - al b1 - be b2: step j of line l is step j + al of line l + be from A
  std::vector<int32_t> al(n), be(n);
  int64_t l0 = INT32_MAX, l1 = INT32_MIN;
  for (int64_t k = 0; k < n; ++k) {
    // twice the sample (0, py) less the centre, in units of b1 and b2
    const int64_t x = -(n - 1), y = 2 * (int64_t)c.py[k] - (n - 1);
    al[k] = (int32_t)near(x * cy - y * cx);
    be[k] = (int32_t)near(bx * y - by * x);
    l0 = std::min<int64_t>(l0, c.spans[c.start[k]].l + be[k]);
    l1 = std::max<int64_t>(l1, c.spans[c.start[k + 1] - 1].l + be[k]);
  }
  out.first = l0;
  out.lines = (uint32_t)(l1 - l0 + 1);
  out.stride = 1 + out.lines;
  struct Range {
    int64_t jmin = INT32_MAX, jmax = INT32_MIN, lo_max = INT32_MIN, hi_min = INT32_MAX, classes = 0;
  };
  std::vector<Range> range(out.lines);
  for (int64_t k = 0; k < n; ++k)
    for (uint32_t i = c.start[k]; i < c.start[k + 1]; ++i) {
      Range& r = range[c.spans[i].l + be[k] - l0];
      const int64_t lo = c.spans[i].lo + al[k], hi = c.spans[i].hi + al[k];
      r.jmin = std::min(r.jmin, lo);
      r.lo_max = std::max(r.lo_max, lo);
      r.jmax = std::max(r.jmax, hi);
      r.hi_min = std::min(r.hi_min, hi);
      ++r.classes;
    }
  out.j0.assign(out.lines, 0);
  out.spans.assign(out.lines, GaussLines::Span{0, 0, 0});
  for (uint32_t i = 0; i < out.lines; ++i) {
    Range r = range[i];
    if (!r.classes) r.jmin = r.jmax = i ? out.j0[i - 1] : 0;
    if (r.classes < n || r.hi_min < r.lo_max) r.lo_max = r.hi_min = r.jmax;
    out.j0[i] = r.jmin;
    out.spans[i] = GaussLines::Span{(int32_t)(r.jmax - r.jmin), (int32_t)(r.lo_max - r.jmin), (int32_t)(r.hi_min - r.jmin)};
    out.steps = std::max(out.steps, (uint32_t)(r.jmax - r.jmin));
  }
  out.rows.assign((size_t)n * out.stride, 0u);
  for (int64_t k = 0; k < n; ++k) {
    uint32_t* row = &out.rows[(size_t)k * out.stride];
    const int64_t ax = -al[k] * bx - be[k] * cx, ay = c.py[k] - al[k] * by - be[k] * cy;
    row[0] = ((uint32_t)ax & 0xFFFFu) | ((uint32_t)ay << 16);
    for (uint32_t i = c.start[k]; i < c.start[k + 1]; ++i) {
      const int64_t l = c.spans[i].l + be[k] - l0, shift = al[k] - out.j0[l];
      row[1 + l] = (uint32_t)(c.spans[i].lo + shift) | ((uint32_t)(c.spans[i].hi + shift) << 16);
    }
  }
  return out;
}

inline GaussLines gauss_lines(int64_t n, int64_t gx, int64_t gy, const LatticeLines& g) {
  return gauss_lines(n, class_lines(n, gx, gy, g), g);
}

// One Gaussian's table for the line form, doubles, interleaved with those of
// the other three of its four (entry i at 4 i): with E(x) = a |x|^2 + bx x +
// by y + c its base-2 exponent and lengths in the unit square,
//   [0..3]   E at the first line's origin less a |O - A|^2, as a function of A:
//            a, then the coefficients of x, y and 1
//   [4..6]   exponent of the step b1 at A, less a |b1|^2: coefficients of x, y, 1
//   [7..9]   the same for b2
//   [11]     1 where the exponents leave FP64's range (counted sample by sample)
//   [12 ..]  per line: ratio of its step factor to that at A, 2^(a |O - A|^2)
//   then     2^(a |b1|^2 j^2) for j = 0 .. steps - 1
constexpr uint32_t GAUSS_HEAD = 12;
inline uint32_t gauss_table_words(const GaussLines& q) { return (GAUSS_HEAD + 2 * q.lines + q.steps + 3) / 4 * 4; }

inline void gauss_table(int64_t n, const LatticeLines& g, const GaussLines& q, double a, double bx, double by, double c,
                        double mx, double my, double* t) {
  const double u = 1.0 / (double)n;
  const double b1x = g.b1[0] * u, b1y = g.b1[1] * u, b2x = g.b2[0] * u, b2y = g.b2[1] * u;
  const double d0x = q.first * b2x + q.j0[0] * b1x, d0y = q.first * b2y + q.j0[0] * b1y;
  t[0] = a;
  t[4] = bx + 2.0 * a * d0x;
  t[8] = by + 2.0 * a * d0y;
  t[12] = c + bx * d0x + by * d0y;
  t[16] = 2.0 * a * b1x;
  t[20] = 2.0 * a * b1y;
  t[24] = bx * b1x + by * b1y;
  t[28] = 2.0 * a * b2x;
  t[32] = 2.0 * a * b2y;
  t[36] = bx * b2x + by * b2y;
  double far = 0.0;
  for (uint32_t i = 0; i < q.lines; ++i) {
    const double l = (double)(q.first + (int64_t)i), j = (double)q.j0[i];
    const double dx = l * b2x + j * b1x, dy = l * b2y + j * b1y;
    t[4 * (GAUSS_HEAD + 2 * i)] = std::exp2(2.0 * a * (dx * b1x + dy * b1y));
    t[4 * (GAUSS_HEAD + 2 * i + 1)] = std::exp2(a * (dx * dx + dy * dy));
    far = std::max(far, std::sqrt(dx * dx + dy * dy));
  }
  const double h = std::sqrt(b1x * b1x + b1y * b1y), k = std::sqrt(b2x * b2x + b2y * b2y);
  for (uint32_t j = 0; j < q.steps; ++j) t[4 * (GAUSS_HEAD + 2 * q.lines + j)] = std::exp2(a * h * h * (double)j * (double)j);
  // base-2 exponents met, over |a|: of a line's factor without and with its
  // |O - A|^2, and of Horner's partial sums, 2^-E at the points of a line from
  // its origin on (A is within half a cell of the centre)
  const double rc = std::sqrt((mx - 0.5) * (mx - 0.5) + (my - 0.5) * (my - 0.5)), half = 0.5 * (h + k), ra = rc + half;
  const double e1 = ra * ra + 2.0 * ra * far, e3 = rc + std::max(far + half, 0.7072);
  const double most = std::max(std::max(e1, far * far), e3 * e3);
  t[40] = 0.0;
  t[44] = -a * most < 1000.0 ? 0.0 : 1.0;
}

// A padded integrand: a crossing far before every line, counted on the m < 0
// side, so that it never counts a sample.
inline LineRec line_padding() { return LineRec{0u, 0, 1e-300, -(1ll << 52), 0}; }

}  // namespace bnlat
