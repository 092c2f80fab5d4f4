// Which of the two batched kernels a launch takes: an estimate of both kernels' times.  Host code, no GPU needed.
#pragma once
#include <algorithm>
#include <cstdint>

#include "tq_format.h"
#include "tq_plan.h"

namespace tq {

struct BatchedMatrix {
  uint32_t n_bands, cols;      // as in BandCount (cols: stored bytes)
  uint32_t n_quads, seg_cols;
  uint64_t code_bytes;
};

// The largest sum over the matrices of a workgroup's share, job(i, bands of matrix i), when the cost line is cut into `grid` equal
// parts (see share_of_bands): the parts that hold an end of a matrix as they are, those inside one by the most bands one can get.
template <typename Job>
double longest_share(int n, const BatchedMatrix* m, uint64_t grid, Job&& job) {
  uint64_t total = 0;
  for (int i = 0; i < n; ++i) total += (uint64_t)m[i].n_bands * m[i].cols;
  double longest = 0;
  uint64_t start = 0, walked = UINT64_MAX, cb0 = 0;   // cb0: where matrix i0, the first of a part's, starts
  int i0 = 0;
  auto walk = [&](uint64_t part) {
    if (part == walked) return;
    walked = part;
    const uint64_t lo = total * part / grid, hi = total * (part + 1) / grid;
    while (cb0 + (uint64_t)m[i0].n_bands * m[i0].cols <= lo) cb0 += (uint64_t)m[i0].n_bands * m[i0].cols, ++i0;
    double sum = 0;
    uint64_t cb = cb0;
    for (int i = i0; i < n && cb < hi; ++i) {
      const uint64_t bc = m[i].cols, ce = cb + m[i].n_bands * bc;
      const uint64_t b0 = lo <= cb ? 0 : (lo - cb + bc / 2) / bc, b1 = hi >= ce ? m[i].n_bands : std::min<uint64_t>(m[i].n_bands, (hi - cb + bc / 2) / bc);
      if (b0 < b1) sum += job(i, (double)(b1 - b0));
      cb = ce;
    }
    longest = std::max(longest, sum);
  };
  for (int i = 0; i < n; ++i) {
    const uint64_t end = start + (uint64_t)m[i].n_bands * m[i].cols;
    const uint64_t first = start * grid / total, last = (end * grid - 1) / total;
    walk(first);
    if (last > first + 1) longest = std::max(longest, job(i, (double)std::min<uint64_t>(m[i].n_bands, ((total + grid - 1) / grid + m[i].cols - 1) / m[i].cols)));
    walk(last);
    start = end;
  }
  return longest;
}

// What the estimate is made of, us.  The unit of account is 16 x 1024 weights (4 segments of 256 columns); narrower units count by
// their width.
struct RingTimes {     // k_matvec_ring: a workgroup walks the quads of its bands, a barrier and an activation tile each
  double start;        // of the launch
  double quad;         // a quad, whatever its width
  double lone, band;   // a quad of b bands: lone + band * b, or full * b where there are enough of them for all wavefronts
  double full;
  double matrix;       // a workgroup's start of another matrix
  double rows;         // more for a tile of 16 rows of x than for one of 8, of the decode's time
  double add;          // a band's sums added to y, per row of x (gated pairs keep theirs in registers)
};
struct RunsTimes {     // k_matvec_runs: the units of a share, side by side
  double start, matrix;
  double piece;                       // a unit, whatever its width
  double rows4, rows8, rows9, row;    // a unit: up to 4 rows of x, up to 8, 9, and each row more
  double hbm;                         // more, of that, where the codes come from HBM
};
constexpr double kAddsPerUs = .105e6;   // floating-point additions to y that the chip takes

// Fitted to the times of 1,060 launches (half of the units 16 x 1024 weights, the others narrower; 1 to 60 matrices of up to three
// shapes, 256 to 28,000 rows, 256 to 18,000 columns, 3 to 100 bands per compute unit; 8-bit and packed weights, products and gated
// pairs) at 3, 4, 5, 6, 8, 9, 10, 12, 14 and 16 rows of x: half of the times are met within 4 % (ring) and 5 % (runs), nine tenths within
// 14 %.  Which is the faster kernel by it costs 0.5 % over the better of both on average, and more than 5 % in one launch of 26; by
// bands per compute unit (24, above 8 rows of x 12) it was 9 % and more than 5 % in one of 4, worst where narrow segments have
// many sums to add (4 times the time), or few bands of many quads leave the ring kernel's wavefronts idle.
// (The kernels have since become faster, the runs kernel by 4 % in the middle and up to 10 in small shares.  4,932 launches of whole units, 1 to 30 matrices: the
// choice costs 1.2 % over the better kernel, more than 5 % in one of 11; with the kernels that the times were fitted to 1.1 %, one of 13.)
inline double ring_time(int n, const BatchedMatrix* m, uint64_t n_cu, int batch, bool packed, bool gate_up) {
  static const RingTimes table[2][2] = {{{2.7, 1.1, 5.1, .56, .79, 1.0, 0., .039}, {1.9, 1.4, 4.6, .67, 1.06, 2.2, .04, 0.}},
                                        {{3.5, 1.25, 3.3, .37, .48, .5, .06, .04}, {1.8, 1.35, 2.6, .6, .76, 1.9, .06, 0.}}};
  const RingTimes& t = table[packed][gate_up];
  uint64_t total = 0, bands = 0, band_cost_max = 1;
  double adds = 0;
  for (int i = 0; i < n; ++i) {
    total += (uint64_t)m[i].n_bands * m[i].cols;
    bands += m[i].n_bands;
    band_cost_max = std::max<uint64_t>(band_cost_max, m[i].cols);
    adds += (double)m[i].n_bands * kUnitRows * (m[i].n_quads - 1) * batch;
  }
  const uint64_t grid = std::max<uint64_t>(1, std::min<uint64_t>({n_cu, bands, total / band_cost_max}));
  const double decode = batch > 8 ? 1 + t.rows : 1;
  double us = longest_share(n, m, grid, [&](int i, double b) {
    const double unit = (packed ? 2. : 1.) * m[i].seg_cols / 256, passes = gate_up ? std::max(1., (double)(((uint64_t)b + 35) / 36)) : 1.;
    const double pass = t.quad + decode * unit * std::max(t.lone + t.band * b / passes, t.full * b / passes);
    return t.matrix + m[i].n_quads * (passes * pass + t.add * batch * b);
  });
  if (!gate_up) us = std::max(us, adds / kAddsPerUs);
  return t.start + us;
}

inline double runs_time(int n, const BatchedMatrix* m, uint64_t n_cu, int batch, bool packed) {
  static const RunsTimes table[2] = {{2.8, 8.0, .07, .83, .87, 1.11, .086, .29}, {2.1, 6.6, .1, .8, .855, .96, .059, .05}};
  const RunsTimes& t = table[packed];
  uint64_t total = 0, bands = 0, band_cost_max = 1, bytes = 0;
  for (int i = 0; i < n; ++i) {
    total += (uint64_t)m[i].n_bands * m[i].cols;
    bands += m[i].n_bands;
    band_cost_max = std::max<uint64_t>(band_cost_max, m[i].cols);
    bytes += m[i].code_bytes;
  }
  const uint64_t grid = std::max<uint64_t>(1, std::min<uint64_t>({n_cu, bands, total / band_cost_max}));
  // (the cache behind the L2 holds 256 MB: codes of 144 MB come from it on every pass, of 336 MB from HBM)
  const double cold = std::min(1., std::max(0., ((double)bytes - 144e6) / 192e6));
  const double rows = batch <= 4 ? t.rows4 : batch <= 8 ? t.rows8 : t.rows9 + t.row * (batch - 9);
  auto job = [&](int i, double b) {
    const double units = (packed ? 2. : 1.) * unit_columns(m[i].cols, m[i].seg_cols) / 1024;   // of a band
    return t.matrix + b * (t.piece * m[i].n_quads + rows * (1 + t.hbm * cold) * units);
  };
  uint32_t wgs[kMaxAssign];
  BandCount count[kMaxAssign];
  for (int i = 0; i < n && i < kMaxAssign; ++i) count[i] = {m[i].n_bands, unit_columns(m[i].cols, m[i].seg_cols)};   // (as the launch counts them)
  if (n > kMaxAssign || !cut_in_workgroups(n, count, std::min(n_cu, bands), grid, wgs)) return t.start + longest_share(n, m, grid, job);
  double us = 0;
  for (int i = 0; i < n; ++i) us = std::max(us, job(i, (m[i].n_bands + wgs[i] - 1) / wgs[i]));
  return t.start + us;
}

}  // namespace tq
