// Host-only exercise of the estimate by which a launch goes to the ring kernel or the runs kernel (csrc/tq_choice.h).
#include <cmath>
#include <cstdio>
#include <vector>
#include "../paper_2509_22951_amd/csrc/tq_choice.h"

using tq::BatchedMatrix;
static uint64_t state = 88172645463325252ull;
static uint32_t rnd(uint32_t n) {
  state ^= state << 13, state ^= state >> 7, state ^= state << 17;
  return (uint32_t)(state % n);
}
static BatchedMatrix matrix(uint32_t rows, uint32_t cols, uint32_t seg, uint64_t bytes) { return {(rows + 15) / 16, cols, (cols + 4 * seg - 1) / (4 * seg), seg, bytes}; }

// The longest share against all workgroups of the cut, one by one: no shorter, and longer by one band of a matrix at most.
static bool shares() {
  for (int trial = 0; trial < 20000; ++trial) {
    const int n = 1 + rnd(trial % 3 ? 6 : 60);
    std::vector<BatchedMatrix> m;
    uint64_t total = 0, bands = 0, widest = 1;
    for (int i = 0; i < n; ++i) {
      m.push_back(matrix(1 + rnd(rnd(2) ? 100 : 20000), 1 + rnd(rnd(2) ? 64 : 9000), 256, 0));
      total += (uint64_t)m[i].n_bands * m[i].cols;
      bands += m[i].n_bands;
      widest = std::max<uint64_t>(widest, m[i].cols);
    }
    const uint64_t grid = std::max<uint64_t>(1, std::min<uint64_t>({256, bands, total / widest}));
    auto job = [&](int i, double b) { return 1000. + b * m[i].cols; };
    const double got = tq::longest_share(n, m.data(), grid, job);
    double want = 0;
    for (uint64_t w = 0; w < grid; ++w) {
      const uint64_t lo = total * w / grid, hi = total * (w + 1) / grid;
      uint64_t cb = 0;
      double sum = 0;
      for (int i = 0; i < n; ++i) {
        const uint64_t bc = m[i].cols, ce = cb + m[i].n_bands * bc;
        if (cb < hi && ce > lo) {
          const uint64_t b0 = lo <= cb ? 0 : (lo - cb + bc / 2) / bc, b1 = hi >= ce ? m[i].n_bands : std::min<uint64_t>(m[i].n_bands, (hi - cb + bc / 2) / bc);
          if (b0 < b1) sum += job(i, (double)(b1 - b0));
        }
        cb = ce;
      }
      want = std::max(want, sum);
    }
    if (got < want || got > want + widest) return std::printf("trial %d: share %.0f, longest %.0f\n", trial, got, want), false;
  }
  return true;
}

// Times are finite and positive, and no shorter for more rows of x or four times the rows of the matrices.
static bool grows() {
  for (int trial = 0; trial < 4000; ++trial) {
    const bool packed = rnd(2), gate = rnd(2);
    const uint32_t seg = 32u << rnd(packed ? 3 : 4), n = 1 + rnd(40);
    std::vector<BatchedMatrix> m;
    for (uint32_t i = 0; i < n; ++i) m.push_back(matrix(1 + rnd(20000), 4 * seg * (1 + rnd(12)), seg, rnd(50) * 1000000ull));
    double before[2] = {0, 0};
    for (int batch = 3; batch <= 16; ++batch) {
      const double t[2] = {tq::ring_time((int)n, m.data(), 256, batch, packed, gate), tq::runs_time((int)n, m.data(), 256, batch, packed)};
      for (int k = 0; k < 2; ++k) {
        if (!std::isfinite(t[k]) || t[k] <= 0 || t[k] < before[k]) return std::printf("trial %d, batch %d: %f after %f\n", trial, batch, t[k], before[k]), false;
        before[k] = t[k];
      }
    }
    for (BatchedMatrix& k : m) k.n_bands = 4 * k.n_bands + 256;
    if (tq::ring_time((int)n, m.data(), 256, 16, packed, gate) < before[0] || tq::runs_time((int)n, m.data(), 256, 16, packed) < before[1])
      return std::printf("trial %d: shorter with four times the rows\n", trial), false;
  }
  return true;
}

// Launches of equal matrices that were timed on both kernels, us; every one has to go where it was faster.
struct Timed {
  bool packed, gate;
  uint32_t seg, rows, cols, n, mbytes;   // cols: of the weights
  int batch;
  double ring, runs;
};
static const Timed timed[] = {
    {false, false, 32, 13414, 18560, 3, 936, 16, 2118, 404}, {false, false, 64, 742, 4864, 60, 255, 9, 219, 93},
    {false, false, 128, 6026, 2560, 5, 87, 16, 78.1, 49.6},  {false, false, 256, 5046, 5120, 9, 250, 9, 123.5, 83.8},
    {false, false, 256, 7918, 1024, 8, 73, 4, 23.4, 32.0},   {false, false, 256, 2398, 14336, 16, 584, 16, 264, 371},
    {false, false, 256, 16004, 1024, 1, 18, 16, 13.1, 16.8}, {false, false, 256, 9420, 3072, 6, 188, 9, 80.4, 60.9},
    {false, true, 32, 5190, 896, 6, 36, 4, 38.9, 19.1},      {false, true, 64, 1626, 11264, 25, 254, 16, 389, 226},
    {false, true, 256, 22528, 4096, 2, 198, 16, 59.4, 79.5}, {false, true, 256, 22604, 1024, 1, 26, 8, 14.7, 18.6},
    {true, false, 32, 1452, 6656, 29, 170, 16, 436, 163},    {true, false, 128, 2502, 16384, 21, 445, 9, 336, 241},
    {true, false, 128, 12100, 1024, 4, 27, 8, 14.6, 22.1},   {true, false, 128, 3804, 3072, 13, 82, 9, 66.4, 50.7},
    {true, false, 128, 1274, 1024, 60, 47, 4, 26.1, 36.5},   {true, true, 32, 524, 12800, 60, 240, 16, 293, 221},
    {true, true, 64, 1298, 2560, 23, 46, 4, 43.7, 26.5},     {true, true, 128, 8192, 1024, 2, 9, 16, 10.5, 16.0},
    {true, true, 128, 12086, 18432, 4, 451, 16, 196, 365},   {true, true, 128, 19200, 10240, 4, 399, 8, 150, 198},
};
static bool choices() {
  bool ok = true;
  // what a matrix of narrow bands costs beside wide ones (packed, batch 5, gated pairs; 31.9 us on the runs kernel alone)
  const uint32_t shape[][2] = {{3830, 3302}, {64, 32}, {422, 6}, {256, 1920}, {15360, 512}, {1044, 28}, {2, 1024}};
  std::vector<BatchedMatrix> mixed;
  for (const auto& s : shape) mixed.push_back(matrix(s[0], s[1], 128, 0));
  const double us = tq::runs_time(7, mixed.data(), 256, 5, true);
  if (us < 24 || us > 40) std::printf("seven matrices: %.1f us by the estimate\n", us), ok = false;
  for (const Timed& t : timed) {
    std::vector<BatchedMatrix> m(t.n, matrix(t.rows, t.cols / (t.packed ? 2 : 1), t.seg, t.mbytes * 1000000ull / t.n));
    const double ring = tq::ring_time((int)t.n, m.data(), 256, t.batch, t.packed, t.gate), runs = tq::runs_time((int)t.n, m.data(), 256, t.batch, t.packed);
    if ((ring <= runs) != (t.ring <= t.runs)) {
      std::printf("%u times %u x %u, segments of %u, batch %d: %.1f / %.1f by the estimate, %.1f / %.1f timed\n", t.n, t.rows, t.cols, t.seg, t.batch, ring, runs, t.ring, t.runs);
      ok = false;
    }
  }
  return ok;
}

int main() {
  if (!shares() || !grows() || !choices()) return 1;
  std::printf("ok\n");
  return 0;
}
