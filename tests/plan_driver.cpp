// Host-only exercise of the index arithmetic in csrc/tq_plan.h over its range.  Prints what was checked; the first
// violation ends the program with status 1.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "../paper_2509_22951_amd/csrc/tq_plan.h"

#define CHECK(c, ...)                                          \
  do {                                                         \
    if (!(c)) {                                                \
      std::printf("line %d: %s: ", __LINE__, #c);              \
      std::printf(__VA_ARGS__);                                \
      std::printf("\n");                                       \
      std::exit(1);                                            \
    }                                                          \
  } while (0)

// Streams of `escapes` escaped groups, then codewords, then a group of `raw` raw values (0: none), whose length lies
// around a multiple of the block: the outputs of the blocks must be the bytes [0, n_values), once each and in order.
static void listing() {
  const uint64_t block = 2048;
  int n = 0;
  for (uint64_t blocks = 1; blocks <= 3; ++blocks)
    for (int d = -8; d <= 8; ++d)
      for (uint64_t escapes = 0; escapes < 8; ++escapes)
        for (uint64_t raw = 0; raw <= 4; ++raw) {
          const uint64_t n_words = blocks * block + d, tail = raw ? 1 + raw : 0, codewords = n_words - 5 * escapes - tail;
          std::vector<uint64_t> start;   // first word of every token
          for (uint64_t e = 0; e < escapes; ++e) start.push_back(5 * e);
          for (uint64_t c = 0; c < codewords; ++c) start.push_back(5 * escapes + c);
          if (raw) start.push_back(n_words - tail);
          const uint64_t n_values = 4 * (start.size() - (raw ? 1 : 0)) + raw;
          uint64_t at = 0, written = 0;   // tokens before the block, bytes before its output
          for (uint64_t b = 0; b * block < n_words; ++b) {
            uint64_t tokens = 0;
            while (at + tokens < start.size() && start[at + tokens] < (b + 1) * block) ++tokens;
            const tq::ListingOutput o = tq::listing_output((uint32_t)at, (uint32_t)tokens, n_values);
            CHECK(o.lo <= o.hi && o.lo < 16 && o.lo == 4 * (at % 4) && o.hi <= 4 * (block + 3), "%lu words, %lu escapes, %lu raw, block %lu: lo %u hi %u",
                  n_words, escapes, raw, b, o.lo, o.hi);
            if (o.hi > o.lo) {
              CHECK(o.piece0 % 16 == 0 && o.piece0 + o.lo == written && o.piece0 + o.hi <= n_values, "%lu words, block %lu", n_words, b);
              written += o.hi - o.lo;
            }
            at += tokens;
          }
          CHECK(written == n_values, "%lu words, %lu escapes, %lu raw: %lu of %lu values", n_words, escapes, raw, written, n_values);
          ++n;
        }
  const uint32_t last = 0xFFFFFFFEu;   // the most tokens a stream may have
  const tq::ListingOutput o = tq::listing_output(last, 1, 4ull * last + 3);
  CHECK(o.piece0 + o.lo == 4ull * last && o.hi - o.lo == 3, "%u", o.hi);
  std::printf("%d listing streams\n", n);
}

// One to three matrices of any number of bands and narrow and ordinary widths on grids of several sizes: the search ends, every
// matrix gets workgroups, no more than there are, and the largest share is near the least possible one.
static void assign() {
  int n = 0;
  auto one = [&](const std::vector<tq::BandCount>& m, uint64_t grid) {
    uint32_t wgs[4] = {};
    const uint64_t worst = tq::assign_workgroups((int)m.size(), m.data(), grid, wgs);
    uint64_t sum = 0, share = 0, total = 0, cols_max = 0;
    for (size_t i = 0; i < m.size(); ++i) {
      CHECK(wgs[i] >= 1 && wgs[i] <= m[i].n_bands, "matrix %zu: %u workgroups", i, wgs[i]);
      sum += wgs[i];
      share = std::max<uint64_t>(share, (uint64_t)((m[i].n_bands + wgs[i] - 1) / wgs[i]) * m[i].cols);
      total += (uint64_t)m[i].n_bands * m[i].cols;
      cols_max = std::max<uint64_t>(cols_max, m[i].cols);
    }
    CHECK(sum <= grid && worst == share, "%zu matrices, first %u x %u, grid %lu: %lu workgroups, share %lu", m.size(), m[0].n_bands, m[0].cols, grid, sum, worst);
    // a share of twice the mean part and a band always suffices (a matrix then needs less than half its mean's
    // workgroups, rounded up) while the matrices are few against the grid; the search ends an eighth of a row above the least
    CHECK(worst <= 2 * ((total + grid - 1) / grid) + 2 * cols_max, "share %lu of %lu on %lu", worst, total, grid);
    ++n;
  };
  for (uint64_t grid : {16, 255, 256, 304})
    for (uint32_t cols = 1; cols <= 20; ++cols)
      for (uint32_t bands = 1; bands < 3000; bands += bands < 600 ? 1 : 7) {
        one({{bands, cols}}, grid);
        if (bands % 5 == 0) one({{bands, cols}, {bands / 3 + 1, 1 + (cols * 3) % 7}, {3 * bands, 1 + cols % 7}}, grid);
      }
  for (uint32_t bands : {1u, 255u, 257u, 1000u, 8016u, (1u << 23) - 1})
    for (uint32_t cols : {1u, 7u, 8u, 9u, 63u, 3072u, 8191u, 1u << 20}) one({{bands, cols}}, 256);
  uint32_t wgs[4];
  const tq::BandCount tall = {1u << 23, 4}, three[3] = {{5, 4}, {5, 4}, {5, 4}};
  CHECK(tq::assign_workgroups(1, &tall, 256, wgs) == 0 && tq::assign_workgroups(3, three, 2, wgs) == 0, "refused cuts");
  std::printf("%d cuts\n", n);
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "listing")) listing();
  else if (!std::strcmp(what, "assign")) assign();
  else return 2;
  return 0;
}
