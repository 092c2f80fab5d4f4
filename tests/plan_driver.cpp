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

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "listing")) listing();
  else return 2;
  return 0;
}
