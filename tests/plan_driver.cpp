// Host-only exercise of the index arithmetic in csrc/tq_plan.h over its range.  Prints what was checked; the first
// violation ends the program with status 1.
#include <algorithm>
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
  // a matrix of few wide bands leaves workgroups over: they go to the narrow ones, whose shares come near the even one
  for (uint32_t cols : {1u, 61u, 256u, 1023u})
    for (uint32_t bands : {100u, 548u, 800u, 20000u}) {
      const tq::BandCount two[2] = {{16, 9344}, {bands, cols}};
      uint32_t w[2];
      tq::assign_workgroups(2, two, 256, w);
      const uint64_t even = (16ull * 9344 + (uint64_t)bands * cols + 255) / 256, share = (uint64_t)((bands + w[1] - 1) / w[1]) * cols;
      CHECK(w[0] <= 16 && w[0] + w[1] <= 256, "%u + %u workgroups", w[0], w[1]);
      CHECK(even > 9344 || share <= std::max<uint64_t>(cols, even + even / 8 + cols), "%u bands of %u: %u workgroups, share %lu, even %lu", bands, cols, w[1], share, even);
    }
  for (uint32_t seg : {16u, 128u, 256u, 1024u})   // by the widest segment of every unit
    for (uint32_t cols = 1; cols < 9 * seg; ++cols) {
      uint32_t want = 0;
      for (uint32_t q = 0; q < cols; q += 4 * seg) want += 4 * std::min(seg, cols - q);
      CHECK(tq::unit_columns(cols, seg) == want && want >= cols, "%u columns in segments of %u: %u", cols, seg, tq::unit_columns(cols, seg));
    }
  uint32_t wgs[4];
  const tq::BandCount tall = {1u << 23, 4}, three[3] = {{5, 4}, {5, 4}, {5, 4}};
  CHECK(tq::assign_workgroups(1, &tall, 256, wgs) == 0 && tq::assign_workgroups(3, three, 2, wgs) == 0, "refused cuts");
  std::printf("%d cuts\n", n);
}

// The cuts that the kernels multiply out: parts of a cost line as the division gives them, bands of a workgroup in order and even, pieces of a
// unit's chunks, and the word that holds a workgroup's place and its bands.
static void cuts() {
  uint64_t state = 88172645463325252ull;
  auto rnd = [&](uint32_t n) {
    state ^= state << 13, state ^= state >> 7, state ^= state << 17;
    return (uint32_t)(state % n);
  };
  for (uint32_t parts = 1; parts <= tq::kMaxParts; ++parts)
    for (uint32_t rest = 0; rest < parts; rest += parts < 300 ? 1 : 1 + rnd(7))
      for (uint32_t k = 0; k <= parts; ++k) {
        const uint64_t share = rnd(2) ? rnd(1000) : 0xFFFFFFFFull / parts - 1, total = share * parts + rest;
        const uint32_t got = tq::even_part((uint32_t)share, rest, 1.f / (float)parts, k);
        CHECK(got == total * k / parts, "part %u of %u, rest %u: %u", k, parts, rest, got);
      }
  for (int trial = 0; trial < 100000; ++trial) {
    const uint32_t w = 1 + rnd(256), n = w + rnd(trial % 2 ? 50 : 1u << 21), bands = n / w;
    uint32_t at = 0;
    for (uint32_t k = 0; k < w; ++k) {
      const uint32_t lo = tq::workgroup_band(bands, n - bands * w, k), hi = tq::workgroup_band(bands, n - bands * w, k + 1);
      CHECK(lo == at && hi - lo >= bands && hi - lo <= bands + 1, "%u bands, workgroup %u of %u: %u..%u", n, k, w, lo, hi);
      at = hi;
    }
    CHECK(at == n, "%u of %u bands", at, n);
    const uint32_t start = rnd(tq::kLineMask + 1), few = rnd(tq::kMaxWorkgroupBands), word = tq::line_word(start, few);
    CHECK((word & tq::kLineMask) == start && word >> tq::kLineBits == few, "%u, %u", start, few);
  }
  for (uint32_t parts = 1; parts <= 64; ++parts)
    for (uint32_t len = parts; len < 70000; len += len < 40000 ? 1 : 97) CHECK(tq::piece_length(len, parts) == len / parts, "%u chunks in %u pieces", len, parts);
  std::printf("cuts of lines, bands and units\n");
}

// k_matvec_runs' decode of one unit by its schedule, in both sizes of its rings, column numbers in place of bytes: a piece of a lane's ring holds the
// columns it was stored with, and every group a look multiplies has to hold the lane's own columns of the run in their places
// and zeros (number 0) elsewhere.
struct LaneStream {
  uint32_t panel_len;              // columns of its segment
  std::vector<uint32_t> advance;   // columns per chunk: 4..8 until it is complete (the last one whatever is left), then pads
};
struct Unit {
  std::vector<LaneStream> lanes;
  uint32_t n_chunks, n_win8;   // windows are taken up to n_win8, in whole groups
  bool ragged;
  uint32_t bytes;              // of a lane's ring
};

// Largest distance between two lanes that are both unfinished after the same number of chunks, as the validator takes it.
static uint32_t spread_of(const std::vector<LaneStream>& lanes, uint32_t n_chunks) {
  std::vector<uint32_t> lo(n_chunks, ~0u), hi(n_chunks, 0);
  for (const LaneStream& l : lanes)
    for (uint32_t k = 0, pos = 0; k < l.advance.size(); ++k) {
      pos += l.advance[k];
      if (pos < l.panel_len) {
        lo[k] = std::min(lo[k], pos);
        hi[k] = std::max(hi[k], pos);
      }
    }
  uint32_t wide = 0;
  for (uint32_t k = 0; k < n_chunks; ++k)
    if (hi[k] > lo[k]) wide = std::max(wide, hi[k] - lo[k]);
  return wide;
}

// Chunks [c0, c_end) of the unit.  taken[lane][column] counts how often a column was multiplied; returns the places that held
// something else than they should.  always_store: the leftover goes to the ring whether there is one or not.
static int decode(const Unit& u, uint32_t c0, uint32_t c_end, bool always_store, std::vector<std::vector<int>>& taken) {
  const uint32_t kG = tq::ring_group(u.bytes), kLook = tq::ring_step(u.bytes), kP = tq::ring_piece(u.bytes);
  struct Lane {
    uint32_t pos = 0, first = 0;                 // first: the column the run starts at
    uint32_t ring[tq::kRingBytes] = {}, carry[8] = {};   // (the first u.bytes of it)
  };
  std::vector<Lane> lanes(u.lanes.size());
  uint32_t done = 0;
  int wrong = 0;
  auto store = [&](Lane& l, uint32_t col, const uint32_t* v) { std::memcpy(l.ring + (col & (u.bytes - 8)), v, 32); };
  const uint32_t zeros[8] = {};
  auto append = [&](size_t i, uint32_t chunk) {
    Lane& l = lanes[i];
    const LaneStream& s = u.lanes[i];
    uint32_t both[16] = {};
    std::memcpy(both, l.carry, 32);
    const uint32_t n = chunk < s.advance.size() ? s.advance[chunk] : 0;   // (pads are zeros behind the end)
    for (uint32_t k = 0; k < n; ++k) both[(l.pos & 7) + k] = l.pos + k + 1;
    const uint32_t after = std::min(l.pos + (n ? n : 8), s.panel_len);
    store(l, l.pos, both);
    std::memcpy(l.carry, (after ^ l.pos) >= 8 ? both + 8 : both, 32);
    l.pos = after;
  };
  auto multiply_ready = [&](bool ready) {
    if (u.ragged)
      for (Lane& l : lanes)
        if (always_store || tq::ring_leftover(l.pos)) store(l, l.pos, l.carry);
    if (done + 8 * kG > u.n_win8) return;
    for (size_t i = 0; i < lanes.size() && !ready; ++i)
      if (lanes[i].pos < std::min(u.lanes[i].panel_len, done + 8 * kG)) return;
    for (size_t i = 0; i < lanes.size(); ++i)
      for (uint32_t col = done; col < std::min(done + 8 * kG, u.lanes[i].panel_len); ++col) {   // (activations are zero behind the panel)
        const uint32_t got = lanes[i].ring[col % u.bytes], want = col >= lanes[i].first && col < lanes[i].pos ? col + 1 : 0;
        wrong += got != want;
        taken[i][col] += want != 0;
      }
    done += 8 * kG;
  };
  if (c0) {   // the run starts inside the unit
    for (size_t i = 0; i < lanes.size(); ++i) {
      for (uint32_t k = 0; k < c0; ++k) lanes[i].pos += k < u.lanes[i].advance.size() ? u.lanes[i].advance[k] : 0;
      lanes[i].first = lanes[i].pos;
    }
    auto passed = [&] {
      for (size_t i = 0; i < lanes.size(); ++i)
        if (lanes[i].pos < std::min(u.lanes[i].panel_len, done + 8 * kG)) return false;
      return true;
    };
    while (done + 8 * kG < u.n_win8 && passed()) done += 8 * kG;
    for (Lane& l : lanes)
      for (uint32_t col = done; col < (l.pos & ~7u); col += 8) store(l, col, zeros);
  }
  const uint32_t len = c_end - c0, pieces = (len + kP - 1) / kP;
  uint32_t at = c0;
  for (uint32_t p = 0; p < pieces; ++p) {
    const uint32_t n = len / pieces + (p < len % pieces ? 1 : 0);
    for (uint32_t k = 0; k < n; ++k) {
      for (size_t i = 0; i < lanes.size(); ++i) append(i, at + k);
      if (k % kLook == kLook - 1 && (n >= kP - 1 ? k + 1 < kP : k + 1 < n)) multiply_ready(false);
    }
    multiply_ready(false);
    at += n;
  }
  if (c_end == u.n_chunks) {
    for (uint32_t before = ~0u; done < u.n_win8 && done != before;) {
      before = done;
      multiply_ready(false);
    }
    CHECK(done == u.n_win8, "unit left at column %u of %u", done, u.n_win8);
  } else {   // the unit goes on elsewhere: what the lanes have, zeros behind it
    for (Lane& l : lanes) store(l, l.pos, l.carry);
    for (;;) {
      bool left = false;
      for (const Lane& l : lanes) left = left || l.pos > done;
      if (!left) break;
      for (Lane& l : lanes)
        for (uint32_t k = 0; k < kG; ++k)
          if (done + 8 * k > l.pos) store(l, done + 8 * k, zeros);
      multiply_ready(true);
    }
  }
  return wrong;
}

// Streams whose lanes come to exactly the distance a size of the ring takes and stay there for a while: a fast lane, a slow
// one, others in between; whole panels, and a shorter one in every ragged unit; units as a whole and cut into runs.
static void ring() {
  uint64_t state = 88172645463325252ull;
  auto random = [&](uint32_t n) {
    state ^= state << 13, state ^= state >> 7, state ^= state << 17;
    return (uint32_t)(state % n);
  };
  int at_limit[2] = {0, 0}, units = 0, planted[2] = {0, 0};
  for (int trial = 0; trial < 20000; ++trial) {
    const int form = trial & 1;
    const bool ragged = trial % 8 != 0;
    const uint32_t limit = form ? tq::kSmallRingSpread : tq::kRingSpread;
    const uint32_t seg = ragged ? 16 * (16 + random(49)) : 32 * (8 + random(25));   // 256..1024
    const uint32_t shorter = ragged ? 1 + random(seg) : seg, hold = random(40), wobble = random(3);
    Unit u;
    u.bytes = form ? tq::kSmallRingBytes : tq::kRingBytes;
    u.ragged = ragged;
    u.lanes.assign(6, LaneStream{seg, {}});
    if (ragged) u.lanes[4].panel_len = u.lanes[5].panel_len = shorter;
    std::vector<uint32_t> pos(6, 0);
    uint32_t held = 0, gap = 0, burst = 0;
    for (bool busy = true; busy;) {
      uint32_t step[6];
      if (gap < limit) {
        step[1] = 4 + (random(4) < wobble);
        step[0] = std::min(8u, step[1] + (limit - gap));
        gap += step[0] - step[1];
      } else if (held++ < hold || pos[0] < seg) {
        if (burst) --burst;
        else if (random(4) == 0) burst = 6;   // pairs alone for a while: the most a lane gains between two looks
        step[0] = step[1] = burst ? 8 : 4 + random(5);
      }
      if (gap >= limit && held >= hold) step[0] = 4 + random(5), step[1] = 4 + random(5);
      for (int i : {2, 3, 4, 5}) {   // between the two (equal steps keep them there)
        const uint32_t low = pos[1] + step[1], high = std::min(pos[0], pos[1] + gap) + step[0];
        const uint32_t least = std::max(low, pos[i] + 4), most = std::min(high, pos[i] + 8);
        step[i] = least <= most ? least - pos[i] + random(most - least + 1) : least > pos[i] + 8 ? 8 : 4;
      }
      busy = false;
      for (int i = 0; i < 6; ++i) {
        const uint32_t len = u.lanes[i].panel_len;
        if (pos[i] >= len) continue;
        const uint32_t n = std::min(step[i], len - pos[i]);
        u.lanes[i].advance.push_back(n);
        pos[i] += n;
        busy = true;
      }
    }
    u.n_chunks = 0;
    for (const LaneStream& l : u.lanes) u.n_chunks = std::max<uint32_t>(u.n_chunks, l.advance.size());
    const uint32_t group = 8 * tq::ring_group(u.bytes), spread = spread_of(u.lanes, u.n_chunks);
    u.n_win8 = (seg + group - 1) / group * group;
    if (spread > limit) continue;
    at_limit[form] += spread == limit && ragged;
    ++units;
    for (int cuts = 0; cuts < 3; ++cuts) {
      std::vector<uint32_t> cut = {0, u.n_chunks};
      for (int c = 0; c < cuts; ++c) cut.push_back(1 + random(u.n_chunks - 1));
      std::sort(cut.begin(), cut.end());
      std::vector<std::vector<int>> taken;
      for (const LaneStream& l : u.lanes) taken.emplace_back(l.panel_len, 0);
      for (size_t c = 0; c + 1 < cut.size(); ++c)
        if (cut[c] < cut[c + 1]) {
          const int wrong = decode(u, cut[c], cut[c + 1], false, taken);
          CHECK(wrong == 0, "trial %d, spread %u, ring of %u, segments of %u and %u, chunks %u..%u of %u: %d columns wrong", trial, spread, u.bytes, seg, shorter, cut[c], cut[c + 1], u.n_chunks, wrong);
        }
      for (size_t i = 0; i < taken.size(); ++i)
        for (size_t col = 0; col < taken[i].size(); ++col) CHECK(taken[i][col] == 1, "trial %d, lane %zu, column %zu taken %d times", trial, i, col, taken[i][col]);
    }
    std::vector<std::vector<int>> taken;
    for (const LaneStream& l : u.lanes) taken.emplace_back(l.panel_len, 0);
    planted[form] += decode(u, 0, u.n_chunks, true, taken) != 0;
  }
  CHECK(at_limit[0] > 500 && at_limit[1] > 500, "%d, %d ragged units at the limits", at_limit[0], at_limit[1]);
  // the streams reach the edge: a store of the empty leftover is found in both sizes
  CHECK(planted[0] > 0 && planted[1] > 0, "%d, %d units with the planted mistake wrong", planted[0], planted[1]);
  std::printf("%d units decoded, %d and %d ragged ones at the limits, %d and %d wrong with the mistake\n", units, at_limit[0], at_limit[1], planted[0], planted[1]);
}

// Marks of units of any lengths: no two in one place, none outside the room for them, none over the offsets.
static void marks() {
  unsigned long total = 0;
  uint32_t state = 12345;
  auto next = [&](uint32_t n) { return (state = state * 1664525u + 1013904223u) / 65536u % n; };
  for (uint32_t longest : {1u, 7u, 8u, 9u, 17u, 36u, 260u}) {
    for (int turn = 0; turn < 60; ++turn) {
      const uint32_t n_units = 1 + next(300);
      uint32_t at = 0;
      uint64_t behind = 0;   // places up to here are taken
      for (uint32_t u = 0; u < n_units; ++u) {
        const uint32_t len = 1 + next(longest);
        for (uint32_t k = 1; k * tq::kMarkChunks < len; ++k, ++total) {
          const uint64_t place = tq::mark_index(at) + k;
          CHECK(!(place < behind), "unit %u mark %u", u, k);
          behind = place + 1;
        }
        at += len;
      }
      for (uint32_t seg_cols : {16u, 496u, 512u, 1024u}) {
        CHECK(!(behind * tq::mark_bytes(seg_cols) > tq::marks_size(at, seg_cols)), "%u units", n_units);
        CHECK(!(tq::marks_size(at, seg_cols) > at * 512ull / 64 * (tq::mark_bytes(seg_cols) / 64) + 128), "%u units of %u chunks", n_units, at);   // of the codes
        const uint32_t most = seg_cols / 2;   // pairs of a lane
        CHECK(!(tq::mark_bytes(seg_cols) == 64 ? most > 255 : most > 65535), "%u columns", seg_cols);
      }
      CHECK(!(tq::marks_at(n_units) < 4 * ((uint64_t)n_units + 1) || tq::marks_at(n_units) % 2), "%u units", n_units);
    }
  }
  std::printf("%lu marks\n", total);
}

// Workgroups that take equal numbers of units: every unit once, in order, no band in more than two shares where bands_cut_once says so.
static void shared() {
  unsigned long cuts = 0, once = 0;
  uint32_t state = 99;
  auto next = [&](uint32_t n) { return (state = state * 1664525u + 1013904223u) / 65536u % n; };
  for (int turn = 0; turn < 20000; ++turn) {
    const uint32_t n_quads = 1 + next(9), n_bands = 1 + next(turn % 4 ? 400 : 9000), wgs = 1 + next(256), units = n_bands * n_quads, first = next(800) * 256;
    for (uint32_t kind : {0u, tq::kShareUnits}) {
      const uint32_t items = (kind ? units : n_bands) / wgs;
      if (items >= tq::kMaxSharedItems) continue;
      const uint32_t word = tq::line_word(first, items) | kind, next_word = tq::line_word(first + wgs, 3) | (turn & 1 ? tq::kShareUnits : 0u);
      std::vector<uint32_t> sharers(n_bands, 0);
      uint32_t at = 0;
      bool empty = false;
      for (uint32_t k = 0; k < wgs; ++k, ++cuts) {
        uint32_t lo, hi;
        tq::shared_share(word, next_word, n_bands, n_quads, first + k, lo, hi);
        CHECK(lo == at && hi >= lo && (kind || lo % n_quads == 0), "%u workgroups, %u bands of %u", wgs, n_bands, n_quads);
        for (uint32_t b = lo / n_quads; lo < hi && b <= (hi - 1) / n_quads; ++b) ++sharers[b];
        empty = empty || lo == hi;
        at = hi;
      }
      CHECK(at == units, "%u of %u units", at, units);
      if (!kind) continue;
      const bool two = *std::max_element(sharers.begin(), sharers.end()) <= 2 && !empty;
      CHECK(two == tq::bands_cut_once(n_bands, n_quads, wgs), "%u workgroups, %u bands of %u", wgs, n_bands, n_quads);
      once += two;
    }
  }
  std::printf("%lu shares, %lu matrices with bands cut once\n", cuts, once);
}

// Which stages of a staged step are cut by units: those that gain by it, whose outputs are in nobody's place, behind a stage in which every
// workgroup has work.
static void stages() {
  struct Shape {
    uint32_t rows, cols;
  };
  typedef std::vector<std::vector<Shape>> Stages;
  // outputs and activations apart, quads of 4 segments of `seg` columns; x, y: from -> to moves an address
  auto plan = [&](const Stages& shapes, uint32_t seg, bool may_share, int no_adds, int from, int to, bool to_x) {
    std::vector<tq::StageItem> m;
    std::vector<uint32_t> first;
    uint64_t at = 1 << 20;
    for (const auto& stage : shapes) {
      first.push_back((uint32_t)m.size());
      for (const Shape& t : stage) {
        const uint64_t x = at, x_end = x + t.cols * 2, y = x_end + 64, y_end = y + t.rows * 4;
        m.push_back({(t.rows + 15) / 16, (t.cols + 4 * seg - 1) / (4 * seg), t.cols, x, x_end, y, y_end});
        at = y_end + 64;
      }
    }
    first.push_back((uint32_t)m.size());
    if (from >= 0) {   // product `from`'s outputs end inside product `to`'s activations or outputs
      const uint64_t bytes = m[from].y_end - m[from].y;
      m[from].y_end = (to_x ? m[to].x : m[to].y) + 4;
      m[from].y = m[from].y_end - bytes;
    }
    const tq::StageLine line = tq::plan_stages((int)m.size(), m.data(), first.data(), (uint32_t)shapes.size(), 256, may_share, [&](int i) { return i != no_adds; });
    std::vector<int> shared;   // the stages that are
    for (size_t k = 0; k < shapes.size(); ++k)
      if (!line.words.empty() && line.words[first[k]] & tq::kShareUnits) shared.push_back((int)k);
    CHECK(line.shared == !shared.empty(), "%zu stages", shared.size());
    return shared;
  };
  typedef std::vector<int> V;
  int n = 0;
  auto same = [&](const V& got, const V& want, const char* what) {
    CHECK(got == want, "%s: %zu stages shared", what, got.size());
    ++n;
  };
  // the shapes that the tests of the device take
  const Stages a = {{{4096, 256}}, {{2033, 2048}}, {{5111, 768}}, {{3000, 768}, {1000, 768}}}, b = {{{4096, 256}}, {{2048, 512}, {3072, 512}}, {{3072, 2000}}, {{2048, 1000}}};
  const Stages c = {{{4096, 256}}, {{2048, 2048}}, {{2048, 4096}}}, d = {{{4096, 256}}, {{2048, 2048}}, {{2048, 2048}}, {{2048, 2048}}};
  same(plan(a, 64, true, -1, -1, -1, false), V{1, 2}, "a");
  same(plan(b, 64, true, -1, -1, -1, false), V{1, 2, 3}, "b");
  same(plan(c, 64, true, -1, -1, -1, false), V{1, 2}, "c");
  same(plan(d, 64, true, -1, -1, -1, false), V{1, 2, 3}, "d");
  // a LLaMA-3.2-3B layer: q, k, v and down; o and gate, up have whole bands
  const Stages layer = {{{3072, 3072}, {1024, 3072}, {1024, 3072}}, {{3072, 3072}}, {{8192, 3072}, {8192, 3072}}, {{3072, 8192}}, {{3072, 3072}, {1024, 3072}, {1024, 3072}}};
  const V of_layer = plan(layer, 256, true, -1, -1, -1, false);
  CHECK(std::count(of_layer.begin(), of_layer.end(), 3) == 1 && std::count(of_layer.begin(), of_layer.end(), 0) == 0, "%zu stages of a layer", of_layer.size());
  same(plan(d, 64, false, -1, -1, -1, false), V{}, "not a kernel that can");
  // (stage 2 in whole bands leaves workgroups without work, and stage 3 with whole bands)
  same(plan(d, 64, true, 2, -1, -1, false), V{1}, "outputs that cannot be added to");
  for (bool x : {false, true}) {
    same(plan(d, 64, true, -1, 2, 1, x), V{1}, "a stage's outputs over the stage before");
    same(plan(d, 64, true, -1, 1, 2, x), x ? V{1, 2, 3} : V{1}, "a stage's outputs over the next one's outputs, or read by the next one");
    same(plan(d, 64, true, -1, 3, 1, x), V{1, 2, 3}, "outputs over those of two stages before");
    same(plan(b, 64, true, -1, 1, 2, x), V{2, 3}, "two outputs of a stage in one place");
  }
  same(plan(d, 64, true, -1, 2, 2, true), V{1}, "outputs over their own activations");
  same(plan({{{16, 256}}, {{2048, 2048}}, {{2048, 2048}}}, 64, true, -1, -1, -1, false), V{}, "workgroups without work in the stage before");
  same(plan({{{4096, 256}}, {{1024, 4096}}}, 64, true, -1, -1, -1, false), V{}, "bands that would be cut three times");
  std::printf("%d plans of stages\n", n);
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "listing")) listing();
  else if (!std::strcmp(what, "assign")) assign();
  else if (!std::strcmp(what, "cuts")) cuts();
  else if (!std::strcmp(what, "ring")) ring();
  else if (!std::strcmp(what, "marks")) marks();
  else if (!std::strcmp(what, "shared")) shared();
  else if (!std::strcmp(what, "stages")) stages();
  else return 2;
  return 0;
}
