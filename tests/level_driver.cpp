// Host-only exercise of level_unit (csrc/tq_level.h): units whose lanes run apart, brought closer together.  Every lane has to
// stand for the same bytes, and no lane may be more than the limit ahead of an unfinished one after any chunk.
#include <algorithm>
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <ctime>
#include <memory>
#include <thread>
#include <vector>
#include "../paper_2509_22951_amd/csrc/tq_level.h"
#include "../paper_2509_22951_amd/csrc/tq_plan.h"

using Codes = std::vector<uint16_t>;
static uint64_t state = 88172645463325252ull;
static uint32_t rnd(uint32_t n) {
  state ^= state << 13, state ^= state >> 7, state ^= state << 17;
  return (uint32_t)(state % n);
}
static uint16_t* scratch(uint32_t n_chunks) {
  static std::vector<uint16_t> room;
  room.assign(tq::level_scratch(n_chunks), 0xFFFF);
  return room.data();
}

// Many units at once: the same codes as one by one, a unit that cannot be levelled refuses them all, and several threads
// take part (process time against the clock, where there are processors for it).
static bool many() {
  const uint32_t n_entries = 1000, n_units = 800, seg = 256;
  std::vector<uint32_t> word(n_entries + 1, 0);
  for (uint32_t c = 0; c < n_entries; ++c) word[c] = c < 256 ? c : rnd(65536);
  auto unit = [&](bool refused) {   // even lanes all pairs, odd ones single bytes; refused: they change places half way
    Codes u((size_t)(refused ? 3 * seg / 16 : seg / 4) * tq::kChunkWords, (uint16_t)n_entries);
    for (uint32_t l = 0; l < 64; ++l)
      for (uint32_t pos = 0, k = 0; pos < seg; ++k) {
        const bool pair = (l % 2 == 0) == (!refused || pos < seg / 2);
        u[(size_t)(k / 4) * tq::kChunkWords + 4 * l + k % 4] = (uint16_t)(pair ? 256 + rnd(n_entries - 256) : rnd(256));
        pos += pair ? 2 : 1;
      }
    return u;
  };
  Codes codes;
  std::vector<uint32_t> uoff = {0}, wide;
  for (uint32_t u = 0; u < n_units; ++u) {
    const Codes c = unit(u == n_units / 2);
    codes.insert(codes.end(), c.begin(), c.end());
    uoff.push_back((uint32_t)(codes.size() / tq::kChunkWords));
    if (u % 50 && u != n_units / 2) wide.push_back(u);
  }
  Codes want;
  for (uint32_t u : wide) {
    Codes c((size_t)(uoff[u + 1] - uoff[u]) * tq::kChunkWords);
    if (!tq::level_unit(codes.data() + (size_t)uoff[u] * tq::kChunkWords, uoff[u + 1] - uoff[u], n_entries, word.data(), tq::kSmallRingSpread, c.data(), scratch(uoff[u + 1] - uoff[u]))) return std::printf("refused\n"), false;
    want.insert(want.end(), c.begin(), c.end());
  }
  std::unique_ptr<uint16_t[]> out;
  for (unsigned threads : {1u, 3u, 64u})
    if (!tq::level_units(codes.data(), uoff.data(), wide, n_entries, word.data(), tq::kSmallRingSpread, threads, out) || !std::equal(want.begin(), want.end(), out.get()))
      return std::printf("%u threads: other codes\n", threads), false;
  std::vector<uint32_t> with = wide;
  with.insert(std::lower_bound(with.begin(), with.end(), n_units / 2), n_units / 2);
  if (tq::level_units(codes.data(), uoff.data(), with, n_entries, word.data(), tq::kSmallRingSpread, 4, out)) return std::printf("taken with a unit that cannot be levelled\n"), false;
  if (!tq::level_units(codes.data(), uoff.data(), {}, n_entries, word.data(), tq::kSmallRingSpread, 4, out)) return std::printf("none refused\n"), false;
  const std::vector<uint32_t> closed = tq::close_gaps({1, 2, 4, 10, 17, 30, 36});
  if (closed != std::vector<uint32_t>{1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 17, 30, 31, 32, 33, 34, 35, 36} || !tq::close_gaps({}).empty()) return std::printf("gaps\n"), false;
  // a unit that is close together: its own codes, zeros for its pads
  Codes plain(4 * tq::kChunkWords, (uint16_t)n_entries), same(plain.size());
  for (uint32_t l = 0; l < 64; ++l)
    for (uint32_t k = 0; k < 8 + l % 8; ++k) plain[(size_t)(k / 4) * tq::kChunkWords + 4 * l + k % 4] = (uint16_t)rnd(n_entries);
  if (!tq::level_unit(plain.data(), 4, n_entries, word.data(), tq::kSmallRingSpread, same.data(), scratch(4))) return std::printf("close unit refused\n"), false;
  for (size_t k = 0; k < plain.size(); ++k)
    if (same[k] != (plain[k] == n_entries ? 0 : plain[k])) return std::printf("close unit changed\n"), false;
  double shared = 0;
  for (int k = 0; k < 5 && shared < 1.5; ++k) {
    const std::clock_t c0 = std::clock();
    const auto t0 = std::chrono::steady_clock::now();
    tq::level_units(codes.data(), uoff.data(), wide, n_entries, word.data(), tq::kSmallRingSpread, 4, out);
    const double wall = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    shared = std::max(shared, (double)(std::clock() - c0) / CLOCKS_PER_SEC / wall);
  }
  std::printf("%zu units at once, %.1f threads at work\n", wide.size(), shared);
  return shared >= 1.5 || std::thread::hardware_concurrency() < 4;
}

int main() {
  if (!many()) return 1;
  const uint32_t n_entries = 1000, pad = n_entries;
  std::vector<uint32_t> word(n_entries + 1, 0);
  for (uint32_t c = 0; c < n_entries; ++c) word[c] = c < 256 ? c : rnd(65536);
  int levelled = 0, refused = 0, late = 0, by_chance = 0;
  for (int trial = 0; trial < 4000; ++trial) {
    const uint32_t limit = trial % 3 == 0 ? tq::kRingSpread : tq::kSmallRingSpread, seg = 16 * (1 + rnd(64)), shorter = rnd(4) ? seg : rnd(seg);
    const uint32_t turn = trial % 4 == 3 ? seg / 2 : seg;   // some units: the lanes change places half way
    // lane l takes pairs with a probability of its own
    std::vector<std::vector<uint16_t>> lane(64);
    uint32_t longest = 1;
    for (uint32_t l = 0; l < 64; ++l) {
      const uint32_t len = trial % 5 == 0 && l % 16 == 15 ? 0 : l >= 48 ? shorter : seg, share = trial % 2 ? rnd(101) : l * 100 / 63;
      for (uint32_t pos = 0; pos < len;) {
        const bool pair = pos + 2 <= len && rnd(100) < (pos < turn ? share : 100 - share);
        lane[l].push_back((uint16_t)(pair ? 256 + rnd(n_entries - 256) : rnd(256)));
        pos += pair ? 2 : 1;
      }
      longest = std::max<uint32_t>(longest, lane[l].size());
    }
    const uint32_t n_chunks = (longest + 3) / 4 + (rnd(8) == 0);
    Codes in((size_t)n_chunks * tq::kChunkWords, (uint16_t)pad), out(in.size(), 0xFFFF);
    auto at = [](uint32_t l, uint32_t k) { return (size_t)(k / 4) * tq::kChunkWords + 4 * l + k % 4; };
    for (uint32_t l = 0; l < 64; ++l)
      for (uint32_t k = 0; k < lane[l].size(); ++k) in[at(l, k)] = lane[l][k];
    if (!tq::level_unit(in.data(), n_chunks, n_entries, word.data(), limit, out.data(), scratch(n_chunks))) {
      ++refused;
      by_chance += turn == seg;   // (a lane that is ahead can wait; of two with the same share of pairs the other may be later on)
      continue;
    }
    std::vector<uint32_t> pos(64, 0), len(64, 0);
    for (uint32_t l = 0; l < 64; ++l) {
      std::vector<uint8_t> want, got;
      for (uint16_t c : lane[l]) {
        want.push_back((uint8_t)word[c]);
        if (c >= 256) want.push_back((uint8_t)(word[c] >> 8));
      }
      for (uint32_t k = 0; k < 4 * n_chunks; ++k) {
        const uint16_t c = out[at(l, k)];
        if (c >= n_entries || (got.size() >= want.size() && c != 0)) {
          std::printf("trial %d, lane %u, code %u: %u\n", trial, l, k, c);
          return 1;
        }
        got.push_back((uint8_t)word[c]);
        if (c >= 256) got.push_back((uint8_t)(word[c] >> 8));
      }
      len[l] = want.size();
      if (got.size() < want.size() || !std::equal(want.begin(), want.end(), got.begin())) {
        std::printf("trial %d, lane %u: other bytes\n", trial, l);
        return 1;
      }
    }
    uint32_t far = 0, before = 0;
    std::vector<uint32_t> was(64, 0);
    for (uint32_t chunk = 0; chunk < n_chunks; ++chunk) {
      uint32_t least = UINT32_MAX, most = 0, least0 = UINT32_MAX, most0 = 0;
      for (uint32_t l = 0; l < 64; ++l) {
        for (uint32_t k = 4 * chunk; k < 4 * chunk + 4; ++k) {
          pos[l] += out[at(l, k)] >= 256 ? 2 : 1;
          was[l] += k < lane[l].size() && lane[l][k] >= 256 ? 2 : 1;
        }
        most = std::max(most, pos[l]);
        most0 = std::max(most0, was[l]);
        if (pos[l] < len[l]) least = std::min(least, pos[l]);
        if (was[l] < len[l]) least0 = std::min(least0, was[l]);
      }
      if (least != UINT32_MAX) far = std::max(far, most - least);
      if (least0 != UINT32_MAX) before = std::max(before, most0 - least0);
    }
    if (far > limit) {
      std::printf("trial %d: %u columns apart, %u before, limit %u\n", trial, far, before, limit);
      return 1;
    }
    levelled += before > limit;
    late += before > limit && turn < seg;
  }
  std::printf("%d units brought together (%d of them with lanes that change places), %d refused (%d of them without)\n", levelled, late, refused, by_chance);
  return levelled > 1000 && refused > 0 && by_chance < 5 ? 0 : 1;
}
