// Host-only exercise of the schedule of k_matvec_ring (tq_plan.h) in both sizes of its rings: units whose lanes are as far apart
// as level_unit leaves them, decoded piece by piece as the kernel does it, lanes that have finished going on by a column a code.
// Every column has to be in the ring, unharmed, when it is multiplied, and every one is multiplied once.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>
#include "../paper_2509_22951_amd/csrc/tq_level.h"
#include "../paper_2509_22951_amd/csrc/tq_plan.h"

static uint64_t state = 88172645463325252ull;
static uint32_t rnd(uint32_t n) {
  state ^= state << 13, state ^= state >> 7, state ^= state << 17;
  return (uint32_t)(state % n);
}

// advance[chunk][lane]: columns; len[lane]: of its segment, `seg` or 0.  Returns the places that held something else.
static int decode(uint32_t bytes, const std::vector<std::vector<uint32_t>>& advance, const std::vector<uint32_t>& len, uint32_t seg) {
  const uint32_t kP = tq::ring_piece(bytes), kLook = tq::ring_step(bytes), group = 8 * tq::ring_group(bytes), n_chunks = (uint32_t)advance.size();
  std::vector<std::vector<uint32_t>> ring(64, std::vector<uint32_t>(bytes, 0)), carry(64, std::vector<uint32_t>(8, 0));
  std::vector<uint32_t> pos(64);
  for (uint32_t l = 0; l < 64; ++l) pos[l] = len[l] ? 0 : seg;   // a row past the end of the matrix
  uint32_t done = 0;
  int wrong = 0;
  auto append = [&](uint32_t chunk) {
    for (uint32_t l = 0; l < 64; ++l) {
      std::vector<uint32_t> both(16, 0);
      std::copy(carry[l].begin(), carry[l].end(), both.begin());
      const uint32_t n = advance[chunk][l], after = pos[l] + n;
      for (uint32_t k = 0; k < n; ++k) both[(pos[l] & 7) + k] = pos[l] + k + 1;
      std::copy(both.begin(), both.begin() + 8, ring[l].begin() + (pos[l] & (bytes - 8)));
      std::copy(both.begin() + ((after ^ pos[l]) >= 8 ? 8 : 0), both.begin() + ((after ^ pos[l]) >= 8 ? 16 : 8), carry[l].begin());
      pos[l] = after;
    }
  };
  auto look = [&] {
    if (done + group > seg) return;
    for (uint32_t l = 0; l < 64; ++l)
      if (pos[l] < done + group) return;
    for (uint32_t l = 0; l < 64; ++l)
      for (uint32_t col = done; len[l] && col < done + group; ++col) wrong += ring[l][col % bytes] != col + 1;
    done += group;
  };
  const uint32_t pieces = (n_chunks + kP - 1) / kP;
  for (uint32_t p = 0, at = 0; p < pieces; ++p) {
    const uint32_t n = n_chunks / pieces + (p < n_chunks % pieces ? 1 : 0);
    if (n >= kP - 1) {
      for (uint32_t k = 0; k < kP - 1; ++k) {
        append(at + k);
        if (k % kLook == kLook - 1) look();
      }
      if (n == kP) append(at + kP - 1);
    } else {
      for (uint32_t k = 0; k < kP - 2; ++k) {
        if (k < n) append(at + k);
        if (k % kLook == kLook - 1 && k + 1 < n) look();
      }
    }
    look();
    at += n;
  }
  if (done != seg) {
    std::printf("ring of %u: unit left at column %u of %u\n", bytes, done, seg);
    return 1 << 20;
  }
  return wrong;
}

int main() {
  const uint32_t n_entries = 1000;
  std::vector<uint32_t> word(n_entries + 1, 0);
  int units[2] = {0, 0}, at_limit[2] = {0, 0}, planted[2] = {0, 0};
  for (int trial = 0; trial < 2000; ++trial) {
    const int form = trial & 1;
    const uint32_t bytes = form ? tq::kSmallRingBytes : tq::kRingBytes, limit = form ? tq::kSmallRingSpread : tq::kRingSpread;
    const uint32_t seg = 32 * (1 + rnd(8)), rows = trial % 5 == 0 ? 1 + rnd(15) : 16;
    std::vector<std::vector<uint16_t>> lane(64);
    std::vector<uint32_t> len(64, 0);
    uint32_t longest = 1;
    for (uint32_t l = 0; l < 64; ++l) {
      len[l] = l % 16 < rows ? seg : 0;
      const uint32_t share = trial % 3 ? (rnd(2) ? 100 : rnd(101)) : l * 100 / 63;
      for (uint32_t pos = 0; pos < len[l];) {
        const bool pair = pos + 2 <= len[l] && rnd(100) < share;
        lane[l].push_back((uint16_t)(pair ? 256 : 1));
        pos += pair ? 2 : 1;
      }
      longest = std::max<uint32_t>(longest, (uint32_t)lane[l].size());
    }
    const uint32_t n_chunks = (longest + 3) / 4 + (rnd(8) ? 0 : rnd(4));   // (a unit may be longer than its longest lane)
    std::vector<uint16_t> in((size_t)n_chunks * tq::kChunkWords, (uint16_t)n_entries), out(in.size());
    auto at = [](uint32_t l, uint32_t k) { return (size_t)(k / 4) * tq::kChunkWords + 4 * l + k % 4; };
    for (uint32_t l = 0; l < 64; ++l)
      for (uint32_t k = 0; k < lane[l].size(); ++k) in[at(l, k)] = lane[l][k];
    auto columns = [&](uint32_t most) {   // of the unit brought within `most` columns; empty: it cannot be
      std::vector<std::vector<uint32_t>> advance;
      if (!tq::level_unit(in.data(), n_chunks, n_entries, word.data(), most, out.data())) return advance;
      advance.assign(n_chunks, std::vector<uint32_t>(64, 0));
      for (uint32_t l = 0; l < 64; ++l)
        for (uint32_t k = 0; k < 4 * n_chunks; ++k) advance[k / 4][l] += out[at(l, k)] >= 256 ? 2 : 1;
      return advance;
    };
    const auto advance = columns(limit);
    if (advance.empty()) continue;
    std::vector<uint32_t> pos(64, 0);
    uint32_t far = 0;
    for (uint32_t k = 0; k < n_chunks; ++k) {
      uint32_t least = UINT32_MAX, most = 0;
      for (uint32_t l = 0; l < 64; ++l) {
        pos[l] += advance[k][l];
        most = std::max(most, pos[l]);
        if (pos[l] < len[l]) least = std::min(least, pos[l]);
      }
      if (least != UINT32_MAX) far = std::max(far, most - least);
    }
    ++units[form];
    at_limit[form] += far >= limit - 1;
    if (const int wrong = decode(bytes, advance, len, seg)) {
      std::printf("trial %d, ring of %u, segments of %u: %d columns wrong\n", trial, bytes, seg, wrong);
      return 1;
    }
    const auto apart = columns(limit + 32);   // further apart than the ring takes: it has to show
    if (!apart.empty()) planted[form] += decode(bytes, apart, len, seg) != 0;
  }
  std::printf("%d / %d units decoded, %d / %d at the limit, %d / %d wrong beyond it\n", units[0], units[1], at_limit[0], at_limit[1], planted[0], planted[1]);
  return at_limit[0] > 100 && at_limit[1] > 100 && planted[0] > 0 && planted[1] > 0 ? 0 : 1;
}
