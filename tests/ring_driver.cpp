// Host-only exercise of the schedules of k_matvec_ring and k_matvec_runs (tq_plan.h) in both sizes of their rings: units whose
// lanes are as far apart as level_unit leaves them, decoded piece by piece as the kernels do it.  Every column has to be in the
// ring, unharmed, when it is multiplied, and every one is multiplied once.
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
static uint16_t* scratch(uint32_t n_chunks) {
  static std::vector<uint16_t> room;
  room.assign(tq::level_scratch(n_chunks), 0xFFFF);
  return room.data();
}

// k_matvec_ring: whole units, lanes that have finished go on by a column a code.
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

// k_matvec_runs: chunks [c0, c_end) of a unit whose panels may be short, lanes that have finished stay at their ends, what a lane
// left over of a segment that ends inside a piece is stored at every look.  taken[lane][column]: how often it was multiplied.
static int decode_run(uint32_t bytes, const std::vector<std::vector<uint32_t>>& advance, const std::vector<uint32_t>& len, uint32_t n_win8,
                      uint32_t c0, uint32_t c_end, std::vector<std::vector<uint32_t>>& taken) {
  const uint32_t kP = tq::ring_piece(bytes), kLook = tq::ring_step(bytes), group = 8 * tq::ring_group(bytes), n_chunks = (uint32_t)advance.size();
  struct Lane {
    uint32_t pos = 0, first = 0, ring[128] = {}, carry[8] = {};
  };
  std::vector<Lane> lanes(64);
  uint32_t done = 0;
  int wrong = 0;
  const uint32_t zeros[8] = {};
  auto store = [&](Lane& l, uint32_t col, const uint32_t* v) { std::copy(v, v + 8, l.ring + (col & (bytes - 8))); };
  auto append = [&](uint32_t chunk) {
    for (uint32_t i = 0; i < 64; ++i) {
      Lane& l = lanes[i];
      uint32_t both[16] = {};
      std::copy(l.carry, l.carry + 8, both);
      const uint32_t n = advance[chunk][i], after = std::min(l.pos + n, len[i]);
      for (uint32_t k = 0; k < n && l.pos + k < len[i]; ++k) both[(l.pos & 7) + k] = l.pos + k + 1;
      store(l, l.pos, both);
      const uint32_t* rest = (after ^ l.pos) >= 8 ? both + 8 : both;
      std::copy(rest, rest + 8, l.carry);
      l.pos = after;
    }
  };
  auto look = [&](bool ready) {
    for (Lane& l : lanes)
      if (tq::ring_leftover(l.pos)) store(l, l.pos, l.carry);
    if (done + group > n_win8) return;
    for (uint32_t i = 0; i < 64 && !ready; ++i)
      if (lanes[i].pos < std::min(len[i], done + group)) return;
    for (uint32_t i = 0; i < 64; ++i)
      for (uint32_t col = done; col < std::min(done + group, len[i]); ++col) {   // (activations are zero behind the panel)
        const uint32_t want = col >= lanes[i].first && col < lanes[i].pos ? col + 1 : 0;
        wrong += lanes[i].ring[col % bytes] != want;
        taken[i][col] += want != 0;
      }
    done += group;
  };
  if (c0) {   // the run starts inside the unit
    bool passed = true;
    for (uint32_t i = 0; i < 64; ++i) {
      for (uint32_t k = 0; k < c0; ++k) lanes[i].pos += advance[k][i];
      lanes[i].first = lanes[i].pos = std::min(lanes[i].pos, len[i]);
    }
    while (passed && done + group < n_win8) {
      for (uint32_t i = 0; i < 64; ++i) passed = passed && lanes[i].pos >= std::min(len[i], done + group);
      if (passed) done += group;
    }
    for (Lane& l : lanes)
      for (uint32_t col = done; col < (l.pos & ~7u); col += 8) store(l, col, zeros);
  }
  const uint32_t chunks = c_end - c0, pieces = (chunks + kP - 1) / kP;
  for (uint32_t p = 0, at = c0; p < pieces; ++p) {
    const uint32_t n = chunks / pieces + (p < chunks % pieces ? 1 : 0);
    for (uint32_t k = 0; k < n; ++k) {
      append(at + k);
      if (k % kLook == kLook - 1 && (n >= kP - 1 ? k + 1 < kP : k + 1 < n)) look(false);
    }
    look(false);
    at += n;
  }
  if (c_end == n_chunks) {
    for (uint32_t before = ~0u; done < n_win8 && done != before;) {
      before = done;
      look(false);
    }
    if (done != n_win8) return 1 << 20;
  } else {   // the unit goes on elsewhere: what the lanes have, zeros behind it
    for (Lane& l : lanes) store(l, l.pos, l.carry);
    for (;;) {
      bool left = false;
      for (const Lane& l : lanes) left = left || l.pos > done;
      if (!left) break;
      for (Lane& l : lanes)
        for (uint32_t k = 0; k < group / 8; ++k)
          if (done + 8 * k > l.pos) store(l, done + 8 * k, zeros);
      look(true);
    }
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
    const bool runs = trial % 4 >= 2;
    const uint32_t seg = runs ? 16 * (1 + rnd(32)) : 32 * (1 + rnd(8)), rows = trial % 5 == 0 ? 1 + rnd(15) : 16;
    const uint32_t shorter = runs && rnd(3) ? 1 + rnd(seg) : seg, panels = runs ? 1 + rnd(4) : 4;   // the last panel there is
    std::vector<std::vector<uint16_t>> lane(64);
    std::vector<uint32_t> len(64, 0);
    uint32_t longest = 1;
    for (uint32_t l = 0; l < 64; ++l) {
      len[l] = l % 16 >= rows || l / 16 >= panels ? 0 : l / 16 + 1 == panels ? shorter : seg;
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
      if (!tq::level_unit(in.data(), n_chunks, n_entries, word.data(), most, out.data(), scratch(n_chunks))) return advance;
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
    if (runs) {
      const uint32_t group = 8 * tq::ring_group(bytes), n_win8 = ((panels > 1 ? seg : shorter) + group - 1) / group * group;
      for (uint32_t parts = 1; parts <= 4 && parts <= n_chunks; ++parts) {
        std::vector<std::vector<uint32_t>> taken(64, std::vector<uint32_t>(seg, 0));
        int wrong = 0;
        for (uint32_t p = 0; p < parts; ++p) wrong += decode_run(bytes, advance, len, n_win8, n_chunks * p / parts, n_chunks * (p + 1) / parts, taken);
        for (uint32_t l = 0; l < 64; ++l)
          for (uint32_t col = 0; col < len[l]; ++col) wrong += taken[l][col] != 1;
        if (wrong) {
          std::printf("trial %d, ring of %u, segments of %u, last panel %u of %u: %d columns wrong in %u runs\n", trial, bytes, seg, shorter, panels, wrong, parts);
          return 1;
        }
      }
      continue;
    }
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
