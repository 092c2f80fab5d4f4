// The code stream of a unit as the device keeps it, where that differs from the container's.  Host code, no GPU needed.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>
#include <memory>
#include <vector>

#include "tq_format.h"
#include "tq_plan.h"

namespace tq {

// Lanes close together.  The ring kernels hold a short stretch of every lane's segment and multiply what all lanes of a unit
// have passed, so the lanes may not be further apart than the ring is long.  In the first units of a matrix that starts a
// dictionary they are: some segments are still all single bytes, others all pairs.  A lane that is ahead can wait: any pair
// may be written as its two single bytes (codes 0..255 are the single bytes), which takes a code more for the same columns,
// and a lane that is ahead has codes to spare, for its stream is filled up with pads to the length of the longest.  So the
// unit keeps its length and its weights; only which of its codes are pairs changes.
//
// codes: the unit's n_chunks chunks as the container holds them (valid, runs of at most 2 bytes); word: the dictionary's.
// out: the same chunks with no lane ever more than `limit` columns ahead of an unfinished one after a chunk, lanes that have
// finished going on by a column a code, as the device's pads do (code 0, a single byte of value 0).  False when that cannot be
// done within the unit's length (a lane that is ahead now and slower than the others later on).
// flat: room for level_scratch(n_chunks) codes.
inline size_t level_scratch(uint32_t n_chunks) { return 64 * ((size_t)n_chunks + 1) * kChunkCodes; }
inline bool level_unit(const uint16_t* codes, uint32_t n_chunks, uint32_t n_entries, const uint32_t* word, uint32_t limit, uint16_t* out, uint16_t* flat) {
  static_assert(kChunkCodes == 4, "four codes are taken as 8 bytes");
  constexpr uint64_t kHigh = 0xFF00FF00FF00FF00ull, kTop = 0x8000800080008000ull;
  struct Lane {
    uint32_t next = 0, n = 0;   // codes taken, codes there are
    uint32_t pos = 0;           // columns passed
    int32_t half = -1;          // second byte of a pair of which the first has been written
  };
  Lane lane[64];
  // every lane's codes in a row, zeros for its pads and behind them
  const size_t stride = ((size_t)n_chunks + 1) * kChunkCodes;
  for (uint32_t k = 0; k < n_chunks; ++k)
    for (uint32_t l = 0; l < 64; ++l) std::memcpy(flat + l * stride + k * kChunkCodes, codes + (size_t)k * kChunkWords + l * kChunkCodes, 8);
  for (uint32_t l = 0; l < 64; ++l) {
    uint16_t* c = flat + l * stride;
    uint32_t n = n_chunks * kChunkCodes;
    std::memset(c + n, 0, 8);
    while (n && c[n - 1] == n_entries) c[--n] = 0;
    lane[l].n = n;
  }
  uint64_t four[64];     // the next four codes of every lane as they are,
  uint32_t after[64];    // and the column they lead to
  for (uint32_t chunk = 0; chunk < n_chunks; ++chunk) {
    uint32_t least = UINT32_MAX;
    for (uint32_t l = 0; l < 64; ++l) {
      const Lane& s = lane[l];
      uint64_t v;
      std::memcpy(&v, flat + l * stride + s.next, 8);
      if (s.half >= 0) v = v << 16 | (uint32_t)s.half;
      const uint64_t high = v & kHigh;   // a code from 256 on is a pair: a set bit in its high byte
      four[l] = v;
      after[l] = s.pos + kChunkCodes + (uint32_t)__builtin_popcountll(((high | (high & ~kTop) + ~kTop) & kTop));
      if (s.next + kChunkCodes - (s.half >= 0) < s.n) least = std::min(least, after[l]);
    }
    const uint64_t most = least == UINT32_MAX ? UINT64_MAX : (uint64_t)least + limit;   // (all finished: what follows is pads)
    for (uint32_t l = 0; l < 64; ++l) {
      Lane& s = lane[l];
      uint16_t* to = out + (size_t)chunk * kChunkWords + l * kChunkCodes;
      if (after[l] <= most) {
        std::memcpy(to, &four[l], 8);
        s.next += kChunkCodes - (s.half >= 0);
        s.pos = after[l];
        s.half = -1;
        continue;
      }
      for (uint32_t j = 0; j < kChunkCodes; ++j) {
        const uint32_t left = kChunkCodes - 1 - j;   // codes of the chunk that follow, of at least a column each
        const bool rest = s.half >= 0;
        const uint32_t c = rest ? (uint32_t)s.half : flat[l * stride + s.next], w = word[c];
        s.next += !rest;
        const bool pair = c >= 256, cut = pair && s.pos + 2 + left > most;
        // (two codes in the place of one must fit)
        if (cut && s.n - s.next >= (n_chunks - chunk) * kChunkCodes - 1 - j) return false;
        to[j] = (uint16_t)(cut ? w & 0xFF : c);
        s.half = cut ? (int32_t)(w >> 8 & 0xFF) : -1;
        s.pos += 1 + (pair && !cut);
      }
      if (s.pos > most) return false;
    }
  }
  for (const Lane& l : lane)
    if (l.next < l.n || l.half >= 0) return false;
  return true;
}

// The units `units` of a container (codes, uoff: its sections), levelled one behind the other into out by up to n_threads threads.
// False when one of them cannot be.  (Few units are wide of a matrix with a full dictionary and segments of 256 columns, nearly all
// with a small dictionary or wider segments; they are then as much work as the matrix's validation: ms, on 8 threads, level | validate:
// 6144 x 1024 with 3,000 entries 2.9 | 2.0, 2048 x 1024 in segments of 1024 2.5 | 2.4, 8192 x 3072 0.2 | 5.3.)
inline bool level_units(const uint16_t* codes, const uint32_t* uoff, const std::vector<uint32_t>& units, uint32_t n_entries, const uint32_t* word,
                        uint32_t limit, unsigned n_threads, std::unique_ptr<uint16_t[]>& out) {
  std::vector<size_t> at(units.size() + 1, 0);   // where in out, in chunks
  for (size_t i = 0; i < units.size(); ++i) at[i + 1] = at[i] + (uoff[units[i] + 1] - uoff[units[i]]);
  out.reset(new uint16_t[at.back() * kChunkWords]);
  constexpr size_t kThreadChunks = 128;   // of work that another thread is started for, a tenth of a millisecond
  std::atomic<size_t> next(0);
  std::atomic<bool> refused(false);
  size_t longest = 0;
  for (size_t i = 0; i < units.size(); ++i) longest = std::max(longest, at[i + 1] - at[i]);
  const size_t threads = std::max<size_t>(1, std::min<size_t>({n_threads, 16, units.size(), at.back() / kThreadChunks})), room = level_scratch((uint32_t)longest);
  std::unique_ptr<uint16_t[]> flat(new uint16_t[threads * room]);
  auto work = [&](size_t thread) {
    for (size_t i; (i = next.fetch_add(1)) < units.size() && !refused.load(std::memory_order_relaxed);)
      if (!level_unit(codes + (size_t)uoff[units[i]] * kChunkWords, (uint32_t)(at[i + 1] - at[i]), n_entries, word, limit, out.get() + at[i] * kChunkWords,
                      flat.get() + thread * room))
        refused = true;
  };
  {
    Threads th;
    for (size_t t = 1; t < threads; ++t) th.start(work, t);   // (a few units, as most matrices have at the start of a dictionary: this thread alone)
    work(0);
  }
  return !refused;
}

// The units between two of the list that are at most kUnitGap apart join it, so that it falls into few runs: a run is a copy to the
// device of its own, some 6 us, and levelling a unit that is close together already changes nothing but its pads.
constexpr uint32_t kUnitGap = 6;
inline std::vector<uint32_t> close_gaps(const std::vector<uint32_t>& units) {
  std::vector<uint32_t> all;
  for (uint32_t u : units) {
    const uint32_t from = !all.empty() && u - all.back() <= kUnitGap ? all.back() + 1 : u;
    for (uint32_t k = from; k <= u; ++k) all.push_back(k);
  }
  return all;
}

// What the ring kernels can do with a valid container whose units `wide` have lanes further apart than the small ring takes:
// 2 - k_matvec_ring and k_matvec_runs with rings of either size, 1 - k_matvec_runs with rings of 128 bytes, 0 - neither.  codes:
// for 2 and 1, what takes the place of those units' codes, one unit behind the other.
inline uint32_t ring_class(const void* blob, const Header& h, const std::vector<uint32_t>& wide, unsigned n_threads, std::unique_ptr<uint16_t[]>& codes) {
  if (h.lmax > 2) return 0;   // (runs of 3 and 4 bytes)
  const uint8_t* base = (const uint8_t*)blob;
  auto level_to = [&](uint32_t limit) {
    return level_units((const uint16_t*)(base + h.off_codes), (const uint32_t*)(base + h.off_uoff), wide, h.n_entries, (const uint32_t*)(base + h.off_dict), limit,
                       n_threads, codes);
  };
  return level_to(kSmallRingSpread) ? 2u : level_to(kRingSpread) ? 1u : 0u;
}

}  // namespace tq
