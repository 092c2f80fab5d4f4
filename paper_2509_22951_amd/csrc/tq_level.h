// The code stream of a unit as the device keeps it, where that differs from the container's.  Host code, no GPU needed.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstdint>
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
inline bool level_unit(const uint16_t* codes, uint32_t n_chunks, uint32_t n_entries, const uint32_t* word, uint32_t limit, uint16_t* out) {
  struct Lane {
    uint32_t next = 0, n = 0;   // codes taken, codes there are
    uint32_t pos = 0;           // columns passed
    int half = -1;              // second byte of a pair of which the first has been written
    bool finished() const { return next == n && half < 0; }
  };
  Lane lane[64];
  auto code = [&](uint32_t l, uint32_t k) { return codes[(size_t)(k / kChunkCodes) * kChunkWords + l * kChunkCodes + k % kChunkCodes]; };
  for (uint32_t k = 0; k < n_chunks * kChunkCodes; ++k)
    for (uint32_t l = 0; l < 64; ++l) lane[l].n += code(l, k) != n_entries;   // (pads only follow)
  // One chunk of a lane that may come to column `most`; false: it has no codes to spare for that.
  auto take = [&](uint32_t l, uint32_t chunk, uint64_t most, Lane& s) {
    for (uint32_t j = 0; j < kChunkCodes; ++j) {
      const uint32_t left = kChunkCodes - 1 - j;   // codes of the chunk that follow, of at least a column each
      uint16_t c = 0;
      if (s.half >= 0) {
        c = (uint16_t)s.half;
        s.half = -1;
      } else if (s.next < s.n) {
        c = code(l, s.next++);
        if (s.pos + 2 + left > most && c >= 256) {
          if (s.n - s.next >= (n_chunks - chunk) * kChunkCodes - 1 - j) return false;   // (two codes in the place of one must fit)
          s.half = (int)(word[c] >> 8 & 0xFF);
          c = (uint16_t)(word[c] & 0xFF);
        }
      }
      s.pos += c >= 256 ? 2 : 1;
      out[(size_t)chunk * kChunkWords + l * kChunkCodes + j] = c;
    }
    return true;
  };
  for (uint32_t chunk = 0; chunk < n_chunks; ++chunk) {
    Lane before[64];
    std::copy(lane, lane + 64, before);
    uint32_t least = UINT32_MAX;
    for (uint32_t l = 0; l < 64; ++l) {
      take(l, chunk, UINT64_MAX, lane[l]);
      if (!lane[l].finished()) least = std::min(least, lane[l].pos);
    }
    if (least == UINT32_MAX) continue;   // (all finished; what follows is pads)
    for (uint32_t l = 0; l < 64; ++l)
      if (lane[l].pos > least + limit) {
        lane[l] = before[l];
        if (!take(l, chunk, (uint64_t)least + limit, lane[l]) || lane[l].pos > least + limit) return false;
      }
  }
  for (const Lane& l : lane)
    if (!l.finished()) return false;
  return true;
}

// The units `units` of a container (codes, uoff: its sections), levelled one behind the other into out by up to n_threads threads.
// False when one of them cannot be.  (A matrix in which all units are wide - every second row zero, say - is as much work as its
// validation: 8192 x 3072 of that kind 85 ms on one thread and 15 on 8, its validation 15 on 8.)
inline bool level_units(const uint16_t* codes, const uint32_t* uoff, const std::vector<uint32_t>& units, uint32_t n_entries, const uint32_t* word,
                        uint32_t limit, unsigned n_threads, std::unique_ptr<uint16_t[]>& out) {
  std::vector<size_t> at(units.size() + 1, 0);   // where in out, in chunks
  for (size_t i = 0; i < units.size(); ++i) at[i + 1] = at[i] + (uoff[units[i] + 1] - uoff[units[i]]);
  out.reset(new uint16_t[at.back() * kChunkWords]);
  constexpr size_t kTake = 8;   // units a thread takes at a time (half a millisecond)
  std::atomic<size_t> next(0);
  std::atomic<bool> refused(false);
  auto work = [&] {
    for (size_t i0; (i0 = next.fetch_add(kTake)) < units.size();)
      for (size_t i = i0; i < std::min(i0 + kTake, units.size()); ++i) {
        if (refused.load(std::memory_order_relaxed)) return;
        if (!level_unit(codes + (size_t)uoff[units[i]] * kChunkWords, (uint32_t)(at[i + 1] - at[i]), n_entries, word, limit, out.get() + at[i] * kChunkWords))
          refused = true;
      }
  };
  {
    Threads th;
    const size_t more = std::min<size_t>({n_threads, 16, (units.size() + kTake - 1) / kTake});
    for (size_t t = 1; t < more; ++t) th.start(work);   // (2 to 8 units, as most matrices have at the start of a dictionary: this thread alone)
    work();
  }
  return !refused;
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
