// Index arithmetic that the kernels and their launches rest on and that needs no GPU: host and device code share it, and
// the host tests run it over its whole range.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "tq_format.h"

#if defined(__HIPCC__)
#define TQ_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define TQ_HD inline
#endif

namespace tq {

// Where part k of `parts` begins on a line of `total` points, floor(total * k / parts), from share = total / parts, rest = total % parts
// and parts_inverse = 1.f / parts: the host divides (a 64-bit division is a hundred instructions, and two of them stood ahead of the first load
// of a wavefront).  Exact for parts and k up to kMaxParts: rest * k + .5 is a whole float and a half, and lies at least half a part's
// share from the next whole number of parts.
constexpr uint32_t kMaxParts = 1024;
TQ_HD uint32_t even_part(uint32_t share, uint32_t rest, float parts_inverse, uint32_t k) {
  return share * k + (uint32_t)(((float)(rest * k) + .5f) * parts_inverse);
}

// `bands` of them for every one of w workgroups, and one more for the first `rest`: the first band of workgroup k.
TQ_HD uint32_t workgroup_band(uint32_t bands, uint32_t rest, uint32_t k) { return bands * k + (k < rest ? k : rest); }

// len / parts for the few parts that a unit's chunks are cut into: units of 256 columns are 33 to 36 chunks long, in pieces of 6 to 12.
TQ_HD uint32_t piece_length(uint32_t len, uint32_t parts) {
  if (len >= 1u << 15) return len / parts;
  switch (parts) {
    case 1: return len;
    case 2: return len >> 1;
    case 3: return len * 43691u >> 17;
    case 4: return len >> 2;
    case 5: return len * 52429u >> 18;
    default: return len / parts;
  }
}

// A launch (or stage) whose matrices have whole workgroups keeps in one word per matrix where its workgroups start on the line of all of
// them, and how many bands each of them has at least.
constexpr int kLineBits = 18;   // a staged step's line: one workgroup per compute unit and stage, up to 896 * 256
constexpr uint32_t kLineMask = (1u << kLineBits) - 1;
constexpr uint32_t kMaxWorkgroupBands = 1u << (32 - kLineBits);
TQ_HD uint32_t line_word(uint32_t start, uint32_t bands) { return bands << kLineBits | start; }

// Stages whose workgroups take equal numbers of units, not of whole bands: two of them may share a band, and both add their part of its sums
// to outputs that were cleared in the stage before (two addends onto zero: the same sum in either order).  The word says so in its top bit.
constexpr uint32_t kBySharedBands = 2, kShareUnits = 1u << 31;
constexpr uint32_t kMaxSharedItems = kMaxWorkgroupBands / 2;
// Workgroup `at` of the line, between the words of its matrix and of the next one: units [lo, hi) of the matrix.
TQ_HD void shared_share(uint32_t word, uint32_t next_word, uint32_t n_bands, uint32_t n_quads, uint32_t at, uint32_t& lo, uint32_t& hi) {
  const uint32_t first = word & kLineMask, wgs = (next_word & kLineMask) - first, items = (word & ~kShareUnits) >> kLineBits;
  const uint32_t size = word & kShareUnits ? 1u : n_quads, total = word & kShareUnits ? n_bands * n_quads : n_bands;
  lo = size * workgroup_band(items, total - items * wgs, at - first);
  hi = size * workgroup_band(items, total - items * wgs, at - first + 1);
}
// Whether no band of a matrix is cut twice when `wgs` workgroups take equal numbers of its units, and each has some.
inline bool bands_cut_once(uint32_t n_bands, uint32_t n_quads, uint32_t wgs) {
  const uint64_t units = (uint64_t)n_bands * n_quads;
  if (units > UINT32_MAX || units < wgs) return false;
  const uint32_t items = (uint32_t)units / wgs, rest = (uint32_t)units % wgs;
  uint32_t last = 0;   // the band cut last, plus 1
  for (uint32_t k = 1; k < wgs; ++k) {
    const uint32_t at = workgroup_band(items, rest, k);
    if (at % n_quads == 0) continue;
    if (at / n_quads + 1 == last) return false;
    last = at / n_quads + 1;
  }
  return true;
}

// What a block of a listing stream writes: `tokens` tokens start in it, `base` start before it, token t stands for the values
// [4 t, 4 t + 4) of n_values (the last one of the stream possibly for fewer).  The block's tokens sit in LDS from dword
// base % 4 on, so that its output lies there as it lies in memory relative to 16-byte pieces.
// No token may start in the block: the last block holds nothing but raw values when the stream's last marker is among the
// last words of the block before.  Its `base` then counts that marker's token too, and 4 * base lies past n_values.
struct ListingOutput {
  uint64_t piece0;   // byte of the output that belongs to byte 0 of the LDS area
  uint32_t lo, hi;   // bytes of the LDS area that are output (lo == hi: none)
};
TQ_HD ListingOutput listing_output(uint32_t base, uint32_t tokens, uint64_t n_values) {
  const uint32_t lo = (base & 3u) * 4u;
  const uint64_t first = (uint64_t)base * 4u, end = first + (uint64_t)tokens * 4u, stop = end < n_values ? end : n_values;
  const uint32_t hi = lo + (uint32_t)(stop - first);   // (a token that starts in the block stands for at least one value: first < stop)
  return {first - lo, lo, tokens ? hi : lo};
}

// The schedule of the ring kernels.  A lane keeps the last kRingBytes of its segment; every kRingStep chunks the wavefront looks
// whether all unfinished lanes have passed the next kRingGroup windows of 8 columns, and multiplies them if so.  (These are
// k_matvec_runs' large rings; the small ones, further down, are its other size and k_matvec_ring's only one.)
constexpr int kRingBytes = 128;
constexpr int kRingPiece = 12;    // chunks per piece of the code stream (two register sets)
constexpr int kRingStep = 4;      // chunks between two looks at the lanes' progress
constexpr int kRingGroup = 4;     // MFMA steps per group
static_assert(kRingPiece % kRingStep == 0 && kRingGroup == 4 && kRingStep <= kRingGroup, "ring schedule");
// How far apart two unfinished lanes may be.  With `done` columns multiplied, a lane at column p may store into the 8-byte
// piece of p only if that piece's place holds columns below done: p - p % 8 <= done + kRingBytes - 8.
//  - After a look the slowest unfinished lane is less than a group past done: between two looks it gains at most a group
//    (8 columns a chunk), and a look takes a group that is ready.
//  - A lane stores where it stands before a chunk.  Before the last of the chunks between two looks it has gained 8 columns
//    in each of the others and stands at most at done + (8 group - 1) + spread + 8 (step - 1): the limits below make
//    that done + kRingBytes - 8.
//  - A lane that completes its segment goes on with pad codes, on the device code 0: a column a code, 4 in a chunk, no faster
//    than an unfinished lane, and the host counts it among the lanes that may be `spread` ahead.  In k_matvec_ring it really
//    moves on; in k_matvec_runs it stays at the segment's end and goes on storing there: from the next look on it is at most
//    (8 group - 1) + spread + 4 past done, which is no further piece, and until then the bound above holds.
//  - When the last lane has finished, less than two groups are left, and none or one after the look that follows.
//  - At a look, after the last chunk, a lane can stand at done + kRingBytes: at a piece's start, and that piece's place
//    still holds columns the look is about to multiply.  Nothing of the lane lies in that piece yet: see ring_leftover.
constexpr uint32_t ring_spread(int bytes, int step, int group) { return bytes - 8 * step - 8 * group + 1; }
constexpr uint32_t kRingSpread = ring_spread(kRingBytes, kRingStep, kRingGroup);
// The small form: half the ring, looks twice as often at half the windows.  Pieces of 9 chunks: a unit of 33..36 chunks, or of
// 17 (packed), is cut into pieces of 8 and 9, and 18 of them in registers leave room for 16 wavefronts.
constexpr int kSmallRingBytes = 64, kSmallRingStep = 2, kSmallRingGroup = 2, kSmallRingPiece = 9;
constexpr uint32_t kSmallRingSpread = ring_spread(kSmallRingBytes, kSmallRingStep, kSmallRingGroup);
static_assert(kSmallRingStep <= kSmallRingGroup, "ring schedule");
constexpr int ring_step(int bytes) { return bytes == kSmallRingBytes ? kSmallRingStep : kRingStep; }
constexpr int ring_group(int bytes) { return bytes == kSmallRingBytes ? kSmallRingGroup : kRingGroup; }
constexpr int ring_piece(int bytes) { return bytes == kSmallRingBytes ? kSmallRingPiece : kRingPiece; }
// Whether a lane that stands at column pos holds bytes of a piece it has not stored (see append_chunk_ring): a unit whose
// segments end inside pieces stores those at every look - those only, never the piece that begins at pos.
TQ_HD bool ring_leftover(uint32_t pos) { return (pos & 7u) != 0; }

// Marks: where every lane of a unit stands at each kMarkChunks-th chunk of it (the pairs it has passed; its columns are those and a column
// a code), so that a wavefront can start inside a unit.  A mark is 64 values, one per lane, of a byte where segments are narrow enough.  A unit
// whose first chunk is c keeps that of its chunk k * kMarkChunks, k >= 1, at mark_index(c) + k: units of any lengths never meet there, since its last one is
// at most the quotient of the chunk behind it, and the next unit's first one lies above that.  (So marks are a 64th of the codes, or a 32nd, however
// short the units are; with a place for k = 0 as well segments of 16 columns had 8 % of them.)
constexpr uint32_t kMarkChunks = 8, kMarkByteCols = 510;   // (pairs of a lane: at most half the columns of its segment)
constexpr uint32_t kMarkAlign = 256;
TQ_HD uint64_t mark_index(uint32_t first_chunk) { return first_chunk / kMarkChunks; }
TQ_HD uint32_t mark_bytes(uint32_t seg_cols) { return seg_cols <= kMarkByteCols ? 64 : 128; }
// The marks lie behind the n_units + 1 unit offsets, at this many bytes from them.
TQ_HD uint64_t marks_at(uint64_t n_units) { return ((n_units + 1) * 4 + kMarkAlign - 1) / kMarkAlign * kMarkAlign; }
inline uint64_t marks_size(uint64_t n_chunks, uint32_t seg_cols) { return (n_chunks / kMarkChunks + 1) * mark_bytes(seg_cols); }

// Whole workgroups for the matrices of a launch (or of a stage): wgs[i] of them for matrix i, `grid` at most together, such
// that the largest share (bands x columns) is as small as possible, to within an eighth of the widest row, and the others' too
// as far as there are workgroups.  Returns the largest share, or 0 when there are more matrices than workgroups (or a matrix is too tall for the kernels' cut).
struct BandCount {
  uint32_t n_bands, cols;   // of a matrix, both at least 1
};
constexpr uint32_t kTallMatrix = 1u << 23;   // bands; (2^14 of them for every workgroup of 256 are more than line_word holds anyway)
inline uint64_t assign_workgroups(int n, const BandCount* m, uint64_t grid, uint32_t* wgs) {
  if ((uint64_t)n > grid) return 0;
  uint64_t total = 0, cols_max = 0;
  for (int i = 0; i < n; ++i) {
    if (m[i].n_bands >= kTallMatrix) return 0;
    total += (uint64_t)m[i].n_bands * m[i].cols;
    cols_max = std::max<uint64_t>(cols_max, m[i].cols);
  }
  auto needed = [&](uint64_t share) {   // workgroups when none takes more than `share`, or a single band
    uint64_t sum = 0;
    for (int i = 0; i < n; ++i) {
      const uint64_t per = std::max<uint64_t>(1, share / m[i].cols);
      sum += (m[i].n_bands + per - 1) / per;
    }
    return sum;
  };
  // Shares of a wide matrix are a band at least; where workgroups are left then, the shares of the narrower ones shrink further (16
  // bands of 7424 columns beside 800 of 256: 44 workgroups of up to 29 bands would meet the largest share, 256 cut the 800 into 3 or 4).
  const uint64_t even = (total + grid - 1) / grid;
  uint64_t lo = even, hi = std::max(cols_max, even);
  while (needed(hi) > grid) lo = hi, hi *= 2;
  if (needed(lo) <= grid) hi = lo;
  // needed(lo) > grid >= needed(hi), and so it stays; hi - lo >= 2 inside the loop, so that it shrinks every time
  while (hi - lo > std::max<uint64_t>(1, hi > cols_max ? cols_max / 8 : hi / 16)) {   // (an eighth of a row below 8 columns is nothing)
    const uint64_t mid = lo + (hi - lo) / 2;
    (needed(mid) <= grid ? hi : lo) = mid;
  }
  uint64_t worst = 0;
  for (int i = 0; i < n; ++i) {
    const uint64_t bands = m[i].n_bands, per = std::max<uint64_t>(1, hi / m[i].cols);
    wgs[i] = (uint32_t)((bands + per - 1) / per);
    worst = std::max(worst, (bands + wgs[i] - 1) / wgs[i] * m[i].cols);
  }
  return worst;
}

// What a band of `cols` columns costs k_matvec_runs, in columns: a unit takes a wavefront as long as its widest segment is, whether it
// has one panel or four.  (Seven matrices, among them 2432 x 64 and 8192 x 1024, batch 9: 65 us cut by columns, 30 like this.)
inline uint32_t unit_columns(uint32_t cols, uint32_t seg_cols) {
  const uint32_t quad = kUnitPanels * seg_cols, whole = (cols - 1) / quad * quad;
  return whole + kUnitPanels * std::min(seg_cols, cols - whole);
}

// What the busiest workgroup does when the line is cut into `grid` equal parts instead: its part to within half a band,
// and, with several matrices, a second start (offsets, activations, barriers) in workgroups that get the end of one
// matrix and the start of the next, worth about kRestartCost of the line (4 us, in which a compute unit streams 100 KB of
// codes: one LLaMA-3.2-1B layer, 7 matrices, 24.9 us when 6 of the 256 workgroups start twice, 18.4 us in whole workgroups).
constexpr uint64_t kRestartCost = 6000;
constexpr int kMaxAssign = 32;   // most matrices that are given whole workgroups
inline uint64_t even_cut_cost(int n, const BandCount* m, uint64_t grid) {
  uint64_t total = 0, cols_max = 0;
  for (int i = 0; i < n; ++i) {
    total += (uint64_t)m[i].n_bands * m[i].cols;
    cols_max = std::max<uint64_t>(cols_max, m[i].cols);
  }
  return total / grid + cols_max / 2 + (n > 1 ? kRestartCost : 0);
}
// Whether a launch of n <= kMaxAssign matrices is cut in whole workgroups, wgs[i] of `most` at most for matrix i, or into `grid` parts.
inline bool cut_in_workgroups(int n, const BandCount* m, uint64_t most, uint64_t grid, uint32_t* wgs) {
  const uint64_t worst = assign_workgroups(n, m, most, wgs);
  return worst && worst <= even_cut_cost(n, m, grid);
}

// How a staged step that is one launch of `grid` workgroups cuts its stages.
struct StageItem {   // a product of it: its matrix, where its activations and its outputs lie
  uint32_t n_bands, n_quads, cols;
  uint64_t x, x_end, y, y_end;
};
// Whether the outputs of the products [f, end) of a stage can be cleared while the stage before, products [before, f), is in work, and added
// to in their own: addable(i) says that of the memory, and they are in no one's place but their own among both stages' activations and outputs.
template <typename Addable>
bool outputs_can_be_added_to(const StageItem* m, int before, int f, int end, Addable&& addable) {
  for (int i = f; i < end; ++i) {
    if (!addable(i)) return false;
    for (int j = before; j < end; ++j) {
      const bool x_apart = m[i].y_end <= m[j].x || m[j].x_end <= m[i].y, y_apart = m[i].y_end <= m[j].y || m[j].y_end <= m[i].y;
      if (!x_apart || (j != i && !y_apart)) return false;
    }
  }
  return true;
}
// Whole workgroups per matrix in every stage, if that is the better cut over all stages.  In equal numbers of units where may_share, that takes a
// sixteenth off the stage's largest share, its outputs can be added to, and every workgroup has work in the stage before (it clears what is
// added to).  first: the first product of every stage, and n.  words: of the line (line_word, shared_share), empty where the cost line in
// weights is cut evenly.
struct StageLine {
  bool shared = false;
  std::vector<uint32_t> words;
};
template <typename Addable>
StageLine plan_stages(int n, const StageItem* m, const uint32_t* first, uint32_t n_stages, uint32_t grid, bool may_share, Addable&& addable) {
  StageLine plan;
  std::vector<uint32_t> line((size_t)n + 1, 0);
  std::vector<uint8_t> by_units((size_t)n, 0);
  uint64_t whole = 0, even = 0;
  bool all_busy = false, wide_words = false;
  if ((uint64_t)n_stages * grid > kLineMask) return plan;
  for (uint32_t k = 0; k < n_stages; ++k) {
    const int f = (int)first[k], cnt = (int)(first[k + 1] - first[k]);
    if (cnt > kMaxAssign) return plan;
    BandCount bands[kMaxAssign], units[kMaxAssign];
    uint32_t wgs[kMaxAssign], unit_wgs[kMaxAssign];
    bool few = true;
    for (int i = 0; i < cnt; ++i) {
      const StageItem& t = m[f + i];
      bands[i] = {t.n_bands, t.cols};
      units[i] = {t.n_bands * t.n_quads, std::max(1u, t.cols / t.n_quads)};
      few = few && (uint64_t)t.n_bands * t.n_quads < kTallMatrix;
    }
    uint64_t largest = assign_workgroups(cnt, bands, grid, wgs);
    if (!largest) return plan;
    if (k && all_busy && may_share && few) {
      const uint64_t unit_largest = assign_workgroups(cnt, units, grid, unit_wgs);
      bool fits = unit_largest && unit_largest * 17 < largest * 16;
      for (int i = 0, left = (int)grid; i < cnt && fits; ++i) {
        const uint32_t take = i + 1 < cnt ? unit_wgs[i] : (uint32_t)left;   // (those left over are the last matrix's)
        left -= (int)unit_wgs[i];
        fits = bands_cut_once(m[f + i].n_bands, m[f + i].n_quads, take) && units[i].n_bands / take < kMaxSharedItems;
      }
      if (fits && outputs_can_be_added_to(m, (int)first[k - 1], f, f + cnt, addable)) {
        std::copy(unit_wgs, unit_wgs + cnt, wgs);
        std::fill(by_units.begin() + f, by_units.begin() + f + cnt, 1);
        largest = unit_largest;
        plan.shared = true;
      }
    }
    all_busy = true;
    uint32_t at = k * grid;
    for (int i = 0, left = (int)grid; i < cnt; ++i) {
      const uint32_t take = i + 1 < cnt ? wgs[i] : (uint32_t)left, items = by_units[f + i] ? units[i].n_bands : bands[i].n_bands;
      left -= (int)wgs[i];
      all_busy = all_busy && items >= take;
      if (items / wgs[i] >= kMaxWorkgroupBands) return StageLine();
      wide_words = wide_words || items / wgs[i] >= kMaxSharedItems;
      line[f + i] = at;
      at += wgs[i];
    }
    whole += largest;
    even += even_cut_cost(cnt, bands, grid);
  }
  line[n] = n_stages * grid;   // (workgroups left over in a stage count as its last matrix's)
  if (whole > even || (plan.shared && wide_words)) return StageLine();
  plan.words.resize((size_t)n + 1);
  for (int i = 0; i < n; ++i)
    plan.words[i] = line_word(line[i], m[i].n_bands * (by_units[i] ? m[i].n_quads : 1u) / (line[i + 1] - line[i])) | (by_units[i] ? kShareUnits : 0u);
  plan.words[n] = line[n];
  return plan;
}

}  // namespace tq
