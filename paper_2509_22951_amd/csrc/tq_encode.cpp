// Host-side encoder of libtq (off the hot path): per-row int8 quantization (paper section 3, 8-bit setting),
// segmentation of the rows, and LZW with a size-capped, frozen dictionary (paper Background "Compression"),
// laid out as interleaved lane streams per unit of 16 rows x 4 segments.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include <sys/mman.h>

#include "../../include/tq.h"
#include "tq_format.h"

namespace tq {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;

unsigned pick_threads(uint32_t asked) {
  unsigned hw = std::thread::hardware_concurrency();
  if (hw == 0) hw = 1;
  unsigned n = asked ? asked : hw;
  return std::max(1u, std::min(n, 16u));
}

// The threads of one call, started once: the caller is number 0, the others wait between the phases of its work, first for a few
// microseconds by looking, then asleep.  (Started anew for each of three phases, 16 threads cost 0.6 of the 2.1 ms that a 2048 x 2048 matrix
// takes.)  Where one cannot be started the constructor throws, and those that run are waited for.
class Crew {
 public:
  explicit Crew(unsigned n) : n_(std::max(1u, n)) {
    try {
      for (unsigned t = 1; t < n_; ++t) threads_.start([this, t] { work(t); });
    } catch (...) {
      finish();
      throw;
    }
  }
  ~Crew() { finish(); }
  unsigned size() const { return n_; }
  // body(t) on every thread but the caller's, which goes on; until wait() has returned, body and what it refers to stay as they are.
  void start(std::function<void(unsigned)> body) {
    body_ = std::move(body);
    left_.store(n_ - 1, std::memory_order_relaxed);
    {
      std::lock_guard<std::mutex> lock(mutex_);
      phase_.fetch_add(1, std::memory_order_release);
    }
    wake_.notify_all();
  }
  void wait() {
    for (unsigned looks = 0; left_.load(std::memory_order_acquire); ++looks)
      if (looks > kLooks) std::this_thread::yield();
  }
  // body(t) on every thread, the caller's among them
  void run(const std::function<void(unsigned)>& body) {
    start(body);
    const Waits all(*this);
    body(0);
  }
  // Waits for the others where its block ends, whatever way that is left.
  class Waits {
   public:
    explicit Waits(Crew& crew) : crew_(crew) {}
    ~Waits() { crew_.wait(); }

   private:
    Crew& crew_;
  };

 private:
  static constexpr unsigned kLooks = 4000;
  void work(unsigned t) {
    for (unsigned seen = 0;;) {
      for (unsigned looks = 0; looks < kLooks && phase_.load(std::memory_order_acquire) == seen; ++looks) {}
      if (phase_.load(std::memory_order_acquire) == seen) {
        std::unique_lock<std::mutex> lock(mutex_);
        wake_.wait(lock, [&] { return phase_.load(std::memory_order_acquire) != seen; });
      }
      ++seen;
      if (stop_.load(std::memory_order_relaxed)) return;
      body_(t);
      left_.fetch_sub(1, std::memory_order_release);
    }
  }
  void finish() {
    stop_.store(true, std::memory_order_relaxed);
    {
      std::lock_guard<std::mutex> lock(mutex_);
      phase_.fetch_add(1, std::memory_order_release);
    }
    wake_.notify_all();
    threads_.join();
  }
  const unsigned n_;
  std::function<void(unsigned)> body_;
  std::atomic<unsigned> phase_{0}, left_{0};
  std::atomic<bool> stop_{false};
  std::mutex mutex_;
  std::condition_variable wake_;
  Threads threads_;   // (last: the others are there before the first thread looks at them)
};

// Dictionary of runs of up to 4 bytes, in the order LZW creates them (the container's code space is that order sorted by
// run length: final_codes()).  Codes 0..255 are the single bytes; a two-byte run is found through a direct table over
// the byte pair, a longer one through a hash table over (code of the run it extends, next byte).
class RunDict {
 public:
  RunDict(uint32_t max_entries, uint32_t lmax, uint32_t unit_budget)
      : max_(max_entries), lmax_(lmax), budget_(unit_budget), units_(256), pair_(65536, kNone) {
    bytes_.reserve(max_entries + 1);
    len_.reserve(max_entries + 1);
    for (uint32_t b = 0; b < 256; ++b) {
      bytes_.push_back(b);
      len_.push_back(1);
    }
    if (lmax > 2) {
      mask_ = 1u << 17;
      while (mask_ < 4u * max_entries) mask_ <<= 1;
      key_.assign(mask_, kNone);
      val_.assign(mask_, 0);
      --mask_;
    }
  }
  uint32_t size() const { return (uint32_t)bytes_.size(); }
  uint32_t length(uint32_t code) const { return len_[code]; }
  uint32_t word(uint32_t code) const { return bytes_[code]; }
  // no further entry can be added (count reached, or not even a two-byte run fits the unit budget)
  bool full() const { return size() >= max_ || lmax_ < 2 || (budget_ && units_ + 1 > budget_); }

  // The run (entry `parent` + byte b) as a new entry; false when it exists, is too long or does not fit.
  bool add(uint32_t parent, uint32_t b) {
    const uint32_t len = len_[parent] + 1, cost = len <= 2 ? 1u : 2u;
    if (len > lmax_ || size() >= max_ || (budget_ && units_ + cost > budget_) || child(parent, b) != kNone) return false;
    const uint32_t code = size();
    if (len == 2) {
      pair_[parent << 8 | b] = code;
    } else {
      uint32_t h = hash(parent << 8 | b);
      while (key_[h] != kNone) h = (h + 1) & mask_;
      key_[h] = parent << 8 | b;
      val_[h] = code;
    }
    bytes_.push_back(bytes_[parent] | b << (8 * len_[parent]));
    len_.push_back((uint8_t)len);
    units_ += cost;
    return true;
  }
  uint32_t child(uint32_t parent, uint32_t b) const {
    if (parent < 256) return pair_[parent << 8 | b];
    if (lmax_ <= 2) return kNone;
    const uint32_t k = parent << 8 | b;
    for (uint32_t h = hash(k); key_[h] != kNone; h = (h + 1) & mask_)
      if (key_[h] == k) return val_[h];
    return kNone;
  }
  // Continue from the dictionary section of another container: its entries from 256 on, which come sorted by length,
  // so each follows the run it extends.  lens[e] = length of entry e.
  bool adopt(const uint32_t* words, const std::vector<uint8_t>& lens, uint32_t n) {
    for (uint32_t e = 256; e < n; ++e) {
      const uint32_t w = words[e], len = lens[e];
      if (len < 2 || len > lmax_) return false;
      uint32_t parent = w & 0xFFu;
      for (uint32_t k = 1; k + 1 < len && parent != kNone; ++k) parent = child(parent, w >> (8 * k) & 0xFFu);
      if (parent == kNone || !add(parent, w >> (8 * (len - 1)) & 0xFFu)) return false;
    }
    return true;
  }

  // Greedy parse of S[gs, ge): longest entry at each position, never crossing ge.  While `kGrow`, the matched run plus
  // the following byte becomes a new entry if it fits.  Codes are written in creation order.
  template <bool kGrow>
  void parse(const uint8_t* S, uint64_t gs, uint64_t ge, std::vector<uint16_t>& out) {
    uint64_t i = gs;
    if (lmax_ <= 2) {   // the common case: one table lookup per position
      while (i < ge) {
        uint32_t code = S[i], m = 1;
        if (lmax_ == 2 && i + 1 < ge) {
          const uint32_t pc = pair_[(uint32_t)S[i] << 8 | S[i + 1]];
          if (pc != kNone) {
            code = pc;
            m = 2;
          }
        }
        out.push_back((uint16_t)code);
        if (kGrow && m < lmax_ && i + m < ge) add(code, S[i + 1]);   // m == 1 here: the new entry is a pair
        i += m;
      }
      return;
    }
    while (i < ge) {
      uint32_t code = S[i], m = 1;
      while (m < lmax_ && i + m < ge) {
        const uint32_t c = child(code, S[i + m]);
        if (c == kNone) break;
        code = c;
        ++m;
      }
      out.push_back((uint16_t)code);
      if (kGrow && m < lmax_ && i + m < ge) add(code, S[i + m]);
      i += m;
    }
  }

  // The two-byte runs by their bytes as they lie in memory (first byte low): their code, or kNoPair.
  static constexpr uint16_t kNoPair = 0xFFFF;
  std::vector<uint16_t> pair_table() const {
    std::vector<uint16_t> t(65536, kNoPair);
    for (uint32_t e = 256; e < size(); ++e)
      if (len_[e] == 2) t[bytes_[e]] = (uint16_t)e;
    return t;
  }

  // parse<true> for runs of at most 2 (lmax 2), with `pairs` kept as pair_table() would give it (pair_, which only longer runs and an
  // inherited dictionary are looked up in, is left as it is).
  uint32_t parse_growing_pairs(const uint8_t* p, uint32_t len, uint16_t* pairs, uint16_t* out) {
    uint32_t i = 0, n = 0;
    while (i + 1 < len) {
      uint16_t key;
      std::memcpy(&key, p + i, 2);
      const uint16_t c = pairs[key];
      if (c != kNoPair) {
        out[n++] = c;
        i += 2;
        continue;
      }
      out[n++] = p[i];
      if (size() < max_) {
        pairs[key] = (uint16_t)size();
        bytes_.push_back(key);
        len_.push_back(2);
      }
      ++i;
    }
    if (i < len) out[n++] = p[i];
    return n;
  }

  // The container's numbering: entries in order of run length, equal lengths in order of creation.
  // final_of[creation code] = container code; class_end[k] = entries of at most k + 1 bytes.
  void final_codes(std::vector<uint16_t>* final_of, std::vector<uint32_t>* words, uint32_t class_end[4]) const {
    const uint32_t n = size();
    uint32_t count[5] = {0, 0, 0, 0, 0};
    for (uint32_t e = 0; e < n; ++e) ++count[len_[e]];
    uint32_t next[5] = {0, 0, count[1], count[1] + count[2], count[1] + count[2] + count[3]};
    for (int k = 0; k < 4; ++k) class_end[k] = next[k + 1] + count[k + 1];
    final_of->assign(n + 1, 0);
    words->assign(n, 0);
    for (uint32_t e = 0; e < n; ++e) {
      const uint32_t f = next[len_[e]]++;
      (*final_of)[e] = (uint16_t)f;
      (*words)[f] = bytes_[e];
    }
    (*final_of)[n] = (uint16_t)n;   // the pad code
  }

 private:
  uint32_t hash(uint32_t k) const { return (k * 2654435761u) >> 7 & mask_; }
  uint32_t max_, lmax_, budget_, units_, mask_ = 0;
  std::vector<uint32_t> pair_, bytes_, key_, val_;
  std::vector<uint8_t> len_;
};

// (packed values: the same number of weights per segment by default)
uint32_t segment_width(const tq_encode_opts* o) {
  return o && o->seg_cols ? o->seg_cols : o && o->packing == TQ_PACK_NIBBLES ? TQ_DEFAULT_SEG_COLS / 2 : TQ_DEFAULT_SEG_COLS;
}

int check_opts(const tq_encode_opts* o, uint32_t* max_entries, uint32_t* lmax, uint32_t* seg_cols, unsigned* n_threads) {
  *max_entries = (o && o->max_entries) ? o->max_entries : TQ_MAX_ENTRIES_DEVICE;
  *lmax = (o && o->lmax) ? o->lmax : TQ_DEFAULT_LMAX;
  *seg_cols = segment_width(o);
  *n_threads = pick_threads(o ? o->n_threads : 0);
  if (*lmax < 1 || *lmax > TQ_MAX_LMAX) {
    set_error("tq_encode: lmax must be 0 (default) or in [1, " + std::to_string(TQ_MAX_LMAX) + "]");
    return TQ_E_INVALID_ARG;
  }
  if (*max_entries < 256 || *max_entries > TQ_MAX_ENTRIES_DEVICE) {
    set_error("tq_encode: max_entries must be 0 or in [256, " + std::to_string(TQ_MAX_ENTRIES_DEVICE) + "]");
    return TQ_E_INVALID_ARG;
  }
  if (*seg_cols < kMinSegCols || *seg_cols > kMaxSegCols || *seg_cols % 16) {
    set_error("tq_encode: seg_cols must be a multiple of 16 in [16, 1024]");
    return TQ_E_INVALID_ARG;
  }
  if (o && (o->dict_from != nullptr) != (o->dict_from_bytes != 0)) {
    set_error("tq_encode: dict_from and dict_from_bytes must be given together");
    return TQ_E_INVALID_ARG;
  }
  if (o && o->dictionary != TQ_DICT_LZW && o->dictionary != TQ_DICT_FREQUENCY) {
    set_error("tq_encode: dictionary must be TQ_DICT_LZW or TQ_DICT_FREQUENCY");
    return TQ_E_INVALID_ARG;
  }
  if (o && o->dictionary == TQ_DICT_FREQUENCY && *lmax > 2) {
    set_error("tq_encode: TQ_DICT_FREQUENCY picks runs of 2 bytes; use lmax 1 or 2 with it");
    return TQ_E_INVALID_ARG;
  }
  if (o && o->bits != 0 && (o->bits < 2 || o->bits > 8)) {
    set_error("tq_encode: bits must be 0 (= 8) or in [2, 8]");
    return TQ_E_INVALID_ARG;
  }
  if (o && o->packing > TQ_PACK_NIBBLES) {
    set_error("tq_encode: packing must be TQ_PACK_NONE or TQ_PACK_NIBBLES");
    return TQ_E_INVALID_ARG;
  }
  return TQ_OK;
}

// Codes of a contiguous range of units as they come out of a parse that grows the dictionary, concatenated in (unit, lane)
// order; cnt[u * 64 + lane] codes each.
struct UnitRange {
  std::vector<uint16_t> codes;
  std::vector<uint16_t> cnt;
};

// Room that all threads write for the first time at once: in large pages, each the size of 512 ordinary ones, whose faults queue behind each
// other.  Below two of them from the ordinary heap.
struct Free {
  void operator()(void* p) const { std::free(p); }
};
constexpr size_t kLargePage = 2u << 20;
std::unique_ptr<void, Free> large_room(size_t bytes) {
  const size_t whole = (size_t)round_up(bytes, kLargePage);
  std::unique_ptr<void, Free> p(bytes < 2 * kLargePage ? std::malloc(std::max<size_t>(bytes, 1)) : std::aligned_alloc(kLargePage, whole));
  if (!p) throw std::bad_alloc();
  if (bytes >= 2 * kLargePage) (void)madvise(p.get(), whole, MADV_HUGEPAGE);   // (a wish: without it the pages are ordinary ones)
  return p;
}

// Room for the codes of all units while their number is not known: for as many as there are bytes.  In large pages (2048 x 2048: 1.75 -> 1.25 ms) up to
// 64 MB; beyond that in ordinary ones, of which those that are not written cost nothing.
class CodeRoom {
 public:
  explicit CodeRoom(size_t words) {
    const size_t bytes = std::max<size_t>(words * 2, 2);
    if (bytes <= kMost) p_ = large_room(bytes);
    else p_.reset(std::malloc(bytes));
    if (!p_) throw std::bad_alloc();
    next_ = (uint16_t*)p_.get();
  }
  uint16_t* take(size_t words) {
    uint16_t* p = next_;
    next_ += words;
    return p;
  }

 private:
  static constexpr size_t kMost = 64u << 20;
  std::unique_ptr<void, Free> p_;
  uint16_t* next_ = nullptr;
};

// The code section of a contiguous range of units, in the container's layout (the offsets follow when all ranges are known).
struct CodedRange {
  uint64_t u_begin = 0, u_end = 0, n_real = 0;
  uint16_t* words = nullptr;
  size_t used = 0;                     // words
  std::vector<uint32_t> chunks;        // per unit
  // Words that n_units may need.  longest: of the segments' lengths (a matrix narrower than its segments would otherwise ask for many
  // times its size)
  static size_t most_words(uint64_t n_units, uint32_t longest) { return (size_t)n_units * 64 * ((longest + kChunkCodes - 1) / kChunkCodes * kChunkCodes); }
  void start(uint64_t begin, uint64_t end, uint32_t longest, CodeRoom& room) {
    u_begin = begin;
    u_end = end;
    words = room.take(most_words(end - begin, longest));
    chunks.reserve(end - begin);
  }
  // lane l's codes at lanes + l * kMaxSegCols (room to pad them to whole chunks of the longest)
  void add_unit(uint16_t* lanes, const uint32_t (&cnt)[64], uint16_t pad) {
    uint32_t mx = 0;
    for (uint32_t l = 0; l < 64; ++l) {
      mx = std::max(mx, cnt[l]);
      n_real += cnt[l];
    }
    const uint32_t n = (mx + kChunkCodes - 1) / kChunkCodes;
    uint16_t* to = words + used;
    for (uint32_t l = 0; l < 64; ++l) {
      uint16_t* src = lanes + (size_t)l * kMaxSegCols;
      std::fill(src + cnt[l], src + n * kChunkCodes, pad);
      for (uint32_t c = 0; c < n; ++c) std::memcpy(to + (size_t)c * kChunkWords + l * kChunkCodes, src + c * kChunkCodes, kChunkCodes * 2);
    }
    used += (size_t)n * kChunkWords;
    chunks.push_back(n);
  }
};
static_assert(kMaxSegCols % kChunkCodes == 0, "a padded lane stream fits kMaxSegCols codes");

// Longest match over single bytes and pairs, p[0 .. len) -> codes; n = their number.  `pairs`: RunDict::pair_table.
inline uint32_t parse_pairs(const uint8_t* p, uint32_t i, uint32_t len, const uint16_t* pairs, uint16_t* out, uint32_t n) {
  while (i + 1 < len) {
    uint16_t key;
    std::memcpy(&key, p + i, 2);
    const uint16_t c = pairs[key];
    const bool pair = c != RunDict::kNoPair;
    out[n++] = pair ? c : p[i];
    i += 1u + pair;
  }
  if (i < len) out[n++] = p[i];
  return n;
}
// Four segments of one length side by side: a step waits for its table entry, the four do so together.
inline void parse_pairs4(const uint8_t* const (&p)[4], uint32_t len, const uint16_t* pairs, uint16_t* const (&out)[4], uint32_t (&n)[4]) {
  uint32_t i[4] = {0, 0, 0, 0};
  n[0] = n[1] = n[2] = n[3] = 0;
  while (std::max(std::max(i[0], i[1]), std::max(i[2], i[3])) + 1 < len) {
    for (int k = 0; k < 4; ++k) {
      uint16_t key;
      std::memcpy(&key, p[k] + i[k], 2);
      const uint16_t c = pairs[key];
      const uint32_t pair = c != RunDict::kNoPair;
      out[k][n[k]++] = pair ? c : (uint16_t)(key & 0xFF);
      i[k] += 1u + pair;
    }
  }
  for (int k = 0; k < 4; ++k) n[k] = parse_pairs(p[k], i[k], len, pairs, out[k], n[k]);
}

// One row: the scale, and the values as bytes.  In IEEE fp32 and in this order: amax = max|w|, s = amax / qmax, q = clamp(rne(w / s),
// -qmax, qmax).  The loops are written for vector instructions: magnitudes compare like their bits, and adding and
// subtracting 1.5 * 2^23 rounds to nearest, ties to even, for values below 2^22 (|w / s| < 2 qmax).
float quantize_row(const float* row, uint32_t cols, float qmax, uint8_t* q) {
  int32_t top = 0;
  for (uint32_t c = 0; c < cols; ++c) {
    int32_t bits;
    std::memcpy(&bits, row + c, 4);
    bits &= 0x7FFFFFFF;
    top = bits > top ? bits : top;
  }
  float amax;
  std::memcpy(&amax, &top, 4);
  if (top > 0x7F800000) {   // a NaN: it counts for nothing
    amax = 0.f;
    for (uint32_t c = 0; c < cols; ++c) amax = std::max(amax, std::fabs(row[c]));
  }
  const float s = amax / qmax;
  if (!(s > 0.f)) {   // all-zero row
    std::memset(q, 0, cols);
    return s;
  }
  for (uint32_t c = 0; c < cols; ++c) {
    float t = row[c] / s;
    t = (t + 12582912.f) - 12582912.f;
    t = std::min(qmax, std::max(-qmax, t));
    q[c] = (uint8_t)(int8_t)(int)t;
  }
  return s;
}

// Two 4-bit values per byte (low nibble: the even column).  false if a value does not fit or the column count is odd.
bool pack_nibbles(const uint8_t* Q, uint32_t rows, uint32_t cols, std::vector<uint8_t>* out) {
  if (cols % 2) {
    set_error("tq_encode: packing needs an even number of columns");
    return false;
  }
  out->assign((size_t)rows * (cols / 2), 0);
  for (size_t i = 0; i < out->size(); ++i) {
    const int a = (int8_t)Q[2 * i], b = (int8_t)Q[2 * i + 1];
    if (a < -8 || a > 7 || b < -8 || b > 7) {
      set_error("tq_encode: packing takes values in [-8, 7]");
      return false;
    }
    (*out)[i] = (uint8_t)((a & 15) | (b & 15) << 4);
  }
  return true;
}

// The bands of the matrix that is coded, where they are made while the dictionary already grows over the first of them: in pieces of whole
// bands, or of single rows where there are too few bands for the threads.
class Bands {
 public:
  // make(first, end): rows of one band, by any thread
  Bands(uint32_t rows, unsigned n_threads, std::function<void(uint32_t, uint32_t)> make)
      : rows_(rows), step_((uint64_t)kUnitRows * 2 * n_threads > rows ? 1u : kUnitRows), n_((rows + step_ - 1) / step_), make_(std::move(make)),
        made_(new std::atomic<bool>[n_]) {
    for (uint32_t k = 0; k < n_; ++k) made_[k].store(false, std::memory_order_relaxed);
  }
  void make_all() {
    while (make_next()) {}
  }
  void wait_for(uint32_t band) {
    const uint32_t first = band * (kUnitRows / step_), end = std::min(n_, first + kUnitRows / step_);
    for (uint32_t k = first; k < end; ++k)
      while (!made_[k].load(std::memory_order_acquire))
        if (!make_next()) std::this_thread::yield();
  }

 private:
  bool make_next() {
    const uint32_t k = next_.fetch_add(1, std::memory_order_relaxed);
    if (k >= n_) return false;
    make_(k * step_, (uint32_t)std::min<uint64_t>(rows_, (uint64_t)(k + 1) * step_));
    made_[k].store(true, std::memory_order_release);
    return true;
  }
  const uint32_t rows_, step_, n_;
  std::function<void(uint32_t, uint32_t)> make_;
  std::unique_ptr<std::atomic<bool>[]> made_;
  std::atomic<uint32_t> next_{0};
};

// The threads of a matrix of rows x cols stored bytes: as many as the caller asks for, but no more than it has units; if it asks for none, one for every
// kThreadBytes, since starting one costs its caller 20 us.  (Bands limit neither phase.  ms on 16 CPUs, no more threads than bands -> now:
// 16 x 262144 4.35 -> 2.5, with a carried dictionary 4.8 -> 1.2; 256 x 256 0.45 -> 0.21, from int8 0.43 -> 0.19.  kThreadBytes of 2^15, 2^16, 2^17: 256 x 2048
// 0.81, 0.61, 0.56; 64 x 8192 0.84, 0.63, 0.56; 1024 x 256 0.76, 0.72, 0.58; 2048 x 512 0.88, 0.85, 0.83.)
constexpr uint64_t kThreadBytes = 1u << 17;
unsigned crew_size(const tq_encode_opts* opts, uint32_t rows, uint32_t cols) {
  const uint64_t unit_cols = (uint64_t)kUnitPanels * std::max(kMinSegCols, segment_width(opts));   // (not checked yet)
  const uint64_t units = (rows + (uint64_t)kUnitRows - 1) / kUnitRows * ((cols + unit_cols - 1) / unit_cols), asked = opts ? opts->n_threads : 0;
  return (unsigned)std::min<uint64_t>(pick_threads((uint32_t)asked), asked ? units : std::max<uint64_t>(1, (uint64_t)rows * cols / kThreadBytes));
}

// Q: the byte matrix rows x cols that is coded (for packing 1 the packed one).  bands: null, or the crew's other threads are making its bands.
int encode_quantized_matrix(const uint8_t* Q, const std::vector<float>& scales_pad, uint32_t rows, uint32_t cols,
                            const tq_encode_opts* opts, Crew& crew, Bands* bands, void** blob_out, size_t* bytes_out) {
  uint32_t max_entries, lmax, seg_cols;
  unsigned n_threads;
  if (int rc = check_opts(opts, &max_entries, &lmax, &seg_cols, &n_threads)) return rc;
  Header h;
  std::memset(&h, 0, sizeof h);
  std::memcpy(h.magic, kMagic, 8);
  h.version = kVersion;
  h.header_bytes = kHeaderBytes;
  h.rows = rows;
  h.cols = cols;
  h.seg_cols = seg_cols;
  h.unit_rows = kUnitRows;
  h.unit_panels = kUnitPanels;
  h.chunk_codes = kChunkCodes;
  h.n_bands = (rows + kUnitRows - 1) / kUnitRows;
  h.n_panels = (cols + seg_cols - 1) / seg_cols;
  h.n_quads = (h.n_panels + kUnitPanels - 1) / kUnitPanels;
  h.n_units = (uint64_t)h.n_bands * h.n_quads;
  h.lmax = lmax;
  h.max_entries = max_entries;
  h.packing = opts ? opts->packing : 0;
  const uint64_t n_units = h.n_units;

  // (runs longer than 2 bytes take two units of the device's dictionary storage each: the unit budget then applies)
  RunDict dict(max_entries, lmax, lmax > 2 ? kUnitBudget : 0u);
  if (opts && opts->dict_from) {
    // One LZW dictionary over a sequence of matrices: start from the entries the earlier container ended with.
    Header fh;
    if (int rc = validate_blob(opts->dict_from, (size_t)opts->dict_from_bytes, &fh, nullptr, nullptr, n_threads)) return rc;
    std::vector<uint8_t> lens(fh.n_entries);
    for (uint32_t e = 0; e < fh.n_entries; ++e) lens[e] = (uint8_t)run_length(fh, e);
    if (fh.lmax > lmax || fh.n_entries > max_entries ||
        !dict.adopt((const uint32_t*)((const uint8_t*)opts->dict_from + fh.off_dict), lens, fh.n_entries)) {
      set_error("tq_encode: the dictionary of dict_from does not fit this lmax / max_entries");
      return TQ_E_INVALID_ARG;
    }
  }
  auto segment_start = [&](uint32_t band, uint32_t quad, uint32_t lane) {
    return (uint64_t)(band * kUnitRows + (lane & 15)) * cols + (uint64_t)(quad * kUnitPanels + (lane >> 4)) * seg_cols;
  };
  auto all_bands = [&] {   // everything is quantized
    if (!bands) return;
    bands->make_all();
    crew.wait();
    bands = nullptr;
  };

  const bool by_frequency = opts && opts->dictionary == TQ_DICT_FREQUENCY;
  if (by_frequency && !(opts && opts->dict_from) && lmax >= 2 && max_entries > 256) {
    all_bands();
    // The most frequent pairs of neighbouring bytes, counted at every offset inside a segment, segments in the order
    // they are parsed in; ties go to the pair seen first.
    std::vector<uint64_t> count(65536, 0), first(65536, 0);
    uint64_t seen = 0;
    for (uint64_t uu = 0; uu < n_units; ++uu) {
      const uint32_t band = (uint32_t)(uu / h.n_quads), quad = (uint32_t)(uu % h.n_quads);
      for (uint32_t lane = 0; lane < 64; ++lane) {
        const uint32_t len = segment_len(h, band, quad, lane);
        if (len < 2) continue;
        const uint8_t* seg = Q + (uint64_t)(band * kUnitRows + (lane & 15)) * cols + (uint64_t)(quad * kUnitPanels + (lane >> 4)) * seg_cols;
        for (uint32_t i = 0; i + 1 < len; ++i) {
          const uint32_t key = (uint32_t)seg[i] << 8 | seg[i + 1];
          if (count[key]++ == 0) first[key] = seen;
          ++seen;
        }
      }
    }
    std::vector<uint32_t> keys;
    for (uint32_t k = 0; k < 65536; ++k)
      if (count[k]) keys.push_back(k);
    std::sort(keys.begin(), keys.end(), [&](uint32_t a, uint32_t b) { return count[a] != count[b] ? count[a] > count[b] : first[a] < first[b]; });
    for (uint32_t k : keys)
      if (!dict.add(k >> 8, k & 0xFF)) break;
  }

  // Phase 1 (sequential): units in order while the dictionary can still grow.
  UnitRange grown;
  std::vector<uint16_t> pairs = lmax <= 2 ? dict.pair_table() : std::vector<uint16_t>();
  uint16_t segment[kMaxSegCols];
  uint64_t u = 0;
  for (; !by_frequency && u < n_units && !dict.full(); ++u) {
    const uint32_t band = (uint32_t)(u / h.n_quads), quad = (uint32_t)(u % h.n_quads);
    if (bands) bands->wait_for(band);
    for (uint32_t lane = 0; lane < 64; ++lane) {
      const size_t before = grown.codes.size();
      if (const uint32_t len = segment_len(h, band, quad, lane)) {
        const uint64_t start = segment_start(band, quad, lane);
        if (lmax == 2) grown.codes.insert(grown.codes.end(), segment, segment + dict.parse_growing_pairs(Q + start, len, pairs.data(), segment));
        else dict.parse<true>(Q, start, start + len, grown.codes);
      }
      grown.cnt.push_back((uint16_t)(grown.codes.size() - before));
    }
  }
  all_bands();
  const uint64_t u_frozen = u;
  const uint32_t n_entries = dict.size();
  const uint16_t pad = (uint16_t)n_entries;
  // The container's code space is sorted by run length; the parse above and below numbers entries as they were created
  // (which is the same while no run is longer than 2).
  std::vector<uint16_t> final_of;
  std::vector<uint32_t> words;
  dict.final_codes(&final_of, &words, h.class_end);

  // Phase 2 (parallel): the dictionary no longer changes, units are independent.
  n_threads = crew.size();
  const uint32_t longest = std::min(seg_cols, cols);
  CodeRoom room(CodedRange::most_words(n_units, longest));
  std::vector<CodedRange> ranges(1 + n_threads);
  {
    auto code_unit = [&](uint64_t uu, uint16_t* lanes, std::vector<uint16_t>& buffer, CodedRange& r) {
      uint32_t cnt[64];
      const uint32_t band = (uint32_t)(uu / h.n_quads), quad = (uint32_t)(uu % h.n_quads);
      for (uint32_t lane = 0; lane < 64; lane += 4) {
        const uint8_t* p[4];
        uint16_t* out[4];
        uint32_t len[4], n[4];
        for (uint32_t k = 0; k < 4; ++k) {
          len[k] = segment_len(h, band, quad, lane + k);
          p[k] = Q + (len[k] ? segment_start(band, quad, lane + k) : 0);
          out[k] = lanes + (size_t)(lane + k) * kMaxSegCols;
        }
        if (lmax <= 2 && len[0] && len[0] == len[1] && len[1] == len[2] && len[2] == len[3]) {
          parse_pairs4(p, len[0], pairs.data(), out, n);
        } else {
          for (uint32_t k = 0; k < 4; ++k) {
            if (lmax <= 2) {
              n[k] = parse_pairs(p[k], 0, len[k], pairs.data(), out[k], 0);
            } else {
              buffer.clear();
              if (len[k]) dict.parse<false>(p[k], 0, len[k], buffer);
              n[k] = (uint32_t)buffer.size();
              for (uint32_t c = 0; c < n[k]; ++c) out[k][c] = final_of[buffer[c]];
            }
          }
        }
        for (uint32_t k = 0; k < 4; ++k) cnt[lane + k] = n[k];
      }
      r.add_unit(lanes, cnt, pad);
    };
    // Laying out a unit that is parsed already is about a third of the work of another: the caller's share is smaller by that.
    const uint64_t rest = n_units - u_frozen, done = u_frozen / 3, all = rest + done;
    auto range_start = [&](unsigned t) { return t == 0 ? 0 : std::min(rest, std::max(all * t / n_threads, done) - done); };   // of thread t, behind u_frozen
    // (what can fail for want of memory is taken here: nothing throws inside the threads but the long-run buffer's growth)
    const size_t lane_words = (size_t)64 * kMaxSegCols;
    std::unique_ptr<uint16_t[]> lanes(new uint16_t[lane_words * (1 + n_threads)]);
    std::vector<std::vector<uint16_t>> buffers(1 + n_threads);
    ranges[0].start(0, u_frozen, longest, room);
    for (unsigned t = 0; t < n_threads; ++t) {
      const uint64_t b = u_frozen + range_start(t), e = t + 1 == n_threads ? n_units : u_frozen + range_start(t + 1);
      ranges[1 + t].start(b, e, longest, room);
      if (lmax > 2) buffers[1 + t].reserve(kMaxSegCols);
    }
    // (range t + 1 is thread t's; the caller begins with the units parsed above)
    auto code_range = [&](unsigned t) {
      CodedRange& r = ranges[1 + t];
      for (uint64_t uu = r.u_begin; uu < r.u_end; ++uu) code_unit(uu, lanes.get() + lane_words * (1 + t), buffers[1 + t], r);
    };
    crew.run([&](unsigned t) {
      if (t == 0) {
        const uint16_t* src = grown.codes.data();
        for (uint64_t uu = 0; uu < u_frozen; ++uu) {
          uint32_t cnt[64];
          for (uint32_t l = 0; l < 64; ++l) {
            cnt[l] = grown.cnt[uu * 64 + l];
            uint16_t* out = lanes.get() + (size_t)l * kMaxSegCols;
            for (uint32_t k = 0; k < cnt[l]; ++k) out[k] = final_of[src[k]];
            src += cnt[l];
          }
          ranges[0].add_unit(lanes.get(), cnt, pad);
        }
      }
      code_range(t);
    });
  }

  // Unit offsets in chunks: a unit is its longest lane stream, rounded up to whole chunks.
  std::vector<uint32_t> uoff(n_units + 1, 0);
  uint64_t acc = 0, n_real = 0;
  for (const CodedRange& r : ranges) {
    n_real += r.n_real;
    for (uint64_t uu = r.u_begin; uu < r.u_end; ++uu) {
      uoff[uu] = (uint32_t)acc;
      acc += r.chunks[uu - r.u_begin];
      if (acc >= 0xFFFFFFFFull / kChunkWords) {
        set_error("tq_encode: code stream exceeds 2^32 codes");
        return TQ_E_UNSUPPORTED;
      }
    }
  }
  uoff[n_units] = (uint32_t)acc;

  h.n_entries = n_entries;
  h.pad_code = n_entries;
  h.n_chunks = acc;
  h.n_real_codes = n_real;
  h.dict_bytes = (uint64_t)(n_entries + 1) * 4;
  h.uoff_bytes = (n_units + 1) * 4;
  h.code_bytes = h.n_chunks * kChunkWords * 2;
  h.scale_bytes = (uint64_t)h.n_bands * kUnitRows * 4;
  h.off_dict = kHeaderBytes;
  h.off_uoff = round_up(h.off_dict + h.dict_bytes, kSectionAlign);
  h.off_codes = round_up(h.off_uoff + h.uoff_bytes, kSectionAlign);
  h.off_scales = round_up(h.off_codes + h.code_bytes, kSectionAlign);
  h.total_bytes = round_up(h.off_scales + h.scale_bytes, kSectionAlign);

  // Every byte is written below: the sections, and zeros between them (the pad entry is the first of those).
  // (in large pages, since all threads write it for the first time at once: 8192 x 3072 through the Python call 33 -> 17 ms on 8 CPUs, 10.7 -> 4.1
  // on 16; tq_free_blob frees it)
  std::unique_ptr<void, Free> owned = large_room(h.total_bytes);
  uint8_t* const blob = (uint8_t*)owned.get();
  auto put = [&](uint64_t at, const void* src, uint64_t n, uint64_t next) {
    std::memcpy(blob + at, src, n);
    std::memset(blob + at + n, 0, next - at - n);
  };
  std::memcpy(blob, &h, sizeof h);
  put(h.off_dict, words.data(), (uint64_t)n_entries * 4, h.off_uoff);
  put(h.off_uoff, uoff.data(), uoff.size() * 4, h.off_codes);
  std::memset(blob + h.off_codes + h.code_bytes, 0, h.off_scales - h.off_codes - h.code_bytes);
  put(h.off_scales, scales_pad.data(), (uint64_t)h.n_bands * kUnitRows * 4, h.total_bytes);
  {
    uint16_t* codes = (uint16_t*)(blob + h.off_codes);
    auto copy = [&](const CodedRange& r) {
      if (r.u_begin < r.u_end) std::memcpy(codes + (uint64_t)uoff[r.u_begin] * kChunkWords, r.words, r.used * 2);
    };
    crew.run([&](unsigned t) {
      if (t == 0) copy(ranges[0]);
      copy(ranges[1 + t]);
    });
  }
  *blob_out = owned.release();
  *bytes_out = (size_t)h.total_bytes;
  return TQ_OK;
}

}  // namespace
}  // namespace tq

using namespace tq;

extern "C" int tq_encode(const float* w, uint32_t rows, uint32_t cols, const tq_encode_opts* opts, void** blob,
                         size_t* blob_bytes) {
  try {
    if (!w || !blob || !blob_bytes || rows == 0 || cols == 0) {
      set_error("tq_encode: null pointer or empty matrix");
      return TQ_E_INVALID_ARG;
    }
    const uint32_t rows_pad = (uint32_t)round_up(rows, kUnitRows);
    std::vector<float> scales(rows_pad, 0.f);
    // Per row (quantize_row), with qmax = 2^(bits - 1) - 1 (paper section 3: a fixed range of levels set by the number of
    // bits; 127 at 8 bits).
    if (opts && opts->bits != 0 && (opts->bits < 2 || opts->bits > 8)) {
      set_error("tq_encode: bits must be 0 (= 8) or in [2, 8]");
      return TQ_E_INVALID_ARG;
    }
    const bool packed = opts && opts->packing == TQ_PACK_NIBBLES;
    if (packed && (opts->bits < 2 || opts->bits > 4)) {
      set_error("tq_encode: TQ_PACK_NIBBLES takes bits 2..4");
      return TQ_E_INVALID_ARG;
    }
    if (packed && cols % 2) {
      set_error("tq_encode: packing needs an even number of columns");
      return TQ_E_INVALID_ARG;
    }
    const float qmax = (float)((1u << ((opts && opts->bits ? opts->bits : 8u) - 1)) - 1u);
    const uint32_t width = packed ? cols / 2 : cols;   // stored bytes of a row
    // (threads take bands as they come, so that all of them meet in the same pages: 8192 x 3072 in ordinary ones 8.7 to 11.4 ms, in large ones, the
    // container's among them, 4.1)
    const std::unique_ptr<void, Free> stored = large_room((size_t)rows * width), unpacked = packed ? large_room((size_t)rows * cols) : nullptr;
    uint8_t* const Q = (uint8_t*)stored.get();
    Crew crew(crew_size(opts, rows, width));
    Bands bands(rows, crew.size(), [&](uint32_t first, uint32_t end) {
      for (uint32_t r = first; r < end; ++r) {
        uint8_t* q = (packed ? (uint8_t*)unpacked.get() : Q) + (size_t)r * cols;
        scales[r] = quantize_row(w + (size_t)r * cols, cols, qmax, q);
        if (packed)   // (the quantizer's values fit: qmax is at most 7)
          for (uint32_t c = 0; c < width; ++c) Q[(size_t)r * width + c] = (uint8_t)((q[2 * c] & 15) | (q[2 * c + 1] & 15) << 4);
      }
    });
    const Crew::Waits all(crew);   // (the bands and what they are made of stay until no thread is at them)
    crew.start([&](unsigned) { bands.make_all(); });
    return encode_quantized_matrix(Q, scales, rows, width, opts, crew, &bands, blob, blob_bytes);
  } catch (const std::bad_alloc&) {
    set_error("tq_encode: out of host memory");
    return TQ_E_OOM;
  } catch (...) {
    set_error("tq_encode: unexpected internal error (could a thread not be started?)");
    return TQ_E_HIP;
  }
}

extern "C" int tq_encode_quantized(const int8_t* q, const float* scales_in, uint32_t rows, uint32_t cols,
                                   const tq_encode_opts* opts, void** blob, size_t* blob_bytes) {
  try {
    if (!q || !scales_in || !blob || !blob_bytes || rows == 0 || cols == 0) {
      set_error("tq_encode_quantized: null pointer or empty matrix");
      return TQ_E_INVALID_ARG;
    }
    const uint32_t rows_pad = (uint32_t)round_up(rows, kUnitRows);
    const uint8_t* Q = (const uint8_t*)q;
    std::vector<float> scales(rows_pad, 0.f);
    std::copy(scales_in, scales_in + rows, scales.begin());
    if (opts && opts->packing == TQ_PACK_NIBBLES) {
      std::vector<uint8_t> P;
      if (!pack_nibbles(Q, rows, cols, &P)) return TQ_E_INVALID_ARG;
      Crew crew(crew_size(opts, rows, cols / 2));
      return encode_quantized_matrix(P.data(), scales, rows, cols / 2, opts, crew, nullptr, blob, blob_bytes);
    }
    Crew crew(crew_size(opts, rows, cols));
    return encode_quantized_matrix(Q, scales, rows, cols, opts, crew, nullptr, blob, blob_bytes);
  } catch (const std::bad_alloc&) {
    set_error("tq_encode_quantized: out of host memory");
    return TQ_E_OOM;
  } catch (...) {
    set_error("tq_encode_quantized: unexpected internal error (could a thread not be started?)");
    return TQ_E_HIP;
  }
}

extern "C" int tq_encode_gate_up(const float* w_gate, const float* w_up, uint32_t rows, uint32_t cols, const tq_encode_opts* opts,
                                 void** blob, size_t* blob_bytes) {
  if (!w_gate || !w_up || !blob || !blob_bytes || rows == 0 || cols == 0 || rows > 0x7FFFFFFFu) {
    set_error("tq_encode_gate_up: null pointer or empty shape");
    return TQ_E_INVALID_ARG;
  }
  try {
    std::vector<float> w((size_t)2 * rows * cols);   // row 2r = gate row r, row 2r + 1 = up row r
    for (uint32_t r = 0; r < rows; ++r) {
      std::memcpy(w.data() + (size_t)(2 * r) * cols, w_gate + (size_t)r * cols, (size_t)cols * 4);
      std::memcpy(w.data() + (size_t)(2 * r + 1) * cols, w_up + (size_t)r * cols, (size_t)cols * 4);
    }
    return tq_encode(w.data(), 2 * rows, cols, opts, blob, blob_bytes);
  } catch (const std::bad_alloc&) {
    set_error("tq_encode_gate_up: out of host memory");
    return TQ_E_OOM;
  } catch (...) {
    set_error("tq_encode_gate_up: unexpected internal error (could a thread not be started?)");
    return TQ_E_HIP;
  }
}

extern "C" void tq_free_blob(void* blob) { std::free(blob); }
