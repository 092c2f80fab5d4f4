// Device side of libtq: the batched product with a ring per lane (decode and MFMA interleaved).
#pragma once
#include "tq_kernels_common.h"
#include "tq_plan.h"
#include "tq_strip_decode.h"

namespace tq {
// ---------------------------------------------------------------------------------------------------------------
// The batched product with a ring of 64 bytes per lane in place of the whole strip, and the activations in LDS.
//
// The 16 rows of a band take their codes in step but reach different columns, so some per-lane storage has to bring
// them back into line before an MFMA can take 8 columns of all of them; what it has to hold is only the distance
// between the slowest and the fastest lane, not the segment.  Every ring_step chunks the wavefront asks whether every
// lane has passed the next ring_group windows (one compare and a look at the condition mask) and, if so,
// multiplies them; a lane advances by at most 8 columns per chunk, so one group per look keeps up.  Bytes of the ring
// are reused 64 columns later: a lane writes 8-byte piece q only when q + 8 - 64 <= done, which holds
// whenever no lane is ever more than ring_spread columns ahead of an unfinished one (derived in tq_plan.h); the host sees to
// that for every unit when the container is loaded (level_unit): 33 columns.  A matrix where it cannot (its lanes change places:
// one ahead now and slower than the others later on, without a code to spare) goes to the runs kernel, whose rings of 128 bytes take
// 65 columns, and beyond that to the whole-strip kernel.  (Of 320 containers of the encoder, normal and Student-t weights in all widths,
// segments and dictionaries, none has such a matrix with segments of up to 256 columns.  One made for it, lanes 40 columns apart,
// eight times 8192 x 3072: 104 us at batch 8 and 198 at batch 16, 83 and 97 by a form of this kernel with rings of 128 bytes.)
// Piece p (8 bytes) of lane l lives at p ^ ring_swizzle(l) within the lane's ring: when the 64 lanes read the same window, the
// 16 lanes served together hit different banks.
//
// With 4 KB of ring per wavefront, 16 wavefronts leave room for the activations of one quad (4 panels) in LDS, laid out
// as the B operands the MFMA steps take: [panel][window][batch row 0..15][8 columns], 16 bytes per lane and step, read
// with one ds_read_b128.  (Taken from global memory, every step's fragment load touches 4 panels x batch rows
// different cache lines; that, not the decode, then bounds the kernel.)  All wavefronts of a workgroup therefore work
// on the same quad at a time: the workgroup walks the quads of its bands in the outer loop, wavefront w takes the
// whole bands, and a band's sums go to y once per quad: a plain store for the first quad, an atomic add (no return
// value, so nothing waits for it) for the others.  The stores and adds to a given y element are issued in quad order,
// one workgroup barrier apart from each other, so the result does not depend on timing.
// Needs rows of a whole number of units (a multiple of 4 * seg_cols columns), segments of 32..256 columns in
// multiples of 32 (packed 4-bit weights: 32..128 bytes), and 16-byte aligned activations.
//
// 16 wavefronts: with rings of 128 bytes there is LDS for 10, which keep the vector ALUs busy for 75 % of the time.  12 of gated pairs,
// whose sums stay in registers (16 would spill them); of the plain forms the one for packed weights and 9 to 16 rows of x spills 9
// registers and is still faster with 16.  us, rings of 128 bytes -> 64 with 16 | 12 wavefronts: eight LLaMA-3.2-3B layers batch 4
// 225 -> 203 | 222, batch 8 228 -> 208 | 223, batch 16 252 -> 228 | 239, packed weights batch 8 182 -> 151 | 169, batch 16 202 ->
// 183 | 189; gated pairs of eight blocks batch 8 116 -> 103 | 99, batch 16 119 -> 113 | 102, packed batch 8 92 -> 80 | 77, batch 16
// 94 -> 90 | 79.  (Two accumulators per wavefront instead of four, which the groups of two windows suggest, made the sums 8 % less
// exact: hence the turns in multiply_ready.)
constexpr int kRingWaves = 16, kRingWavesGated = 12;
constexpr uint32_t kRingMaxSeg = 256;
constexpr int kRingMinBandsPerCu = 24;   // tq_set_ring_min_bands_per_cu's default: the choice by estimate (tq_choice.h)
constexpr uint32_t ring_x_tile(int rows) { return kUnitPanels * kRingMaxSeg * rows * 2; }   // bytes: 4 panels x 256 columns x batch rows of bf16

// 8 * swizzle(lane): lanes 2 (4) apart start on the same bank when a ring is 128 (64) bytes
template <int kRing>
__device__ __forceinline__ uint32_t ring_swizzle(int lane) { return (kRing == 128 ? (uint32_t)lane & 15u : (uint32_t)lane >> 2 & 7u) << 3; }

// append_chunk for the ring: the complete 8-byte piece goes to its swizzled place; sw8 = ring_swizzle(lane).
// kClamp: pos never passes seg_len (pad codes fall off the end).  A piece is complete when pos crosses a multiple of 8.
template <int kRing, bool kClamp>
__device__ __forceinline__ void append_chunk_ring(uint2 c, uint32_t ring, uint32_t sw8, uint32_t seg_len, uint32_t& pos, uint64_t& carry) {
  uint32_t s0, s1, n;
  chunk_string(c, s0, s1, n);                                           // the 4..8 bytes of the chunk, zero above them
  const uint64_t str = (uint64_t)s1 << 32 | s0;
  const uint32_t after = kClamp ? min(pos + n, seg_len) : pos + n;
  const uint32_t sh = (pos & 7u) << 3;
  const uint64_t lo = carry | str << sh, hi = (str >> 1) >> (63 - sh);  // the 16 bytes carry + string; hi is 0 when pos % 8 == 0
  const bool full = (after ^ pos) >= 8;
  // stored whether the piece is complete or not (an incomplete one holds zeros above its bytes and is stored again,
  // complete, by a later chunk; nobody reads a piece before every lane has passed it): no branch in the chunk's code
  *(lds_u64*)(size_t)(ring | ((pos ^ sw8) & (kRing - 8u))) = lo;
  carry = full ? hi : lo;
  pos = after;
}

typedef __attribute__((address_space(3))) const u32x4 lds_cu128;

// Decode and multiply units of quad `quad`, one band after the other (every unit has 4 whole panels of seg_cols
// columns): first the one of band first_band, then those of the bands claim() hands out, until it returns kNoBand.
// ring: LDS address of the lane's ring; xfrag: LDS address of the lane's 16 bytes of window 0 in the activation tile
// (window w is 16 kRows w bytes further).  on_unit(band, next_band, sums) is called with a unit's 16 x 16 sums after its
// last MFMA step; next_band is the band that follows (claimed a piece of chunks ahead), or kNoBand.
constexpr uint32_t kNoBand = 0xFFFFFFFFu;
// kPacked: the ring holds packed 4-bit weights; an 8-byte piece is then two MFMA steps (16 columns), and the activation
// tile has two windows per piece.
template <int kRows, bool kPacked, typename Claim, typename OnUnit>
__device__ __forceinline__ void decode_units_ring(const DevMat& m, uint32_t quad, uint32_t first_band, Claim&& claim, int lane, uint32_t ring,
                                                  uint32_t xfrag, OnUnit&& on_unit) {
  if (first_band == kNoBand) return;
  constexpr int kRing = kSmallRingBytes;
  constexpr int kP = ring_piece(kRing), kG = ring_group(kRing), kLook = ring_step(kRing), kParts = (kP + kLook - 1) / kLook;
  static_assert((kP - 1) / kLook == kParts - 1 && (kP - 2) / kLook >= kParts - 2, "the parts of a piece that the loops below request");
  constexpr int kFold = 16 / kRows;   // windows per B operand (fold_sums)
  const uint32_t sw8 = ring_swizzle<kRing>(lane);
  const uint32_t n_win8 = m.seg_cols;
  // A row past the end of the matrix has no segment: its lane holds pads alone and stands behind the last window from the start.
  auto first_column = [&](uint32_t band) { return band != kNoBand && band * kUnitRows + (lane & 15) < m.rows ? 0u : n_win8; };
  uint32_t cur_band = first_band;
  // walker over the pieces: the band it is in (the decoder is at most one band behind), pieces left in it, next chunk
  uint32_t w_band = kNoBand, wc = 0, w_left = 0, w_base = 0, w_rem = 0;
  bool w_started = false;
  auto next_piece = [&](uint32_t& start, uint32_t& n, bool& ends) {
    if (w_left == 0) {
      if (w_started && w_band == kNoBand) {   // nothing left to claim
        n = 0;
        ends = false;
        start = wc;
        return;
      }
      w_band = w_started ? claim() : first_band;
      w_started = true;
      if (w_band == kNoBand) {
        n = 0;
        ends = false;
        start = wc;
        return;
      }
      const uint32_t u = w_band * m.n_quads + quad;
      wc = unit_offset(m, u);
      const uint32_t len = unit_offset(m, u + 1) - wc;
      w_left = (len + kP - 1) / kP;
      // (the kernel for 16 rows and packed weights is at its register limit and loses by the branches of piece_length: us, with them -> a division, 30
      // matrices of 1420 x 1536 55.4 -> 53.8, seven LLaMA-3.2-3B pairs of 8192 x 3072 and back 121.9 -> 120.5, batch 9 117.9 -> 117.2; the one for 8 rows gains by them, 71.8 -> 71.0)
      w_base = kPacked && kRows == 16 ? len / w_left : piece_length(len, w_left);
      w_rem = len - w_base * w_left;
    }
    n = w_base + (w_rem ? 1u : 0u);
    if (w_rem) --w_rem;
    start = wc;
    wc += n;
    ends = --w_left == 0;
  };
  // Every piece issues exactly kP loads (those past its end repeat its last chunk), kLook of them at a time.
  auto load_part = [&](uint2 (&cw)[kP], uint32_t start, uint32_t n, int part) {
    const uint32_t last = n ? start + n - 1 : start - 1;   // n == 0 (past the last unit, start >= 1): the chunk before, never used
#pragma unroll
    for (int k = part * kLook; k < (part + 1) * kLook && k < kP; ++k) cw[k] = load_chunk(m.codes, min(start + k, last), lane);
  };
  uint32_t pos = first_column(first_band), done = 0;
  uint64_t carry = 0;
  f32x4 part[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  // One group of MFMA steps if every lane that is still decoding has written the columns [done, done + 8 kG).
  // The operands are read before it is known whether the group is ready (volatile: the reads stay ahead of the test),
  // so that their latency overlaps the test; an unready group just reads them again at the next look.
  // look: the looks take the accumulators in turn where a group has fewer windows than there are of them.
  auto multiply_ready = [&](auto look) {
    constexpr int kFirst = decltype(look)::value * kG;
    const uint32_t at = min(done, n_win8 - 8 * kG);   // at the unit's end: any place inside the ring and the tile
    const uint32_t base = at ^ sw8;
    constexpr int kX = kPacked ? 2 : 1;             // activation windows per 8-byte piece of the ring
    const uint32_t xa = xfrag + at * (2 * kRows * kX);   // 16 kRows bytes per window
    u32x2 a8[kG];
    u32x4 x8[kG * kX / kFold];
#pragma unroll
    for (int k = 0; k < kG; ++k) a8[k] = *(volatile lds_cu64*)(size_t)(ring | ((base ^ (8u * k)) & (kRing - 8u)));
#pragma unroll
    for (int k = 0; k < kG * kX / kFold; ++k) x8[k] = *(volatile lds_cu128*)(size_t)(xa + 16 * kRows * kFold * k);
    const uint32_t next = done + 8 * kG;
    if (next > n_win8) return;
    if (__builtin_amdgcn_ballot_w64(pos < next) != 0) return;
#pragma unroll
    for (int k = 0; k < kG; ++k) {
      if constexpr (kPacked) {
        f32x4 &p0 = part[2 * k & 3], &p1 = part[(2 * k + 1) & 3];
        p0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nib8_to_bf16x8(a8[k].x), __builtin_bit_cast(bf16x8, x8[2 * k / kFold]), p0, 0, 0, 0);
        p1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(nib8_to_bf16x8(a8[k].y), __builtin_bit_cast(bf16x8, x8[(2 * k + 1) / kFold]), p1, 0, 0, 0);
      } else {
        f32x4& p = part[(kFirst + k) & 3];
        p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(i8x8_to_bf16x8(make_uint2(a8[k].x, a8[k].y)), __builtin_bit_cast(bf16x8, x8[k / kFold]), p, 0, 0, 0);
      }
    }
    done = next;
  };
  auto decode_piece = [&](auto turn, const uint2 (&cw)[kP], uint32_t n, bool ends, uint2 (&cw_next)[kP], uint32_t next_start, uint32_t next_n) {
    if (n == 0) return;
    constexpr int kTurn = decltype(turn)::value;
    if (n >= kP - 1) {
      static_for<kP - 1>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        append_chunk_ring<kRing, false>(cw[k], ring, sw8, 0u, pos, carry);
        if constexpr (k % kLook == kLook - 1) {
          multiply_ready(std::integral_constant<int, kTurn + k / kLook>{});
          load_part(cw_next, next_start, next_n, k / kLook);
        }
      });
      if (n == kP) append_chunk_ring<kRing, false>(cw[kP - 1], ring, sw8, 0u, pos, carry);
    } else {
      static_for<kP - 2>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        if ((uint32_t)k < n) append_chunk_ring<kRing, false>(cw[k], ring, sw8, 0u, pos, carry);
        if constexpr (k % kLook == kLook - 1) {
          if ((uint32_t)k + 1 < n) multiply_ready(std::integral_constant<int, kTurn + k / kLook>{});
          load_part(cw_next, next_start, next_n, k / kLook);
        }
      });
      if constexpr ((kP - 2) / kLook < kParts - 1) load_part(cw_next, next_start, next_n, kParts - 2);
    }
    multiply_ready(std::integral_constant<int, kTurn + kParts - 1>{});
    load_part(cw_next, next_start, next_n, kParts - 1);
    if (ends) {   // every lane is complete and at most one whole group was left: the unit has been multiplied
      // the walker is one piece ahead: w_band is the band of the unit that follows, if there is one
      const uint32_t next_band = w_band == cur_band ? kNoBand : w_band;
      on_unit(cur_band, next_band, fold_sums<kFold>(part));
#pragma unroll
      for (int k = 0; k < 4; ++k) part[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      cur_band = next_band;
      pos = first_column(cur_band);
      carry = 0;
      done = 0;
    }
  };
  uint2 cwa[kP], cwb[kP];
  uint32_t sa, na, sb, nb;
  bool ea, eb;
  next_piece(sa, na, ea);
#pragma unroll
  for (int j = 0; j < kParts; ++j) load_part(cwa, sa, na, j);
  while (na) {   // two register sets: one is decoded while the other is filled
    next_piece(sb, nb, eb);
    decode_piece(std::integral_constant<int, 0>{}, cwa, na, ea, cwb, sb, nb);
    next_piece(sa, na, ea);
    decode_piece(std::integral_constant<int, kParts & 1>{}, cwb, nb, eb, cwa, sa, na);
  }
}

// kGateUp: y = silu(gate row) * (up row) needs a band's whole sums, so nothing is added to y: the bands are taken in passes
// of kGateUpBands per wavefront, each wavefront's bands fixed, with their sums in registers from the first quad to the
// last.  A pass takes 32 bands at least (gated pairs of eight LLaMA-3.2-3B blocks, batch 16, 12 wavefronts: 102 us in one pass of
// 36 bands, 121 in two of 24).
template <int kWaves, int kRows, bool kPacked, bool kGateUp = false>
__global__ __launch_bounds__(kWaves * 64, 1) void k_matvec_ring(MatvecArgs a) {
  constexpr int kRing = kSmallRingBytes, kRingThreads = kWaves * 64, kGateUpBands = (32 + kWaves - 1) / kWaves;
  constexpr uint32_t kRingXTile = ring_x_tile(kRows);
  // A wavefront's bands are fixed then, and the others wait for it at the end of the quad (us, packed gated pairs of eight LLaMA-3.2-3B blocks:
  // batch 8 76.9 -> 75.3, batch 16 79.7 -> 78.0; with one weight per byte nothing).
  constexpr bool kPaced = kGateUp && kPacked;
  extern __shared__ uint4 lds4[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t rings = a.x_off, xtile = a.slot_off;   // LDS addresses (the LDS segment starts at 0)
  uint32_t lo, hi;
  even_share(a, lo, hi);
  const uint32_t* staged = nullptr;
  const int bn = lane & 15, kg = lane >> 4;   // B operand: batch row and k-group (panel) of this lane
  const uint32_t ring = rings + (uint32_t)wave * (64 * kRing) + (uint32_t)lane * kRing;
  for (int i = first_job(a, 0, a.n, lo, lane); i < a.n; ++i) {
    if (hi <= cost_at(a, i)) break;
    Job job;
    DevMat m;
    fetch_job(a, i, job, m);
    uint32_t band_lo, band_hi;
    share_of_bands(a, false, m, i, lo, hi, band_lo, band_hi);
    if (band_lo >= band_hi) continue;
    constexpr uint32_t pk = kPacked ? 2u : 1u;             // columns of the weight matrix per stored byte
    const uint32_t nq = m.n_quads, n_win = pk * m.seg_cols / 8;   // activation windows (8 columns) per segment
    __syncthreads();   // the previous matrix's dictionary and activation tile are no longer in use
    // Bands are handed out one at a time, per quad, through a counter in LDS: wavefront w starts with band w of the
    // workgroup's range and claims the next free one while it decodes the last piece of chunks of the one in work.
    // (An even split up front leaves wavefronts waiting at the end of every quad: for the slowest, and for the one more
    // band that some of them have.)
    const uint32_t n_bands = band_hi - band_lo, pass_bands = kGateUp ? (uint32_t)(kGateUpBands * kWaves) : n_bands;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    lds_u32* next_band_counter = (lds_u32*)(size_t)(xtile + kRingXTile);
    uint32_t pass_lo = band_lo, pass_hi = band_lo, own_band = 0;
    auto claim = [&]() {
      if constexpr (kGateUp) {
        own_band += kWaves;
        return own_band < pass_hi ? own_band : kNoBand;
      } else {
        uint32_t b = 0;
        if (lane == 0) b = __hip_atomic_fetch_add(next_band_counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        b = __builtin_amdgcn_readfirstlane(b);
        return b < n_bands ? band_lo + b : kNoBand;
      }
    };
    // 16 columns of a B operand: 16 / kRows windows of kRows rows (fold_sums)
    const uint32_t xfrag = xtile + ((uint32_t)kg * n_win * kRows + bn) * 16;
    // Activation tile of a quad: piece ((panel * n_win + w) * kRows + batch row) holds 8 columns; rows past the batch are
    // zero.  The pieces of the next quad's tile are requested into registers before this quad is decoded and written
    // to LDS when everybody has finished it, so that nobody waits for device memory between two quads.
    constexpr int kTileRegs = (kRingXTile / 16 + kRingThreads - 1) / kRingThreads;
    const uint32_t pieces = kUnitPanels * n_win * kRows, per_row = kUnitPanels * n_win;
    u32x4 tile[kTileRegs];
    auto request_tile = [&](uint32_t q) {
      const uint32_t col0 = q * kUnitPanels * pk * m.seg_cols;
#pragma unroll
      for (int k = 0; k < kTileRegs; ++k) {
        const uint32_t o = min((uint32_t)tid + k * kRingThreads, pieces - 1);
        const uint32_t r = o / per_row, c = o - r * per_row;   // batch row, 8-column piece of the quad
        tile[k] = *(global_cu128*)((global_cu16*)job.x + (size_t)min(r, (uint32_t)a.batch - 1) * (pk * m.cols) + col0 + 8 * c);
      }
    };
    auto commit_tile = [&]() {
#pragma unroll
      for (int k = 0; k < kTileRegs; ++k) {
        const uint32_t o = (uint32_t)tid + k * kRingThreads;
        const uint32_t r = o / per_row, c = o - r * per_row;
        u32x4 v = tile[k];
        if (r >= (uint32_t)a.batch) v = u32x4{0u, 0u, 0u, 0u};
        if (o < pieces) *(__attribute__((address_space(3))) u32x4*)(size_t)(xtile + (c * kRows + r) * 16) = v;   // c = panel * n_win + w
      }
    };
    request_tile(0);
    if (m.dict != staged) {
      stage_image(m, lane, wave, kWaves, lds4);
      lds_arrived();
      staged = m.dict;
    }
    for (; pass_lo < band_hi; pass_lo = pass_hi) {
      pass_hi = min(band_hi, pass_lo + pass_bands);
      f32x4 acc[kGateUpBands];   // kGateUp: the sums of this wavefront's bands of the pass
#pragma unroll
      for (int k = 0; k < kGateUpBands; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (uint32_t q = 0; q < nq; ++q) {
        if (q || pass_lo != band_lo) __syncthreads();   // everybody has finished the previous quad: its activation tile can go
        if (!kGateUp && tid == 0) *next_band_counter = kWaves;   // bands 0 .. kWaves - 1 are the wavefronts' first ones
        commit_tile();
        if (q + 1 < nq || pass_hi < band_hi) request_tile(q + 1 < nq ? q + 1 : 0);
        __syncthreads();
        // Sums of lane l: rows 4 * (l / 16) + v of the band, batch row l % 16.  The scales of the next band are requested
        // when this one's have been used, a unit ahead of their use: waiting for them is then not a wait for the code
        // chunks requested in between.
        const uint32_t band0 = (uint32_t)wave < pass_hi - pass_lo ? pass_lo + wave : kNoBand;
        own_band = pass_lo + wave;
        float scale[4];
        auto request_scales = [&](uint32_t band) {
#pragma unroll
          for (int v = 0; v < 4; ++v) scale[v] = global_load(m.scales + min(band, m.n_bands - 1) * kUnitRows + 4 * kg + v);
        };
        if constexpr (!kGateUp) request_scales(band0);
        auto finish_unit = [&](uint32_t band, uint32_t next_band, f32x4 sums) {
          if constexpr (kGateUp) {
            const uint32_t mine = (band - pass_lo) / kWaves;
#pragma unroll
            for (int k = 0; k < kGateUpBands; ++k)   // (a sum of selected values: indexed, the array would go to memory)
#pragma unroll
              for (int v = 0; v < 4; ++v) acc[k][v] += mine == (uint32_t)k ? sums[v] : 0.f;
            if constexpr (kPaced) {   // a level for every band done
              if (mine == 0) __builtin_amdgcn_s_setprio(2);
              else if (mine == 1) __builtin_amdgcn_s_setprio(1);
              else __builtin_amdgcn_s_setprio(0);
            }
            return;
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const uint32_t row = band * kUnitRows + 4 * kg + v;
            if (bn < a.batch && row < m.rows) {
              float* y = job.y + (size_t)bn * m.rows + row;
              if (q == 0) global_store(y, sums[v] * scale[v]);
              else (void)__builtin_amdgcn_global_atomic_fadd_f32((__attribute__((address_space(1))) float*)y, sums[v] * scale[v]);
            }
          }
          request_scales(next_band);
        };
        if constexpr (kPaced) __builtin_amdgcn_s_setprio(3);
        decode_units_ring<kRows, kPacked>(m, q, band0, claim, lane, ring, xfrag, finish_unit);
        if constexpr (kPaced) __builtin_amdgcn_s_setprio(0);
      }
      if constexpr (kGateUp) {
#pragma unroll
        for (int k = 0; k < kGateUpBands; ++k) {
          const uint32_t band = pass_lo + k * kWaves + wave;
          if (band < pass_hi) BandSums::store(a, job, m, band, acc[k], lane);
        }
      }
    }
  }
}

}  // namespace tq
