// Device side of libtq: the batched product with a ring per lane over runs of units (activations from global memory).
#pragma once
#include "tq_kernels_common.h"
#include "tq_kernel_ring.h"
#include "tq_strip_decode.h"

namespace tq {
// ---------------------------------------------------------------------------------------------------------------
// The ring decode of k_matvec_ring without its activation tile: every wavefront takes a contiguous run of units, bands
// one after the other and a band's quads in order, with the band's sums in registers from its first quad to its last.  No
// wavefront waits for another, so small launches are cut as finely as whole units allow, and the epilogue sees whole sums
// (silu(gate) * up needs them; k_matvec_ring adds to y quad by quad).
// The B operands come from global memory, 16 bytes per lane and MFMA step (they stay in the caches: a band after the other
// takes the same rows of x), requested a look ahead of their use.  x needs no alignment beyond its elements' (16-byte loads of
// global memory work at any 2-byte address), and rows need not be whole units: in a unit that reaches past the row's end
// (or whose segments are no multiple of a group of windows) a fragment is loaded where it still lies inside the row and
// shifted into place, zeros behind it.
// Batches of up to 8 rows take two windows per load, up to 4 rows four (fold_sums).
// Measured, us, buffers warm in the caches (in brackets: the whole-strip kernel, which took these launches before): 4099 x
// 2999 batch 5 17.5 (41), one LLaMA-3.2-3B layer batch 8 35.8 (56), batch 4 33.7, batch 16 52.0, 8192 x 3072 packed batch 4 14.1.
// Launches that fill k_matvec_ring go there (tq_choice.h): eight such layers, batch 8, 215 us there, 248 here, batch 16 228 and 484;
// the gated pairs of eight blocks, batch 16, 107 and 239.  What they differ in is x.  Counters of the eight layers at batch 8, M
// cycles summed over the compute units, there / here: busy 109 / 133, address unit of the vector memory path busy 64 / 107 (39 / 88 M
// cache accesses), vector instructions issued 86 / 89, LDS pipe busy 74 / 68.  The 16-byte pieces of up to 16 rows of x keep
// the address unit busy four fifths of the time here; with 16 rows in place of 8 there are twice as many of them.
constexpr int kRunWaves = 12;        // 60 KB of dictionary and 12 rings of 8 KB fill the LDS
constexpr int kRunSmallUnits = 6;    // units per workgroup up to which the rings are 64 bytes (batches above 4, one weight per byte)
constexpr int kRunWavesPacked = 8;   // packed 4-bit weights: two fragments and more conversion per piece, 12 wavefronts leave too few registers
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef __attribute__((address_space(1))) const u32x4_any global_cu128_any;

// The fragment's elements from element `by` on, zeros behind them (by >= 8: all zero).
__device__ __forceinline__ u32x4 drop_elements(u32x4 v, uint32_t by) {
  const bool four = by & 4u, two = by & 2u;
  u32x4 r = {four ? v.z : v.x, four ? v.w : v.y, four ? 0u : v.z, four ? 0u : v.w};
  r = u32x4{two ? r.y : r.x, two ? r.z : r.y, two ? r.w : r.z, two ? 0u : r.w};
  const uint32_t bits = (by & 1u) << 4;
  r = u32x4{__builtin_amdgcn_alignbit(r.y, r.x, bits), __builtin_amdgcn_alignbit(r.z, r.y, bits), __builtin_amdgcn_alignbit(r.w, r.z, bits), r.w >> bits};
  return by >= 8 ? u32x4{0u, 0u, 0u, 0u} : r;
}

// Decode and multiply the chunks [c0, c_end) of the units [u0, u1).  The first unit may begin and the last one end outside
// the run (see kSplit in k_matvec_runs): started says that the lanes stand at column `start` of the first one, and what
// a lane has not written itself counts as zeros.  x: the activations, row_first: where the
// batch row of this lane's B operand starts; part: the sums of the band in work.  on_unit(band, quad) is called when a unit has been multiplied.
// kFold: windows per B operand (fold_sums).
// ready() is called once, when the first codes have been requested (they are on their way while it waits for the dictionary), and returns `start`.
template <int kRing, bool kPacked, int kFold, typename Ready, typename OnUnit>
__device__ __forceinline__ void decode_run_ring(const DevMat& m, uint32_t u0, uint32_t u1, uint32_t c0, uint32_t c_end, bool started, Ready&& ready,
                                                global_cu16* x, uint32_t row_first, int lane, uint32_t ring, f32x4 (&part)[4], OnUnit&& on_unit) {
  if (u0 >= u1 || c0 >= c_end) {
    (void)ready();
    return;
  }
  constexpr int kP = ring_piece(kRing), kG = ring_group(kRing), kLook = ring_step(kRing), kParts = (kP + kLook - 1) / kLook;
  constexpr uint32_t pk = kPacked ? 2u : 1u;   // columns of the weight matrix per stored byte, windows per 8-byte piece of the ring
  constexpr uint32_t kLoads = kG * pk / kFold;
  const uint32_t behind = (lane & 15) / (16 / kFold) * 8;   // the columns this lane's window lies behind the operand's first
  const uint32_t sw8 = ring_swizzle<kRing>(lane), kg = (uint32_t)lane >> 4;
  const uint32_t nq = m.n_quads, n_panels = (m.cols + m.seg_cols - 1) / m.seg_cols, x_cols = pk * m.cols;
  // walker over the pieces of the run
  uint32_t wu = u0, wc = c0, w_left = 0, w_base = 0, w_rem = 0;
  bool w_ends = false;   // the unit the walker is in ends inside the run
  auto next_piece = [&](uint32_t& start, uint32_t& n, bool& ends) {
    if (w_left == 0) {
      if (wu == u1) {
        n = 0;
        ends = false;
        start = wc;
        return;
      }
      const uint32_t unit_end = unit_offset(m, wu + 1), len = min(unit_end, c_end) - wc;
      w_ends = unit_end <= c_end;
      w_left = (len + kP - 1) / kP;
      w_base = piece_length(len, w_left);
      w_rem = len - w_base * w_left;
      ++wu;
    }
    n = w_base + (w_rem ? 1u : 0u);
    if (w_rem) --w_rem;
    start = wc;
    wc += n;
    ends = --w_left == 0 && w_ends;
  };
  // every piece issues exactly kP loads (those past its end repeat its last chunk), kLook of them at a time
  auto load_part = [&](uint2 (&cw)[kP], uint32_t start, uint32_t n, int p) {
    const uint32_t last = min(start + max(n, 1u) - 1, c_end - 1);
#pragma unroll
    for (int k = p * kLook; k < (p + 1) * kLook && k < kP; ++k) cw[k] = load_chunk(m.codes, min(start + k, last), lane);
  };
  // the unit in work: its place, the lane's panel (length, first column of x) and segment (none past the last row), the
  // windows it takes (whole groups)
  uint32_t band = u0 / nq, quad = u0 - band * nq, panel_len, x_first, seg_len, n_win8, pos = 0, done = 0;
  bool ragged;
  uint64_t carry = 0;
  auto enter_unit = [&] {
    const uint32_t first = quad * kUnitPanels * m.seg_cols, panel = quad * kUnitPanels + kg;
    panel_len = panel < n_panels ? min(m.seg_cols, m.cols - panel * m.seg_cols) : 0u;
    seg_len = band * kUnitRows + (lane & 15) < m.rows ? panel_len : 0u;
    n_win8 = (min(m.seg_cols, m.cols - first) + 8 * kG - 1) / (8 * kG) * (8 * kG);
    ragged = first + kUnitPanels * m.seg_cols > m.cols || m.seg_cols % (8 * kG) != 0;
    x_first = pk * panel * m.seg_cols;
    pos = 0;
    done = 0;
    carry = 0;
  };
  u32x4 x8[kLoads];   // B operands of the next group
  auto request_x = [&] {
    const uint32_t at = x_first + pk * min(done, n_win8 - 8 * kG) + behind;
#pragma unroll
    for (uint32_t k = 0; k < kLoads; ++k) {
      const uint32_t col = ragged ? min(at + 8 * kFold * k, x_cols - 8) : at + 8 * kFold * k;
      x8[k] = *(global_cu128_any*)(x + (row_first + col));
    }
  };
  // One group of MFMA steps if every lane that is still decoding has written the columns [done, done + 8 kG).  The weights
  // are read before it is known whether the group is ready (volatile: the reads stay ahead of the test).
  auto multiply_ready = [&](auto look, bool ready = false) {   // look: see k_matvec_ring's
    constexpr int kFirst = decltype(look)::value * kG;
    const uint32_t at = min(done, n_win8 - 8 * kG);   // at the unit's end: any place inside the ring
    const uint32_t base = at ^ sw8;
    // a segment that ends inside a piece: what its last chunk left over is not in the ring yet
    if (ragged && ring_leftover(pos)) *(lds_u64*)(size_t)(ring | ((pos ^ sw8) & (kRing - 8u))) = carry;
    u32x2 a8[kG];
#pragma unroll
    for (int k = 0; k < kG; ++k) a8[k] = *(volatile lds_cu64*)(size_t)(ring | ((base ^ (8u * k)) & (kRing - 8u)));
    const uint32_t next = done + 8 * kG;
    if (next > n_win8) return;
    if (!ready && __builtin_amdgcn_ballot_w64(pos < min(seg_len, next)) != 0) return;
    if (ragged) {
#pragma unroll
      for (uint32_t k = 0; k < kLoads; ++k) {
        const uint32_t in_panel = pk * at + 8 * kFold * k + behind, col = x_first + in_panel;
        x8[k] = drop_elements(x8[k], in_panel >= pk * panel_len ? 8u : col + 8 > x_cols ? col + 8 - x_cols : 0u);
      }
    }
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
  typedef std::integral_constant<int, 0> First;
  auto decode_piece = [&](auto turn, const uint2 (&cw)[kP], uint32_t n, bool ends, uint2 (&cw_next)[kP], uint32_t next_start, uint32_t next_n) {
    if (n == 0) return;
    constexpr int kTurn = decltype(turn)::value;
    // a look: multiply what is ready, request the operands of the group that follows (again, if it was not)
    auto look = [&](auto number) {
      multiply_ready(number);
      request_x();
    };
    if (n >= kP - 1) {
      static_for<kP - 1>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        append_chunk_ring<kRing, true>(cw[k], ring, sw8, seg_len, pos, carry);
        if constexpr (k % kLook == kLook - 1) {
          look(std::integral_constant<int, kTurn + k / kLook>{});
          load_part(cw_next, next_start, next_n, k / kLook);
        }
      });
      if (n == kP) append_chunk_ring<kRing, true>(cw[kP - 1], ring, sw8, seg_len, pos, carry);
    } else {
      static_for<kP - 2>([&](auto kk) {
        constexpr int k = decltype(kk)::value;
        if ((uint32_t)k < n) append_chunk_ring<kRing, true>(cw[k], ring, sw8, seg_len, pos, carry);
        if constexpr (k % kLook == kLook - 1) {
          if ((uint32_t)k + 1 < n) look(std::integral_constant<int, kTurn + k / kLook>{});
          load_part(cw_next, next_start, next_n, k / kLook);
        }
      });
      if constexpr ((kP - 2) / kLook < kParts - 1) load_part(cw_next, next_start, next_n, kParts - 2);
    }
    multiply_ready(std::integral_constant<int, kTurn + kParts - 1>{});
    if (ends) {
      while (done < n_win8) {   // every lane is complete: whatever is left (at most a group, more in a ragged unit)
        request_x();
        multiply_ready(First{});
      }
      on_unit(band, quad);
      if (++quad == nq) {
        quad = 0;
        ++band;
      }
      if (band * nq + quad < u1) enter_unit();
    }
    request_x();
    load_part(cw_next, next_start, next_n, kParts - 1);
  };
  uint2 cwa[kP], cwb[kP];
  uint32_t sa, na, sb, nb;
  bool ea, eb;
  auto ring_piece = [&](uint32_t col) { return (lds_u64*)(size_t)(ring | ((col ^ sw8) & (kRing - 8u))); };
  enter_unit();
  next_piece(sa, na, ea);
#pragma unroll
  for (int j = 0; j < kParts; ++j) load_part(cwa, sa, na, j);
  const uint32_t start = ready();
  if (started) {   // the groups that every lane has passed are others' work; of the next ones, what a lane has passed is zeros here
    pos = min(start, seg_len);
    while (done + 8 * kG < n_win8 && __builtin_amdgcn_ballot_w64(pos < min(seg_len, done + 8 * kG)) == 0) done += 8 * kG;
    for (uint32_t col = done; __builtin_amdgcn_ballot_w64(col < (pos & ~7u)) != 0; col += 8)
      if (col < (pos & ~7u)) *ring_piece(col) = 0;
  }
  request_x();
  while (na) {   // two register sets: one is decoded while the other is filled
    next_piece(sb, nb, eb);
    decode_piece(First{}, cwa, na, ea, cwb, sb, nb);
    next_piece(sa, na, ea);
    decode_piece(std::integral_constant<int, kParts & 1>{}, cwb, nb, eb, cwa, sa, na);
  }
  if (c_end < unit_offset(m, u1)) {   // the last unit goes on elsewhere: multiply what the lanes have, zeros behind it
    *ring_piece(pos) = carry;
    while (__builtin_amdgcn_ballot_w64(pos > done) != 0) {
#pragma unroll
      for (int k = 0; k < kG; ++k)
        if (done + 8 * k > pos) *ring_piece(done + 8 * k) = 0;
      request_x();
      multiply_ready(First{}, true);
    }
  }
}

// kSplit: as in k_matvec, a share of few units is cut into equal runs of chunks, and the marks say where the lanes stand at the start of one
// (4099 x 2999 batch 5 17.8 -> 15.8 us against counts of each wavefront's part, exchanged through LDS).  A lone wavefront takes 8 us for a unit of 33 chunks, but the
// windows around a cut are multiplied on both sides of it, each time with zeros for the other side's columns: shares that
// leave less than half the wavefronts idle (above 8 batch rows, where the operands are twice as many loads: two thirds) are
// faster in whole units.  (us, whole units -> split: 2048 x 2048 batch 8 19.7 -> 15.0, 700 x 1999 batch 5 20.2 -> 16.6; 6 units of
// packed weights for 8 wavefronts 18.0 -> 23.2; batch 16, 6 units for 12 wavefronts: 4099 x 2999 27.7 -> 33.8, 8192 x 3072 22.7 -> 26.4.  That
// is with counts; with marks, beyond the line: 8192 x 3072 batch 16 21.4 -> 22.7, 4096 x 8192 batch 5 17.5 -> 19.3, batch 16 21.7 -> 26.8, 8192 x 3072 packed batch 4
// 12.0 -> 13.5; only 9 units gain, 12288 x 3072 batch 3 20.0 -> 19.3, batch 8 20.8 -> 19.9.)
// Rings of 64 bytes take such shares (kRunSmallUnits): groups of two windows leave half as much around a cut to be multiplied
// twice, and in ragged units.  us, rings of 128 -> 64 bytes: 4099 x 2999 batch 5 19.7 -> 18.6, 700 x 1999 batch 8 17.6 -> 16.7, batch 16 26.2 ->
// 22.9, 2048 x 2048 batch 16 15.5 -> 14.3, 3072 x 3072 batch 16 18.8 -> 16.4; larger shares equal or slower (16384 x 3072 batch 8 21.2 -> 22.6), and
// so are batches of up to 4 rows, whose operands then bring two windows instead of four (2048 x 2048 batch 3 12.4 -> 12.8).
constexpr uint32_t kRunSplitMin = 11;   // least chunks of a run, a third of a unit (4 / 6 / 8 / 11, us: 1024 x 1024 batch 3 14.8 / 14.5 /
                                        // 13.7 / 13.0, 2048 x 2048 batch 8 16.3 / 16.3 / 16.0 / 15.0, 700 x 1999 batch 5 17.8 / 17.9 / 18.0 / 16.6)
constexpr uint32_t kRunSplitMinSmall = 9;   // with rings of 64 bytes, whose pieces are 9 chunks (11 / 9, us: 1024 x 1024 batch 8 10.8 / 10.1, 2048 x 2048 12.9 /
                                            // 12.5, 700 x 1999 15.9 / 16.7; batch 16 14.3 / 14.5)
// kOne: as in k_matvec (one LLaMA-3.2-3B layer batch 8 37.1 -> 36.5 us; 4099 x 2999 batch 5, which has the loop over jobs, 18.1 -> 16.9 by the
// first codes requested ahead of the dictionary alone).
template <int kRing, int kWaves, bool kPacked, int kFold, bool kOne>
__global__ __launch_bounds__(kWaves * 64, 1) void k_matvec_runs(MatvecArgs a) {
  touch_arguments();
  extern __shared__ uint4 lds4[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t lo = blockIdx.x, hi = blockIdx.x + 1;
  if constexpr (!kOne) even_share(a, lo, hi);
  const uint32_t* staged = nullptr;
  const uint32_t rings = a.x_off;   // LDS address (the LDS segment starts at 0)
  const uint32_t ring = rings + (uint32_t)wave * (64 * kRing) + (uint32_t)lane * kRing;
  bool lds_used = false;
  for (int i = kOne ? mapped_job(a) : first_job(a, 0, a.n, lo, lane); kOne || i < a.n; ++i) {
    if (!kOne && hi <= cost_at(a, i)) break;
    Job job;
    DevMat m;
    fetch_job(a, i, job, m);
    uint32_t band_lo, band_hi;
    share_of_bands(a, kOne, m, i, lo, hi, band_lo, band_hi);
    if (band_lo >= band_hi) {
      if constexpr (kOne) return;
      continue;
    }
    const uint32_t nq = m.n_quads, unit_lo = band_lo * nq, n_units = (band_hi - band_lo) * nq;
    EvenRun run;
    const bool split = (kFold == 1 && !kPacked ? 3 : 2) * n_units <= kWaves;
    if (split) {
      const uint32_t uoff_lane = global_load(m.uoff + unit_lo + min((uint32_t)lane, n_units));
      run = even_run(uoff_lane, unit_lo, n_units, wave, kWaves, kRing == kSmallRingBytes && kFold > 1 ? kRunSplitMinSmall : kRunSplitMin);
    } else {
      run.u0 = unit_lo + (uint32_t)((uint64_t)n_units * wave / kWaves);
      run.u1 = unit_lo + (uint32_t)((uint64_t)n_units * (wave + 1) / kWaves);
      run.c0 = run.u0 < run.u1 ? unit_offset(m, run.u0) : 0u;
      run.c_end = run.u0 < run.u1 ? unit_offset(m, run.u1) : 0u;
      run.head = run.tail = false;
    }
    const bool new_dict = m.dict != staged;
    staged = m.dict;
    if (lds_used) __syncthreads();   // the previous matrix's dictionary and partial sums are no longer in use
    lds_used = true;
    // Called when the wavefront's first codes are on their way: the dictionary behind them.  Returns the columns of the run's first unit
    // that earlier wavefronts pass.
    auto ready = [&]() -> uint32_t {
      Place place;
      if (run.head) request_place(m, run.unit_start, run.c0, lane, place);
      if (new_dict) stage_image(m, lane, wave, kWaves, lds4);
      const uint32_t start = run.head ? columns_passed(place, run.unit_start, run.c0) : 0u;
      if (new_dict) {
        lds_arrived();
        __syncthreads();
      }
      return start;
    };
    BandSums sums;
    sums.start(run.u0, nq, run.head);
    f32x4 part[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto on_unit = [&](uint32_t band, uint32_t quad) {
      if (quad + 1 != nq && band * nq + quad + 1 != run.u1) return;
      sums.finish(a, job, m, band, quad + 1 == nq, fold_sums<kFold>(part), lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) part[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    global_cu16* x = (global_cu16*)job.x;
    // lanes past the batch repeat its last row: their sums are never stored
    const uint32_t row_first = min((uint32_t)(lane & 15) % (16 / kFold), (uint32_t)a.batch - 1) * (kPacked ? 2 : 1) * m.cols;
    decode_run_ring<kRing, kPacked, kFold>(m, run.u0, run.u1, run.c0, run.c_end, run.head, ready, x, row_first, lane, ring, part, on_unit);
    if (run.tail) sums.finish(a, job, m, (run.u1 - 1) / nq, false, fold_sums<kFold>(part), lane);
    __syncthreads();   // every wavefront is done with its ring: the partial sums go over the ring area
    sums.combine(a, job, m, rings, wave, kWaves, lane);
    if constexpr (kOne) return;
  }
}

}  // namespace tq
