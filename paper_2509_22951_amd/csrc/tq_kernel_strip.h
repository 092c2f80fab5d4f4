// Device side of libtq: the whole-strip batched product and the expansion to int8 matrices.
#pragma once
#include "tq_kernels_common.h"
#include "tq_strip_decode.h"

namespace tq {
// kLong: the matrices of the launch hold runs of up to 4 bytes (append_chunk_long).
template <bool kXFast, bool kPacked, bool kLong = false>
__global__ __launch_bounds__(kThreads, 1) void k_matvec_mfma(MatvecArgs a) {
  extern __shared__ uint4 lds4[];
  uint8_t* tiles = (uint8_t*)lds4 + a.x_off;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_waves = blockDim.x >> 6;
  uint32_t lo, hi;
  even_share(a, lo, hi);
  const uint32_t* staged = nullptr;
  const int bn = lane & 15, kg = lane >> 4;   // B operand: batch row and k-group of this lane
  for (int i = first_job(a, 0, a.n, lo, lane); i < a.n; ++i) {
    if (hi <= cost_at(a, i)) break;
    Job job;
    DevMat m;
    fetch_job(a, i, job, m);
    uint32_t band_lo, band_hi;
    share_of_bands(a, false, m, i, lo, hi, band_lo, band_hi);
    if (band_lo >= band_hi) continue;
    const uint32_t nq = m.n_quads;
    const uint32_t unit_lo = band_lo * nq, n_units = (band_hi - band_lo) * nq;
    const uint32_t u0 = unit_lo + (uint32_t)((uint64_t)n_units * wave / n_waves);
    const uint32_t u1 = unit_lo + (uint32_t)((uint64_t)n_units * (wave + 1) / n_waves);
    __syncthreads();   // the previous matrix's dictionary and partial sums are no longer in use
    if (m.dict != staged) {
      stage_image(m, lane, wave, n_waves, lds4);
      lds_arrived();
      staged = m.dict;
    }
    __syncthreads();
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    BandSums sums;
    sums.start(u0, nq);
    // lanes past the batch repeat its last row: their output columns are never stored
    constexpr uint32_t pk = kPacked ? 2u : 1u;   // columns of the weight matrix per stored byte
    const uint32_t x_cols = pk * m.cols;
    global_cu16* xrow = (global_cu16*)job.x + (size_t)min(bn, a.batch - 1) * x_cols;
    // acc holds the sums of the band in work when its last unit (or the run's) has been multiplied
    auto finish_unit = [&](uint32_t band, uint32_t quad) {
      if (quad + 1 != nq && band * nq + quad + 1 != u1) return;
      sums.finish(a, job, m, band, quad + 1 == nq, acc, lane);
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    {
      const uint32_t strip = m.seg_cols + 8;   // bytes between the strips of two lanes
      const uint32_t my_strip = lds_address(tiles) + (uint32_t)wave * a.tile_area + (uint32_t)lane * strip;
      constexpr int kG = kXFast ? kMfmaGroup : kMfmaGroupAny;
      uint4 xa[kG];   // activation fragments of the first MFMA group of the unit being decoded
      decode_run_to_tile<kLong>(m, u0, u1, lane, my_strip, [&](uint32_t, uint32_t quad) {
#pragma unroll
        for (int k = 0; k < kG; ++k)
          xa[k] = load_x_fragment<kXFast>(xrow, x_cols, pk * (quad * kUnitPanels + (uint32_t)kg) * m.seg_cols + 8 * k);
      }, [&](uint32_t band, uint32_t quad) {
        const uint32_t col0 = quad * kUnitPanels * m.seg_cols;                            // first (byte) column of the unit
        const uint32_t width = min(m.seg_cols, m.cols - col0);                            // its widest segment is the first panel's
        const uint32_t n_win = (pk * width + 7) / 8;
        const uint32_t xcol = pk * (col0 + (uint32_t)kg * m.seg_cols);
        const bool ragged = !kXFast || col0 + kUnitPanels * m.seg_cols > m.cols;          // some fragment reaches past the row's end
        if (ragged) acc = multiply_unit<kXFast, true, kPacked>(acc, my_strip, xrow, x_cols, xcol, n_win, xa);
        else acc = multiply_unit<kXFast, false, kPacked>(acc, my_strip, xrow, x_cols, xcol, n_win, xa);
        finish_unit(band, quad);
      });
    }
    __syncthreads();   // every wavefront is done with its tile: the partial sums go over the tile area
    sums.combine(a, job, m, lds_address(tiles), wave, n_waves, lane);
  }
}

// Expansion to the row-major int8 matrices (the paper's own online step: every codeword is replaced by its table
// sequence).  Same work split and same tile decode as the batched product; a finished unit is copied out in 16-byte
// pieces, consecutive lanes taking consecutive pieces of a row (4 panels x seg_cols contiguous bytes per row).
// The y pointer of a job is the int8 output matrix here; the activation pointer is not used.
template <bool kLong = false>
__global__ __launch_bounds__(kThreads, 1) void k_decompress(MatvecArgs a) {
  touch_arguments();   // (one 8192 x 3072 matrix 24.2 -> 23.5 us: the job is looked up by an index, so each of its lines would cost a round trip)
  extern __shared__ uint4 lds4[];
  uint8_t* tiles = (uint8_t*)lds4 + a.x_off;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_waves = blockDim.x >> 6;
  uint32_t lo, hi;
  even_share(a, lo, hi);
  const uint32_t* staged = nullptr;
  for (int i = first_job(a, 0, a.n, lo, lane); i < a.n; ++i) {
    if (hi <= cost_at(a, i)) break;
    Job job;
    DevMat m;
    fetch_job(a, i, job, m);
    uint32_t band_lo, band_hi;
    share_of_bands(a, false, m, i, lo, hi, band_lo, band_hi);
    if (band_lo >= band_hi) continue;
    const uint32_t nq = m.n_quads;
    const uint32_t unit_lo = band_lo * nq, n_units = (band_hi - band_lo) * nq;
    const uint32_t u0 = unit_lo + (uint32_t)((uint64_t)n_units * wave / n_waves);
    const uint32_t u1 = unit_lo + (uint32_t)((uint64_t)n_units * (wave + 1) / n_waves);
    if (m.dict != staged) {
      __syncthreads();   // nobody reads the previous dictionary any more
      stage_image(m, lane, wave, n_waves, lds4);
      lds_arrived();
      staged = m.dict;
      __syncthreads();
    }
    const uint32_t strip = m.seg_cols + 8;
    const uint32_t tile_lds = lds_address(tiles) + (uint32_t)wave * a.tile_area;   // matrices of different segment width may be in work at once
    int8_t* out = (int8_t*)job.y;
    const bool aligned = ((m.packing ? 2 * m.cols : m.cols) % 16 == 0) && ((uintptr_t)out % 16 == 0);
    const uint32_t ppp = m.seg_cols / 16;   // 16-byte pieces per segment
    decode_run_to_tile<kLong>(m, u0, u1, lane, tile_lds + (uint32_t)lane * strip, [](uint32_t, uint32_t) {}, [&](uint32_t band, uint32_t quad) {
      for (uint32_t pc = lane; pc < 64 * ppp; pc += 64) {
        const uint32_t seg = pc / ppp, part = pc - seg * ppp;            // segment (row seg / 4, panel seg % 4) of the unit
        const uint32_t row = band * kUnitRows + (seg >> 2), col = (quad * kUnitPanels + (seg & 3)) * m.seg_cols + part * 16;
        if (row >= m.rows || col >= m.cols) continue;
        const uint32_t src = tile_lds + ((seg >> 2) + 16 * (seg & 3)) * strip + part * 16;   // strip of lane (row, panel)
        const u32x2 lo8 = *(lds_cu64*)(size_t)src, hi8 = *(lds_cu64*)(size_t)(src + 8);
        if (m.packing) {   // 16 bytes -> 32 int8: columns 2 col .. 2 col + 31 of a row of 2 cols values
          int8_t* dst2 = out + ((size_t)row * m.cols + col) * 2;
          const uint32_t w[4] = {lo8.x, lo8.y, hi8.x, hi8.y};
          uint32_t e[8];
#pragma unroll
          for (int k = 0; k < 4; ++k) {   // nibbles to bytes with their sign (8 -> 0xF8 inside its own byte), then in column order
            uint32_t even = w[k] & 0x0F0F0F0Fu, odd = (w[k] >> 4) & 0x0F0F0F0Fu;
            even |= (even & 0x08080808u) * 0x1Eu;
            odd |= (odd & 0x08080808u) * 0x1Eu;
            e[2 * k] = __builtin_amdgcn_perm(odd, even, 0x05010400u);
            e[2 * k + 1] = __builtin_amdgcn_perm(odd, even, 0x07030602u);
          }
          if (aligned && col + 16 <= m.cols) {
            *(__attribute__((address_space(1))) u32x4*)dst2 = u32x4{e[0], e[1], e[2], e[3]};
            *(__attribute__((address_space(1))) u32x4*)(dst2 + 16) = u32x4{e[4], e[5], e[6], e[7]};
          } else {
#pragma unroll
            for (int k = 0; k < 32; ++k)
              if (col + k / 2 < m.cols) *(__attribute__((address_space(1))) int8_t*)(dst2 + k) = (int8_t)(e[k >> 2] >> (8 * (k & 3)));
          }
          continue;
        }
        int8_t* dst = out + (size_t)row * m.cols + col;
        if (aligned && col + 16 <= m.cols) {
          u32x4 v = {lo8.x, lo8.y, hi8.x, hi8.y};
          *(__attribute__((address_space(1))) u32x4*)dst = v;
        } else {
          const uint32_t w[4] = {lo8.x, lo8.y, hi8.x, hi8.y};
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (col + k < m.cols) *(__attribute__((address_space(1))) int8_t*)(dst + k) = (int8_t)(w[k >> 2] >> (8 * (k & 3)));
        }
      }
    });
  }
}

}  // namespace tq
