// Device side of libtq: the dot-product kernel for one or two activation rows (dictionary lookup, activation gather,
// one dot product per code and row).
#pragma once
#include "tq_kernels_common.h"

namespace tq {
// Staging is split in two so that the loads of the dictionary, of the activations and of the first code chunks are
// all in flight together before anything waits: issue_* only loads into registers, commit_* writes LDS; the dictionary's loads write LDS
// themselves (request_to_lds).

// LDS image of one activation row: dword (panel * x_span + c) = (x[panel * seg_cols + c], x[panel * seg_cols + c + 1])
// as two bf16, zero past the end of the row; the gap dwords between panels and the tail are zero.
// Thread t of a round handles the column pair (2 j, 2 j + 1), j = first_pair + k * kThreads + t: it loads x[2j], x[2j + 1];
// x[2j + 2] is the next lane's, but for the last lane, which loads it (or every lane, when x is not aligned).
template <bool kAligned, int kThreads, int kXRegs, bool kCoherent = false>   // kXRegs x kThreads x 2 columns per round (8192)
__device__ __forceinline__ void issue_activations(const DevMat& m, const uint16_t* __restrict__ x, uint32_t first_pair, int tid,
                                                  uint32_t (&lo)[kXRegs], uint32_t (&hi)[kXRegs]) {
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    const uint32_t j = first_pair + k * kThreads + tid, col = 2 * j;
    lo[k] = hi[k] = 0u;
    if (2 * (first_pair + k * kThreads) >= m.cols) continue;   // (the same for all: rows are mostly shorter than a round of loads)
    if (kAligned) {   // x is 4-byte aligned and cols is even
      lo[k] = col < m.cols ? x_load<kCoherent>((const uint32_t*)x + j) : 0u;
    } else {
      lo[k] = (col < m.cols ? x_load<kCoherent>(x + col) : 0u) | (col + 1 < m.cols ? x_load<kCoherent>(x + col + 1) << 16 : 0u);
    }
  }
  if ((tid & 63) == 63) {
#pragma unroll
    for (int k = 0; k < kXRegs; ++k) {
      const uint32_t col = 2 * (first_pair + k * kThreads + tid) + 2;
      if (2 * (first_pair + k * kThreads) >= m.cols) continue;
      if (col < m.cols) hi[k] = x_load<kCoherent>(x + col);
    }
  }
}
template <int kThreads, int kXRegs>
__device__ __forceinline__ void commit_activations(const DevMat& m, uint32_t first_pair, int tid, const uint32_t (&lo)[kXRegs],
                                                   const uint32_t (&hi)[kXRegs], uint32_t* lds_x, uint32_t image_cols) {
  const uint32_t gap = m.x_span - m.seg_cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    if (2 * (first_pair + k * kThreads) >= image_cols) continue;
    const uint32_t col = 2 * (first_pair + k * kThreads + tid);
    // the next lane's pair (wave shift by one lane; the last lane keeps what it loaded itself)
    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)hi[k], (int)lo[k], 0x130, 0xf, 0xf, false);
    if (col < image_cols) {   // image_cols and seg_cols are even: both dwords of the pair lie in one panel
      const uint32_t i = col + gap * __umulhi(col, m.seg_magic);
      lds_x[i] = lo[k];
      lds_x[i + 1] = lo[k] >> 16 | next << 16;
    }
  }
}
// The same for x at 8-byte aligned addresses and rows of whole 4 columns: thread t of a round handles 4 columns, with one load and one
// store.  v: the 4 columns; hi: the one behind them, loaded by the last lane of a wavefront only.
template <int kThreads, int kXRegs, bool kCoherent>   // 2 * kXRegs registers as above, kXRegs x kThreads x 4 columns per round
__device__ __forceinline__ void issue_activations_wide(const DevMat& m, const uint16_t* __restrict__ x, uint32_t first, int tid, uint32_t (&v)[2 * kXRegs],
                                                       uint32_t (&hi)[2 * kXRegs]) {
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    v[2 * k] = v[2 * k + 1] = hi[k] = 0u;
    if (first + k * kThreads * 4 >= m.cols) continue;   // (the same for all)
    const uint32_t col = first + 4 * (k * kThreads + tid);
    if (col < m.cols) {
      if constexpr (kCoherent) {
        const uint64_t w = __hip_atomic_load((__attribute__((address_space(1))) const uint64_t*)(x + col), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v[2 * k] = (uint32_t)w;
        v[2 * k + 1] = (uint32_t)(w >> 32);
      } else {
        const uint2 w = global_load((const uint2*)(x + col));
        v[2 * k] = w.x;
        v[2 * k + 1] = w.y;
      }
    }
    if ((tid & 63) == 63 && col + 4 < m.cols) hi[k] = x_load<kCoherent>(x + col + 4);
  }
}
template <int kThreads, int kXRegs>
__device__ __forceinline__ void commit_activations_wide(const DevMat& m, uint32_t first, int tid, const uint32_t (&v)[2 * kXRegs], const uint32_t (&hi)[2 * kXRegs],
                                                        uint32_t* lds_x, uint32_t image_cols) {
  const uint32_t gap = m.x_span - m.seg_cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    if (first + k * kThreads * 4 >= image_cols) continue;
    const uint32_t col = first + 4 * (k * kThreads + tid), lo = v[2 * k], up = v[2 * k + 1];
    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)hi[k], (int)lo, 0x130, 0xf, 0xf, false);   // the next lane's first two
    if (col < image_cols)   // (image_cols and seg_cols are multiples of 16: the 4 columns lie in one panel)
      *(u32x4*)&lds_x[col + gap * __umulhi(col, m.seg_magic)] = u32x4{lo, __builtin_amdgcn_alignbyte(up, lo, 2), up, __builtin_amdgcn_alignbyte(next, up, 2)};
  }
}
template <int kThreads, int kDwords = 1>   // kDwords: dwords per column of the image (2: two rows of packed weights)
__device__ __forceinline__ void zero_activation_gaps(const DevMat& m, int tid, uint32_t* lds_x, uint32_t n_slots) {
  const uint32_t gap = m.x_span - m.seg_cols;
  constexpr uint32_t kGap = 16 * kDwords;
  if (gap)   // gap is 16 columns
    for (uint32_t i = tid; i < n_slots * kGap; i += kThreads) lds_x[kDwords * ((i / kGap) * m.x_span + m.seg_cols) + i % kGap] = 0u;
  for (uint32_t i = kDwords * n_slots * m.x_span + tid; i < kDwords * m.x_dwords; i += kThreads) lds_x[i] = 0u;
}

// One chunk = 4 codes per lane.  xa = LDS byte address of the activation pair of the lane's next code, minus 4 bytes
// per code consumed since the start of the piece; code k of the piece therefore reads at xa + 4 k, and the constant
// part goes into the instruction's offset field.  A single advances the lane by one column (already counted by the
// 4 k), a pair by one more.  The dictionary sits at LDS address 0, so a code's word offset is its address.
// Per chunk and lane: 4 dictionary words, 4 activation pairs, 4 v_dot2_f32_bf16 into two accumulators.
// xa + 4 * pair as one instruction.  Written out because the compiler otherwise keeps a running count of the pairs and
// forms every address from it with a second instruction: a shorter dependency chain, but a quarter more vector
// instructions per code.
__device__ __forceinline__ uint32_t advance_by_pair(uint32_t pair, uint32_t xa) {
  uint32_t r;
  asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(r) : "v"(pair), "v"(xa));
  return r;
}
__device__ __forceinline__ uint32_t advance_by_wide_pair(uint32_t pair, uint32_t xa) {   // xa + 8 * pair: an image of 8 bytes per column
  uint32_t r;
  asm("v_lshl_add_u32 %0, %1, 3, %2" : "=v"(r) : "v"(pair), "v"(xa));
  return r;
}

// In two halves, so that the reads of the next chunk can be issued ahead of the dot products of this one (left to
// itself the compiler finishes a chunk before it requests anything of the next: one LDS round trip per chunk that a
// wavefront with few neighbours cannot hide).
template <int kCode0>
__device__ __forceinline__ void chunk4_read(uint2 c, uint32_t& xa, uint32_t (&w)[4], uint32_t (&x)[8]) {
  w[0] = lds_read32(word_offset_lo(c.x));
  w[1] = lds_read32(word_offset_hi(c.x));
  w[2] = lds_read32(word_offset_lo(c.y));
  w[3] = lds_read32(word_offset_hi(c.y));
  x[0] = lds_read32_off<4 * kCode0>(xa);
  xa = advance_by_pair(is_pair_lo(c.x), xa);
  x[1] = lds_read32_off<4 * kCode0 + 4>(xa);
  xa = advance_by_pair(is_pair_hi(c.x), xa);
  x[2] = lds_read32_off<4 * kCode0 + 8>(xa);
  xa = advance_by_pair(is_pair_lo(c.y), xa);
  x[3] = lds_read32_off<4 * kCode0 + 12>(xa);
  xa = advance_by_pair(is_pair_hi(c.y), xa);
}
__device__ __forceinline__ void chunk4_dot(const uint32_t (&w)[4], const uint32_t (&x)[8], float& a0, float& a1) {
  a0 = dot2(w[0], x[0], a0);
  a1 = dot2(w[1], x[1], a1);
  a0 = dot2(w[2], x[2], a0);
  a1 = dot2(w[3], x[3], a1);
}

// The same for a matrix of packed 4-bit weights.  A dictionary word holds the entry's four weights as fp8 (e4m3 holds
// -8..7 exactly; two zeros after a single byte), one activation dword holds the two columns of a byte: code k reads the
// dwords at xa + 4 k and the next one, and two conversions give the bf16 pairs for two dot products.
__device__ __forceinline__ float dot2_fp8(uint32_t w, bool high, uint32_t x, float acc) {
  const bf16x2 wb = high ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
  return __builtin_amdgcn_fdot2_f32_bf16(wb, __builtin_bit_cast(bf16x2, x), acc, false);
}
template <int kCode0>
__device__ __forceinline__ void chunk4_packed_read(uint2 c, uint32_t& xa, uint32_t (&w)[4], uint32_t (&x)[8]) {
  w[0] = lds_read32(word_offset_lo(c.x));
  w[1] = lds_read32(word_offset_hi(c.x));
  w[2] = lds_read32(word_offset_lo(c.y));
  w[3] = lds_read32(word_offset_hi(c.y));
  x[0] = lds_read32_off<4 * kCode0>(xa);
  x[1] = lds_read32_off<4 * kCode0 + 4>(xa);
  xa = advance_by_pair(is_pair_lo(c.x), xa);
  x[2] = lds_read32_off<4 * kCode0 + 4>(xa);
  x[3] = lds_read32_off<4 * kCode0 + 8>(xa);
  xa = advance_by_pair(is_pair_hi(c.x), xa);
  x[4] = lds_read32_off<4 * kCode0 + 8>(xa);
  x[5] = lds_read32_off<4 * kCode0 + 12>(xa);
  xa = advance_by_pair(is_pair_lo(c.y), xa);
  x[6] = lds_read32_off<4 * kCode0 + 12>(xa);
  x[7] = lds_read32_off<4 * kCode0 + 16>(xa);
  xa = advance_by_pair(is_pair_hi(c.y), xa);
}
__device__ __forceinline__ void chunk4_packed_dot(const uint32_t (&w)[4], const uint32_t (&x)[8], float& a0, float& a1) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    a0 = dot2_fp8(w[k], false, x[2 * k], a0);
    a1 = dot2_fp8(w[k], true, x[2 * k + 1], a1);
  }
}

// LDS image of one activation row for packed weights: dword (panel * x_span + c) = the two activations of byte column
// panel * seg_cols + c, zero past the end of the row.  Thread t of a round handles dword first + k * kThreads + t.
template <bool kAligned, int kThreads, int kXRegs, bool kCoherent = false>
__device__ __forceinline__ void issue_activations_packed(const DevMat& m, const uint16_t* __restrict__ x, uint32_t first, int tid,
                                                         uint32_t (&v)[kXRegs]) {
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    const uint32_t j = first + k * kThreads + tid;
    v[k] = 0u;
    if (first + k * kThreads >= m.cols) continue;
    if (kAligned) v[k] = j < m.cols ? x_load<kCoherent>((const uint32_t*)x + j) : 0u;   // x is 4-byte aligned
    else v[k] = j < m.cols ? x_load<kCoherent>(x + 2 * j) | x_load<kCoherent>(x + 2 * j + 1) << 16 : 0u;
  }
}
template <int kThreads, int kXRegs>
__device__ __forceinline__ void commit_activations_packed(const DevMat& m, uint32_t first, int tid, const uint32_t (&v)[kXRegs], uint32_t* lds_x,
                                                          uint32_t image_cols) {
  const uint32_t gap = m.x_span - m.seg_cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    if (first + k * kThreads >= image_cols) continue;
    const uint32_t j = first + k * kThreads + tid;
    if (j < image_cols) lds_x[j + gap * __umulhi(j, m.seg_magic)] = v[k];
  }
}

// Two activation rows of packed weights.  The image holds two dwords per byte column: the two activations of that byte
// in row 0, then those in row 1; a code reads the 16 bytes of its byte column and the next one at xa + 8 k, and each
// half of the dictionary word, converted once, meets the dword of either row: a0 collects row 0, a1 row 1.
template <int kCode0>
__device__ __forceinline__ void chunk4_packed_two_read(uint2 c, uint32_t& xa, uint32_t (&w)[4], uint64_t (&x)[8]) {
  w[0] = lds_read32(word_offset_lo(c.x));
  w[1] = lds_read32(word_offset_hi(c.x));
  w[2] = lds_read32(word_offset_lo(c.y));
  w[3] = lds_read32(word_offset_hi(c.y));
  x[0] = lds_read64_off<8 * kCode0>(xa);
  x[1] = lds_read64_off<8 * kCode0 + 8>(xa);
  xa = advance_by_wide_pair(is_pair_lo(c.x), xa);
  x[2] = lds_read64_off<8 * kCode0 + 8>(xa);
  x[3] = lds_read64_off<8 * kCode0 + 16>(xa);
  xa = advance_by_wide_pair(is_pair_hi(c.x), xa);
  x[4] = lds_read64_off<8 * kCode0 + 16>(xa);
  x[5] = lds_read64_off<8 * kCode0 + 24>(xa);
  xa = advance_by_wide_pair(is_pair_lo(c.y), xa);
  x[6] = lds_read64_off<8 * kCode0 + 24>(xa);
  x[7] = lds_read64_off<8 * kCode0 + 32>(xa);
  xa = advance_by_wide_pair(is_pair_hi(c.y), xa);
}
__device__ __forceinline__ void chunk4_packed_two_dot(const uint32_t (&w)[4], const uint64_t (&x)[8], float& a0, float& a1) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bf16x2 first = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[k], 1.0f, false);   // the weights of the code's first byte
    const bf16x2 second = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[k], 1.0f, true);   // of its second byte (zeros after a single)
    a0 = __builtin_amdgcn_fdot2_f32_bf16(first, __builtin_bit_cast(bf16x2, (uint32_t)x[2 * k]), a0, false);
    a1 = __builtin_amdgcn_fdot2_f32_bf16(first, __builtin_bit_cast(bf16x2, (uint32_t)(x[2 * k] >> 32)), a1, false);
    a0 = __builtin_amdgcn_fdot2_f32_bf16(second, __builtin_bit_cast(bf16x2, (uint32_t)x[2 * k + 1]), a0, false);
    a1 = __builtin_amdgcn_fdot2_f32_bf16(second, __builtin_bit_cast(bf16x2, (uint32_t)(x[2 * k + 1] >> 32)), a1, false);
  }
}
template <int kThreads, int kXRegs>
__device__ __forceinline__ void commit_activations_packed_two(const DevMat& m, uint32_t first, int tid, const uint32_t (&r0)[kXRegs],
                                                              const uint32_t (&r1)[kXRegs], uint32_t* lds_x, uint32_t image_cols) {
  const uint32_t gap = m.x_span - m.seg_cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    if (first + k * kThreads >= image_cols) continue;
    const uint32_t j = first + k * kThreads + tid;
    if (j < image_cols) {
      const uint32_t i = 2 * (j + gap * __umulhi(j, m.seg_magic));
      lds_x[i] = r0[k];
      lds_x[i + 1] = r1[k];
    }
  }
}

// Two activation rows (batch 2).  The image holds one dword per column, (x0[c], x1[c]); a code reads the dwords of its
// column and of the next one (the reads of chunk4_packed_read), two byte permutes put each row's pair together, and one
// dot product per row follows: a0 collects row 0, a1 row 1.
__device__ __forceinline__ void chunk4_two_dot(const uint32_t (&w)[4], const uint32_t (&x)[8], float& a0, float& a1) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    a0 = dot2(w[k], __builtin_amdgcn_perm(x[2 * k + 1], x[2 * k], 0x05040100u), a0);   // (x0[c], x0[c + 1])
    a1 = dot2(w[k], __builtin_amdgcn_perm(x[2 * k + 1], x[2 * k], 0x07060302u), a1);   // (x1[c], x1[c + 1])
  }
}
// Thread t of a round handles the columns (2 j, 2 j + 1), j = first_pair + k * kThreads + t, of both rows.
template <bool kAligned, int kThreads, int kXRegs, bool kCoherent = false>   // kAligned: both rows start 4-byte aligned and cols is even
__device__ __forceinline__ void issue_activations_two(const DevMat& m, const uint16_t* __restrict__ x, uint32_t first_pair, int tid,
                                                      uint32_t (&r0)[kXRegs], uint32_t (&r1)[kXRegs]) {
  const uint16_t* x1 = x + m.cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    const uint32_t j = first_pair + k * kThreads + tid, col = 2 * j;
    r0[k] = r1[k] = 0u;
    if (2 * (first_pair + k * kThreads) >= m.cols) continue;
    if (kAligned) {
      r0[k] = col < m.cols ? x_load<kCoherent>((const uint32_t*)x + j) : 0u;
      r1[k] = col < m.cols ? x_load<kCoherent>((const uint32_t*)x1 + j) : 0u;
    } else {
      r0[k] = (col < m.cols ? x_load<kCoherent>(x + col) : 0u) | (col + 1 < m.cols ? x_load<kCoherent>(x + col + 1) << 16 : 0u);
      r1[k] = (col < m.cols ? x_load<kCoherent>(x1 + col) : 0u) | (col + 1 < m.cols ? x_load<kCoherent>(x1 + col + 1) << 16 : 0u);
    }
  }
}
template <int kThreads, int kXRegs>
__device__ __forceinline__ void commit_activations_two(const DevMat& m, uint32_t first_pair, int tid, const uint32_t (&r0)[kXRegs],
                                                       const uint32_t (&r1)[kXRegs], uint32_t* lds_x, uint32_t image_cols) {
  const uint32_t gap = m.x_span - m.seg_cols;
#pragma unroll
  for (int k = 0; k < kXRegs; ++k) {
    if (2 * (first_pair + k * kThreads) >= image_cols) continue;
    const uint32_t col = 2 * (first_pair + k * kThreads + tid);
    if (col < image_cols) {   // image_cols and seg_cols are even: both columns lie in one panel
      const uint32_t i = col + gap * __umulhi(col, m.seg_magic);
      lds_x[i] = (r0[k] & 0xFFFFu) | r1[k] << 16;
      lds_x[i + 1] = r0[k] >> 16 | (r1[k] & 0xFFFF0000u);
    }
  }
}

// Containers with runs of up to 4 bytes (one activation row).  The dictionary image has one dword (two bf16 weights) per
// slot; an entry of 3 or 4 bytes takes two slots, so a code reads the two dwords at its slot (for a shorter entry the
// second one belongs to the next entry and is dropped), the activation pairs of its column and of the column two
// further on, and multiplies both; its run length follows from the code's place in the sorted code space.
// xa = LDS byte address of the activation pair of the lane's next column.
struct LongClasses {
  uint32_t class2, class3;
};
__device__ __forceinline__ void code_long_dot(uint32_t code, const LongClasses& cl, uint32_t& xa, float& a0, float& a1) {
  const uint32_t da = long_slot(code, cl.class2) << 2;
  const uint32_t w0 = lds_read32(da), w1 = lds_read32_off<4>(da);
  const uint32_t x0 = lds_read32(xa), x1 = lds_read32_off<8>(xa);
  a0 = dot2(w0, x0, a0);
  a1 = dot2(code >= cl.class2 ? w1 : 0u, x1, a1);
  xa += 4u * long_run_length(code, cl.class2, cl.class3);
}
__device__ __forceinline__ void chunk4_long(uint2 c, const LongClasses& cl, uint32_t& xa, float& a0, float& a1) {
  code_long_dot(c.x & 0xFFFFu, cl, xa, a0, a1);
  code_long_dot(c.x >> 16, cl, xa, a0, a1);
  code_long_dot(c.y & 0xFFFFu, cl, xa, a0, a1);
  code_long_dot(c.y >> 16, cl, xa, a0, a1);
}

// Sum of the four panel lanes of each row: afterwards every lane l holds the sum over lanes l % 16 + {0, 16, 32, 48}.
__device__ __forceinline__ float sum_over_panels(float v) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

// The gated product of a feed-forward block: silu(gate) * up, silu(g) = g / (1 + exp(-g)).
__device__ __forceinline__ float silu_times(float gate, float up) { return gate / (1.f + __expf(-gate)) * up; }

// Fused decode + dequantize + matrix-vector product for one or two activation rows (kB) and up to kMaxMulti matrices
// (kMaxStep when the jobs come from a prepared step's table).
//
// The launch's work is the line of all bands (16 rows each) of all matrices, each band weighted by its number of
// weights; workgroup g takes the bands whose middle lies in the g-th equal share of that line, so a workgroup serves a
// contiguous range of whole bands of one matrix after the other.  Inside a matrix the units of those bands are
// contiguous in the code stream and are cut into one contiguous run per wavefront.  A wavefront owns every band that
// lies entirely inside its run (it scales and stores those rows itself); a band it shares with its neighbours goes to
// one of two partial-sum slots in LDS, and after a workgroup barrier the slots of a band are added in wavefront order,
// so the result does not depend on timing.
// kStaged: the jobs form stages (MatvecArgs::stage_first); the workgroups take the stages in turn, each one's bands cut
// into equal shares as above, with a grid-wide hand-over between two stages; the dictionary stays in LDS across them.
// kOne: every workgroup serves one job (a launch whose matrices have whole workgroups), found in the arguments' map: no loop over jobs,
// which the compiler prepares for with some 200 instructions ahead of the first load.  A small launch is bound by what its wavefronts do
// before they decode: every instruction of a wavefront with one neighbour on its SIMD is 2 to 4 ns, a round trip to memory only 160.
// 2048 x 2048, batch 1, us after the first wavefront's start, before -> now (no search and no 64-bit divisions either, 4 columns of x to a
// load, the dictionary through request_to_lds, behind the first codes): its job known 1.5 -> 0.6, everything requested 3.7 -> 2.4, decode
// from 6.1 -> 3.9, end of a pass 10.1 -> 8.7 (7.7 with marks, see kSplit); one LLaMA-3.2-1B layer 18.3 -> 17.2.
// kShared: a staged step whose workgroups may share bands (shared_share).  A stage's largest share is then its units over the workgroups, rounded up, where
// whole bands of 3 or 8 units leave some workgroups 6 units of 3.75, or 8 of 6.  us, whole bands -> shared, four LLaMA-3.2-3B layers in 16 stages 199.0 ->
// 192.8, batch 2 209 -> 200, four 1B layers 165.5 -> 158.2; packed ones gained nothing (batch 1 160 -> 158, batch 2 87.3 -> 87.6, 1B 107.1 -> 107.7).  A kernel of its own:
// with the choice made inside it, steps that share nothing lost 3 % (four layers of 1024 x 2048, batch 2, 122 -> 126).  A shared band's sum is no longer one
// sum in double: each workgroup's part is scaled in double and rounded, and the two are added in fp32, so its low bits depend on where the outputs
// lie (which decides whether bands are shared).  Relative error of 15 staged steps of up to 4 layers against 64 bits, in the 2-norm: 5.45e-8, whole bands (longer
// runs of fp32 sums in a wavefront) 5.84e-8, none of them further off; rounded before and after the scale, as whole sums are, 5.51e-8.
template <int kPiece, int kWaves, bool kPacked, int kB, bool kLong = false, bool kStaged = false, bool kOne = false, bool kShared = false>
__global__ __launch_bounds__(kWaves * 64, 1) void k_matvec(MatvecArgs a) {
  static_assert(kB == 1 || kB == 2, "one activation row or two");
  static_assert(!kShared || (kStaged && !kPacked), "workgroups share bands in staged steps of one-weight-per-byte matrices");
  static_assert(!kLong || (kB == 1 && !kPacked), "runs of 3 and 4 bytes: one activation row of one-weight-per-byte matrices");
  constexpr int kImage = kPacked && kB == 2 ? 2 : 1;   // dwords of the activation image per column
  // kSplit: a share of few units is cut into equal runs of chunks, wherever a run starts inside a unit.  (Whole units leave wavefronts
  // idle: a 2048 x 2048 matrix gives a workgroup two units for its eight wavefronts.)  Where a lane stands at the start of such a run the
  // matrix's marks say, to within 7 chunks that are counted while the dictionary is on its way (request_place).  (Counted from the codes of
  // the whole unit, each wavefront its part and the counts exchanged through LDS, it took as long again as the decode and paid in shares of up
  // to two units: 2048 x 2048 8.74 -> 7.67 us, 3072 x 3072 10.7 -> 9.1.)
  // What is left of the cost is the sums of bands that are shared.  It pays where whole units leave a quarter of the wavefronts' time idle (of 8 wavefronts:
  // 1 to 6 units, 9 to 12, 17 and 18); packed ones, which fewer chunks keep busier, where they leave half of the wavefronts without any.  us, whole units -> split, batch 1: 3 units
  // (3072 x 3072) 10.7 -> 9.1, 6 units (8192 x 3072) 12.0 -> 11.8, 9 units 15.0 -> 13.8, 12 units 15.9 -> 15.5, 14 units (8192 x 7168) 16.3 -> 16.7, 14
  // to 16 (a LLaMA-3.2-1B layer) 17.1 -> 17.9, 18 units (24576 x 3072) 20.8 -> 19.3; batch 2: 6 units 13.8 -> 13.3, 12 units 19.1 -> 18.1, 18 units 25.2 -> 22.7; packed: 6 units 9.7 -> 9.5, batch 2 11.0 -> 10.5; 9
  // units 10.9 -> 11.5, batch 2 12.3 -> 12.8.
  constexpr bool kSplit = !kLong;
  // Packed weights are bound by issue and the LDS pipe and gain most from wavefronts that end together (see pace; us, eight LLaMA-3.2-3B layers 87 -> 83,
  // one 17.7 -> 16.0, batch 2 104 -> 98, four in 16 stages 171 -> 164); plain ones in large launches 1 % (eight layers 154 -> 153, staged at
  // batch 2 221 -> 218), where a workgroup serves one matrix they lose as much (a 1B layer 17.2 -> 17.5, a 3B layer batch 2 26.1 -> 26.8).
  constexpr bool kPaced = kPacked || (!kOne && (kB == 2 || !kStaged));
  constexpr int kThreads = kWaves * 64, kXRegs = 64 / kWaves;
  if constexpr (!kStaged) touch_arguments();
  extern __shared__ uint4 lds4[];
  uint32_t* lds_dict = (uint32_t*)lds4;
  uint32_t* lds_x = (uint32_t*)((uint8_t*)lds4 + a.x_off);
  float* slot_val = (float*)((uint8_t*)lds4 + a.slot_off);           // [2 * kWaves][kB][16]
  int* slot_band = (int*)(slot_val + 2 * kWaves * kB * 16);          // [2 * kWaves]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t* staged = nullptr;
  const uint32_t n_stages = kStaged ? a.n_stages : 1u;
  constexpr uint32_t kNoStage = 0xFFFFFFFFu;
  uint32_t wait_for = kNoStage;   // staged: the number of stages whose outputs this workgroup has yet to wait for
  bool lds_used = false;          // an earlier matrix may still be in work
  // Where the workgroup stands: a stage (the only one unless kStaged), a job of it, its share of the stage's cost line.
  struct Cursor {
    uint32_t stage;
    int i, end;
    uint32_t lo, hi;
  };
  auto enter_stage = [&](Cursor& c) {
    const int first = kStaged ? (int)((const_u32*)a.stage_first)[c.stage] : 0;
    c.end = kStaged ? (int)((const_u32*)a.stage_first)[c.stage + 1] : a.n;
    if (kOne || (kStaged && a.by_workgroup)) {
      c.lo = (kStaged ? c.stage * a.share : 0u) + blockIdx.x;
      c.hi = c.lo + 1;
      if constexpr (kOne) {
        c.i = mapped_job(a);
        return;
      }
    } else if constexpr (kStaged) {
      const uint32_t cost_first = cost_at(a, first);
      const uint64_t total = cost_at(a, c.end) - cost_first;
      c.lo = cost_first + (uint32_t)(total * blockIdx.x / gridDim.x);
      c.hi = cost_first + (uint32_t)(total * (blockIdx.x + 1) / gridDim.x);
    } else {
      even_share(a, c.lo, c.hi);
    }
    c.i = first_job(a, first, c.end, c.lo, lane);
  };
  auto settle = [&](Cursor& c) {   // moves on, over stages the workgroup has no share in, to a job it has; false at the end
    while (c.i >= c.end || cost_at(a, c.i) >= c.hi) {
      if (++c.stage >= n_stages) return false;
      enter_stage(c);
    }
    return true;
  };
  // kStaged: jobs are looked up ahead, so that of the chain table entry -> unit offsets -> code chunks -> decode nothing but
  // the activations is left behind the hand-over between two stages: while one job is staged, the entry of the job after
  // the next and the offsets of the next one are requested; when a wavefront has decoded its run it plans its run of the
  // next job and requests the run's first chunk; the rest of the first piece follows when the workgroup has announced
  // itself.  (Requested together, ahead of the announcement, they hold it up: the next matrix's pages are new to the
  // compute unit's address translation, and whatever is issued behind a miss waits for it.)
  // (Looked up between two stages the chain took 4 to 6 us of every stage of a LLaMA-3.2-3B layer: every stage's matrices
  // are new to the caches and to address translation.)
  constexpr uint32_t kEntryDwords = sizeof(StepEntry) / 4;
  auto request_entry = [&](int i) { return global_load((const uint32_t*)(a.table + i) + min((uint32_t)lane, kEntryDwords - 1)); };
  auto open_entry = [&](uint32_t entry, Job& job, DevMat& m) {   // entry: dword k in lane k
    uint32_t w[kEntryDwords];
#pragma unroll
    for (uint32_t k = 0; k < kEntryDwords; ++k) w[k] = __builtin_amdgcn_readlane(entry, k);
    StepEntry v;
    __builtin_memcpy(&v, w, sizeof v);
    m = v.m;
    job.m = nullptr;
    job.x = v.x;
    job.y = v.y;
  };
  // The unit offsets of a share of few units sit in the lanes: lane k has that of unit k, the lanes behind them the end.
  constexpr uint32_t kLaneUnits = 64;
  auto request_offsets = [&](const DevMat& m, uint32_t share_lo, uint32_t share_hi) {
    const uint32_t n_units = share_hi - share_lo;
    return n_units < kLaneUnits ? global_load(m.uoff + share_lo + min((uint32_t)lane, n_units)) : 0u;
  };
  // The units of job i that a cursor's share holds.
  auto share_of_units = [&](const DevMat& m, const Cursor& c, uint32_t& share_lo, uint32_t& share_hi) {
    if constexpr (kShared) {
      shared_share(a.u.cost_long[c.i], a.u.cost_long[c.i + 1], m.n_bands, m.n_quads, c.lo, share_lo, share_hi);
    } else {
      uint32_t band_lo, band_hi;
      share_of_bands(a, kOne || (kStaged && a.by_workgroup), m, c.i, c.lo, c.hi, band_lo, band_hi);
      share_lo = band_lo * m.n_quads;
      share_hi = band_hi * m.n_quads;
    }
  };
  // This wavefront's run of a job: the chunks [c0, c_end) of the units [u0, u1).
  uint32_t uoff_lane = 0;
  uint32_t unit_lo = 0, u0 = 0, u1 = 0, c0 = 0, c_end = 0, unit_start = 0, passed = 0;   // (passed: columns of its first unit that earlier wavefronts take)
  bool in_lanes = false, head_shared = false, tail_shared = false;   // the run starts / ends inside a unit
  uint2 cwa[kPiece], cwb[kPiece];
  Place place;
  auto offset_of = [&](const DevMat& m, uint32_t u) {
    if (in_lanes) return (uint32_t)__builtin_amdgcn_readlane(uoff_lane, u - unit_lo);
    return unit_offset(m, u);
  };
  // The chunks of the run come in pieces of at most kPiece that never straddle a unit (a unit, or the part of it that
  // lies in the run, is cut into equal pieces); two register sets alternate and every piece issues exactly kPiece
  // loads (those past its end repeat its last chunk), so the loads of the next piece are in flight while this one is
  // worked on.  A piece runs as straight-line code: the LDS reads of later chunks overlap the dot products of earlier ones.
  uint32_t wu = 0, wc = 0, w_left = 0, w_base = 0, w_rem = 0;
  bool w_ends = false;   // the unit in work ends inside the run
  auto next_piece = [&](const DevMat& m, uint32_t& start, uint32_t& n, bool& ends) {
    if (w_left == 0) {
      if (wu == u1) {
        n = 0;
        ends = false;
        start = wc;
        return;
      }
      const uint32_t unit_end = offset_of(m, wu + 1);
      w_ends = unit_end <= c_end;
      const uint32_t len = min(unit_end, c_end) - wc;
      w_left = (len + kPiece - 1) / kPiece;
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
  auto load_piece = [&](const DevMat& m, uint2 (&cw)[kPiece], uint32_t start, uint32_t n, bool all = true, bool only_first = false) {
    const uint32_t last = min(start + max(n, 1u) - 1, c_end - 1);
#pragma unroll
    for (int k = 0; k < kPiece; ++k)
      if (all || (k == 0) == only_first) cw[k] = load_chunk(m.codes, min(start + k, last), lane);
  };
  uint32_t sa = 0, na = 0, sb, nb;
  bool ea = false, eb;
  // Cuts the share of a job, its units [share_lo, share_hi), and requests the first piece of the wavefront's run (ahead of the staging of
  // dictionary and activations, so that a small launch does not wait for device memory twice in a row).
  auto plan_run = [&](const DevMat& m, uint32_t share_lo, uint32_t share_hi) {
    unit_lo = share_lo;
    const uint32_t n_units = share_hi - share_lo;
    in_lanes = n_units < kLaneUnits;
    const bool split = kSplit && in_lanes && (kPacked ? 2 * n_units <= kWaves : 4 * n_units <= 3 * kWaves * ((n_units + kWaves - 1) / kWaves));
    // (values of the two ways meet in local variables and are assigned once: assigned in each branch, the compiler keeps
    // them in memory)
    uint32_t first = unit_lo + (uint32_t)((uint64_t)n_units * wave / kWaves), end = unit_lo + (uint32_t)((uint64_t)n_units * (wave + 1) / kWaves);
    uint32_t lo = 0, hi = 0, start = 0;
    bool head = false, tail = false;
    if (split) {   // few units per wavefront: see kSplit above
      const uint32_t all_lo = offset_of(m, unit_lo), all_n = offset_of(m, unit_lo + n_units) - all_lo;
      lo = all_lo + all_n * wave / kWaves;
      hi = all_lo + all_n * (wave + 1) / kWaves;
      const uint64_t lanes = (2ull << n_units) - 1;   // lanes 0 .. n_units hold the offsets
      first = unit_lo + (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(uoff_lane <= lo) & lanes) - 1;
      const uint32_t last = unit_lo + (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(uoff_lane < max(hi, lo + 1)) & lanes) - 1;
      end = lo < hi ? last + 1 : first;
      start = offset_of(m, first);
      head = lo < hi && lo > start;
      tail = lo < hi && hi < offset_of(m, last + 1);
    } else if (first < end) {
      lo = offset_of(m, first);
      hi = offset_of(m, end);
    }
    u0 = first;
    u1 = end;
    c0 = lo;
    c_end = hi;
    unit_start = start;
    head_shared = head;
    tail_shared = tail;
    wu = u0;
    wc = c0;
    w_left = 0;
    na = 0;
    ea = false;
    if (u0 < u1) next_piece(m, sa, na, ea);
  };
  Cursor at, next;   // (next: one job further, kStaged only)
  at.stage = 0;
  enter_stage(at);
  uint32_t arrived = 0;   // kStaged: the stages this workgroup has announced to have behind it
  uint32_t entry_at = 0, entry_next = 0, entry_later = 0;
  bool have = kOne || settle(at), have_next = false, have_later = false, planned = false;
  if (kStaged && have) {
    entry_at = request_entry(at.i);
    next = at;
    ++next.i;
    have_next = settle(next);
    if (have_next) entry_next = request_entry(next.i);
  }
  Cursor later;
  auto look_further = [&] {
    if constexpr (kStaged) {
      later = next;
      ++later.i;
      have_later = have_next && settle(later);
      if (have_later) entry_later = request_entry(later.i);
    }
  };
  auto advance = [&] {
    if constexpr (kStaged) {
      at = next;
      next = later;
      have = have_next;
      have_next = have_later;
      entry_at = entry_next;
      entry_next = entry_later;
    } else {
      ++at.i;
      have = settle(at);
    }
  };
  while (have) {
    Job job;
    DevMat m;
    if constexpr (kStaged) open_entry(entry_at, job, m);
    else fetch_job(a, at.i, job, m);
    uint32_t share_lo, share_hi;
    share_of_units(m, at, share_lo, share_hi);
    if (kStaged && at.stage > arrived) {
      wait_for_stores();
      stage_arrive(a, at.stage);
      wait_for = at.stage;
      arrived = at.stage;
    }
    if (share_lo >= share_hi) {
      if constexpr (kOne) return;
      look_further();
      planned = false;
      advance();
      continue;
    }
    const bool new_dict = m.dict_bf16 != staged;
    staged = m.dict_bf16;
    const uint32_t nq = m.n_quads, n_slots = nq * kUnitPanels, image_cols = n_slots * m.seg_cols;
    // lane's panel inside a unit is lane >> 4; quad q adds 4 q panels
    const uint32_t xa_lane = lds_address(lds_x) + 4u * kImage * m.x_span * (uint32_t)(lane >> 4);
    const uint32_t xa_quad = 16u * kImage * m.x_span;
    const bool x_aligned = (kPacked || m.cols % 2 == 0) && ((uintptr_t)job.x % 4 == 0);   // (cols even: a second row is aligned like the first)
    const bool x_wide = !kPacked && kB == 1 && m.cols % 4 == 0 && (uintptr_t)job.x % 8 == 0;
    if (!planned) uoff_lane = request_offsets(m, share_lo, share_hi);
    {   // one activation row, or two: larger batches run the MFMA kernels
      const uint16_t* xb = job.x;
      float* yb = job.y;
      // Activations and dictionary are requested first: their addresses wait for nothing but the description.  (A further matrix's
      // dictionary goes to LDS when the one before it is no longer in use; in staged steps so does the first, see lds_arrived.)
      uint32_t xlo[kXRegs], xhi[kXRegs];
      auto request_activations = [&] {
        if constexpr (kPacked) {
          if (x_aligned) issue_activations_packed<true, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo);
          else issue_activations_packed<false, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo);
          if constexpr (kB == 2) {   // the second row starts 2 * cols activations later, aligned like the first
            if (x_aligned) issue_activations_packed<true, kThreads, kXRegs, kStaged>(m, xb + 2 * m.cols, 0, tid, xhi);
            else issue_activations_packed<false, kThreads, kXRegs, kStaged>(m, xb + 2 * m.cols, 0, tid, xhi);
          }
        } else if constexpr (kB == 2) {
          if (x_aligned) issue_activations_two<true, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo, xhi);
          else issue_activations_two<false, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo, xhi);
        } else {
          if (x_wide) issue_activations_wide<kThreads, kXRegs / 2, kStaged>(m, xb, 0, tid, xlo, xhi);
          else if (x_aligned) issue_activations<true, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo, xhi);
          else issue_activations<false, kThreads, kXRegs, kStaged>(m, xb, 0, tid, xlo, xhi);
        }
      };
      if constexpr (!kStaged) request_activations();   // (staged: they may still be in the making)
      const bool dict_first = !kStaged && new_dict && !lds_used;
      constexpr uint32_t kDictAhead = 4;   // rounds of the dictionary that are on their way while the unit offsets arrive; the others behind the first codes
      if (dict_first) request_to_lds(m.dict_bf16, m.dict_words / 4, lane, wave, kWaves, lds_dict, 0, kDictAhead);
      if (!planned) {
        plan_run(m, share_lo, share_hi);
        if (u0 < u1) load_piece(m, cwa, sa, na);
      } else if (u0 < u1) {
        load_piece(m, cwa, sa, na, false, false);
      }
      if (head_shared) request_place(m, unit_start, c0, lane, place);
      if (dict_first) request_to_lds(m.dict_bf16, m.dict_words / 4, lane, wave, kWaves, lds_dict, kDictAhead);
      if constexpr (kStaged) {   // while the other workgroups arrive
        if (head_shared) passed = columns_passed(place, unit_start, c0);
      }
      // the previous dictionary, activation image and slots are no longer in use; staged: nor is anyone still writing
      // the activations (the wait ends with the same barrier)
      if (kStaged && wait_for != kNoStage) {
        stage_wait(a, wait_for);
        wait_for = kNoStage;
      } else if (lds_used) {
        __syncthreads();
      }
      lds_used = true;
      if constexpr (kStaged) request_activations();
      if (new_dict && !dict_first) {
        request_to_lds(m.dict_bf16, m.dict_words / 4, lane, wave, kWaves, lds_dict);
        lds_arrived();
      }
      look_further();
      uint32_t uoff_next = 0, next_lo = 0, next_hi = 0;
      if (kStaged && have_next) {
        Job next_job;
        DevMat next_m;
        open_entry(entry_next, next_job, next_m);
        share_of_units(next_m, next, next_lo, next_hi);
        if (next_lo < next_hi) uoff_next = request_offsets(next_m, next_lo, next_hi);
      }
      {
        zero_activation_gaps<kThreads, kImage>(m, tid, lds_x, n_slots);
        if (tid < 2 * kWaves) slot_band[tid] = -1;
        if constexpr (kPacked && kB == 2) {
          commit_activations_packed_two<kThreads, kXRegs>(m, 0, tid, xlo, xhi, lds_x, image_cols);
          for (uint32_t first = kXRegs * kThreads; first < image_cols; first += kXRegs * kThreads) {
            if (x_aligned) {
              issue_activations_packed<true, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo);
              issue_activations_packed<true, kThreads, kXRegs, kStaged>(m, xb + 2 * m.cols, first, tid, xhi);
            } else {
              issue_activations_packed<false, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo);
              issue_activations_packed<false, kThreads, kXRegs, kStaged>(m, xb + 2 * m.cols, first, tid, xhi);
            }
            commit_activations_packed_two<kThreads, kXRegs>(m, first, tid, xlo, xhi, lds_x, image_cols);
          }
        } else if constexpr (kPacked) {
          commit_activations_packed<kThreads, kXRegs>(m, 0, tid, xlo, lds_x, image_cols);
          for (uint32_t first = kXRegs * kThreads; first < image_cols; first += kXRegs * kThreads) {
            if (x_aligned) issue_activations_packed<true, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo);
            else issue_activations_packed<false, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo);
            commit_activations_packed<kThreads, kXRegs>(m, first, tid, xlo, lds_x, image_cols);
          }
        } else if constexpr (kB == 2) {
          commit_activations_two<kThreads, kXRegs>(m, 0, tid, xlo, xhi, lds_x, image_cols);
          for (uint32_t first = kXRegs * kThreads; 2 * first < image_cols; first += kXRegs * kThreads) {
            if (x_aligned) issue_activations_two<true, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo, xhi);
            else issue_activations_two<false, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo, xhi);
            commit_activations_two<kThreads, kXRegs>(m, first, tid, xlo, xhi, lds_x, image_cols);
          }
        } else if (x_wide) {
          commit_activations_wide<kThreads, kXRegs / 2>(m, 0, tid, xlo, xhi, lds_x, image_cols);
          for (uint32_t first = 2 * kXRegs * kThreads; first < image_cols; first += 2 * kXRegs * kThreads) {
            issue_activations_wide<kThreads, kXRegs / 2, kStaged>(m, xb, first, tid, xlo, xhi);
            commit_activations_wide<kThreads, kXRegs / 2>(m, first, tid, xlo, xhi, lds_x, image_cols);
          }
        } else {
          commit_activations<kThreads, kXRegs>(m, 0, tid, xlo, xhi, lds_x, image_cols);
          for (uint32_t first = kXRegs * kThreads; 2 * first < image_cols; first += kXRegs * kThreads) {
            if (x_aligned) issue_activations<true, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo, xhi);
            else issue_activations<false, kThreads, kXRegs, kStaged>(m, xb, first, tid, xlo, xhi);
            commit_activations<kThreads, kXRegs>(m, first, tid, xlo, xhi, lds_x, image_cols);
          }
        }
        if (!kStaged && head_shared) passed = columns_passed(place, unit_start, c0);   // (last: requested after everything else)
      }
      if (dict_first) lds_arrived();
      __syncthreads();
      float slot_scale = 0.f;   // row scales of the bands in this wavefront's two slots: the first one's in lanes 0..31
      if (u0 < u1) {
        uint32_t q = u0 % nq, band = u0 / nq;
        bool whole = q == 0 && !head_shared;             // the current band started inside this wavefront's run
        float a0 = 0.f, a1 = 0.f;
        uint32_t xa = xa_lane + q * xa_quad;
        if (head_shared) xa += 4u * kImage * passed;
        // the scales of the band in work are requested when the band starts (the array is padded to whole bands)
        float scale = global_load(m.scales + band * kUnitRows + (lane & 15));
        auto finish_band = [&](bool complete) {
          // one activation row: a0 and a1 are two chains of the same sum; two rows: one sum each
          float v[kB];
          if constexpr (kB == 1) {
            v[0] = sum_over_panels(a0 + a1);
          } else {
            v[0] = sum_over_panels(a0);
            v[1] = sum_over_panels(a1);
          }
          if (complete) {
            const uint32_t row = band * kUnitRows + lane;
#pragma unroll
            for (int b = 0; b < kB; ++b) {
              if (a.gate_up) {   // lanes 2r, 2r + 1 hold the gate and the up row of output r
                const float t = v[b] * scale, other = __shfl_xor(t, 1);
                if (lane < 16 && !(lane & 1) && row + 1 < m.rows) y_store<kStaged>(yb + (size_t)b * (m.rows / 2) + row / 2, silu_times(t, other));
              } else if (lane < 16 && row < m.rows) {
                y_store<kStaged>(yb + (size_t)b * m.rows + row, v[b] * scale);
              }
            }
          } else {
            const int s = 2 * wave + (whole ? 1 : 0);   // slot 2w: band begun by an earlier wavefront; 2w + 1: band left unfinished
#pragma unroll
            for (int b = 0; b < kB; ++b)
              if (lane < 16) slot_val[(s * kB + b) * 16 + lane] = v[b];
            if (lane == 0) slot_band[s] = (int)band;
            slot_scale = (lane >= 32) == whole ? scale : slot_scale;
          }
        };
        auto run_piece = [&](const uint2 (&cw)[kPiece], uint32_t n, bool ends) {
          // kSets register sets: the operands of the next kSets - 1 chunks are read while one chunk is multiplied, so a
          // wavefront that works alone (a small launch, the tail of a stage) does not sit out an LDS round trip per chunk
          constexpr int kSets = kDotSets;
          uint32_t w[kSets][4];
          std::conditional_t<kImage == 2, uint64_t, uint32_t> x[kSets][8];
          auto read = [&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (kImage == 2) chunk4_packed_two_read<4 * k>(cw[k], xa, w[k % kSets], x[k % kSets]);
            else if constexpr (kPacked || kB == 2) chunk4_packed_read<4 * k>(cw[k], xa, w[k % kSets], x[k % kSets]);   // this dword and the next
            else chunk4_read<4 * k>(cw[k], xa, w[k % kSets], x[k % kSets]);
          };
          auto dot = [&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (kImage == 2) chunk4_packed_two_dot(w[k % kSets], x[k % kSets], a0, a1);
            else if constexpr (kPacked) chunk4_packed_dot(w[k % kSets], x[k % kSets], a0, a1);
            else if constexpr (kB == 2) chunk4_two_dot(w[k % kSets], x[k % kSets], a0, a1);
            else chunk4_dot(w[k % kSets], x[k % kSets], a0, a1);
          };
          auto straight = [&](auto nn) {   // a piece of nn chunks as straight-line code
            constexpr int kN = decltype(nn)::value;
            static_for<(kSets - 1 < kN ? kSets - 1 : kN)>([&](auto kk) { read(kk); });
            static_for<kN>([&](auto kk) {
              constexpr int k = decltype(kk)::value;
              if constexpr (k + kSets - 1 < kN) read(std::integral_constant<int, k + kSets - 1>{});
              dot(kk);
            });
          };
          if constexpr (kLong) {
            const LongClasses cl = {m.class2, m.class3};
            static_for<kPiece>([&](auto kk) {
              if ((uint32_t)decltype(kk)::value < n) chunk4_long(cw[decltype(kk)::value], cl, xa, a0, a1);
            });
          } else if (n == kPiece) {
            straight(std::integral_constant<int, kPiece>{});
          } else if (n == kPiece - 1) {
            straight(std::integral_constant<int, kPiece - 1>{});
          } else if (n == kPiece - 2) {
            straight(std::integral_constant<int, kPiece - 2>{});
          } else {   // shorter pieces: ends of shared units, narrow segments
            static_for<kPiece - 3>([&](auto kk) {
              if (n == (uint32_t)decltype(kk)::value + 1) straight(std::integral_constant<int, decltype(kk)::value + 1>{});
            });
          }
          if constexpr (!kLong) xa += 16 * kImage * n;   // (the long form keeps xa at the lane's column itself)
          if (ends) {   // every lane restarts at the first column of its next segment
            if (++q == nq) {
              const bool more = (band + 1) * nq < u1;
              finish_band(whole);
              q = 0;
              ++band;
              if (more) scale = global_load(m.scales + band * kUnitRows + (lane & 15));
              whole = true;
              a0 = 0.f;
              a1 = 0.f;
            }
            xa = xa_lane + q * xa_quad;
          }
        };
        while (na) {
          if constexpr (kPaced) pace(sa - c0, c_end - c0);
          next_piece(m, sb, nb, eb);
          load_piece(m, cwb, sb, nb);
          run_piece(cwa, na, ea);
          if constexpr (kPaced) pace(sb - c0, c_end - c0);
          next_piece(m, sa, na, ea);
          load_piece(m, cwa, sa, na);
          run_piece(cwb, nb, eb);
        }
        if constexpr (kPaced) __builtin_amdgcn_s_setprio(0);
        if (u1 % nq || tail_shared) finish_band(false);   // the run ends inside a band (a band that ends with the run was finished above)
      }
      planned = kStaged && next_lo < next_hi;
      if (planned) {
        Job next_job;
        DevMat next_m;
        open_entry(entry_next, next_job, next_m);
        uoff_lane = uoff_next;
        plan_run(next_m, next_lo, next_hi);
        if (u0 < u1) load_piece(next_m, cwa, sa, na, false, true);
        // a band of the next stage that this workgroup begins and another ends: both add to its outputs, from zero on (nobody reads or
        // writes these in this stage, and the arrival after it waits for these stores too)
        if constexpr (kShared) {
          const uint32_t row = next_hi / next_m.n_quads * kUnitRows + (uint32_t)lane;
          if (next_hi % next_m.n_quads && wave == 0 && lane < (int)kUnitRows && row < next_m.rows)
#pragma unroll
            for (int b = 0; b < kB; ++b) y_store<true>(next_job.y + (size_t)b * next_m.rows + row, 0.f);
        }
      }
      __syncthreads();
      // Combine the shared bands: the first slot of a band adds the later slots of the same band in slot order.  Every
      // wavefront sees to its own two slots, whose row scales it still holds; lanes are (slot, activation row, row).
      {
        const int slots = lane < 2 * kWaves ? slot_band[lane] : -1;
        static_assert(2 * kWaves <= 32, "a bit per slot");
        uint32_t same[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int band = __builtin_amdgcn_readlane(slots, 2 * wave + j);
          same[j] = (uint32_t)__builtin_amdgcn_ballot_w64(slots == band && slots >= 0);
          if (same[j] & ((1u << (2 * wave + j)) - 1)) same[j] = 0;   // an earlier slot of the band does it
        }
        const int j = lane >> 5, b = lane >> 4 & 1, r16 = lane & 15;
        if (b < kB && (same[0] | same[1])) {
          double total = 0.;   // (so that the number of wavefronts that share a band adds no rounding)
#pragma unroll
          for (int t = 0; t < 2 * kWaves; ++t) {   // all slots are read at once, the ones of other bands dropped
            const float v = slot_val[(t * kB + b) * 16 + r16];
            total += (j ? same[1] : same[0]) >> t & 1 ? v : 0.f;
          }
          const float sum = (float)total;
          const int bnd = j ? __builtin_amdgcn_readlane(slots, 2 * wave + 1) : __builtin_amdgcn_readlane(slots, 2 * wave);
          const bool mine = (j ? same[1] : same[0]) != 0;
          const uint32_t row = (uint32_t)bnd * kUnitRows + r16;
          const bool part = kShared && ((uint32_t)bnd * nq < share_lo || ((uint32_t)bnd + 1) * nq > share_hi);   // another workgroup has the rest
          // (a part is rounded once, behind its scale, and their sum once: as often as a whole band's sum)
          const float t = kShared && part ? (float)(total * (double)slot_scale) : sum * slot_scale;
          if (a.gate_up) {   // lanes 2r, 2r + 1 hold the gate and the up row of output r
            const float other = __shfl_xor(t, 1);
            if (mine && !(r16 & 1) && row + 1 < m.rows) y_store<kStaged>(yb + (size_t)b * (m.rows / 2) + row / 2, silu_times(t, other));
          } else if (mine && row < m.rows) {
            float* out = yb + (size_t)b * m.rows + row;
            if (part) y_add(out, t);
            else y_store<kStaged>(out, t);
          }
        }
      }
    }
    if constexpr (kOne) return;
    advance();
  }
  if constexpr (kStaged) {
    wait_for_stores();
    if (arrived + 1 < n_stages) stage_arrive(a, n_stages - 1);   // (stages without a share; nobody waits for the last one)
    stage_end(a);
  }
}

}  // namespace tq
