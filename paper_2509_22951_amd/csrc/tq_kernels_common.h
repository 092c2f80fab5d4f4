// Device side of libtq: constants, kernel-argument structures and the small device helpers every kernel uses.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <utility>

#include "../../include/tq.h"
#include "tq_format.h"
#include "tq_plan.h"

namespace tq {

constexpr int kWaves = 8;            // most wavefronts per workgroup of the tile kernels (one workgroup per CU: LDS-bound)
constexpr int kThreads = kWaves * 64;
constexpr int kDotWavesPacked = 12;  // the same kernel for packed 4-bit weights: more work per byte read, more wavefronts to
                                     // hide it (config 4, ms per step: 8 wavefronts 0.379, 12 0.370, 16 0.379)
#ifndef TQ_STAGED_WAVES
#define TQ_STAGED_WAVES 8
#endif
constexpr int kDotWavesStaged = TQ_STAGED_WAVES;   // the staged form of the batch-1 and batch-2 kernel (the 113 dependent stages
                                                   // of the 3B sweep, ms per step: 8 wavefronts 1.59, 12 1.87, 16 1.88)
constexpr int kDotWavesMax = kDotWavesStaged > 12 ? kDotWavesStaged : 12;
constexpr int kDotPiecePacked = 6;   // its units are half as long (segments of 128 bytes: 17 chunks, three pieces of 5 or 6)
constexpr int kDotWaves = 8;         // wavefronts per workgroup of the batch-1 kernel (measured on the 3B sweep, TB/s:
                                     // 6 waves 4.61, 8 waves 5.12, 10 waves 4.64, 12 waves 4.90, 16 waves 4.28)
constexpr int kDotPiece = 8;         // chunks per piece in the batch-1 kernel: two pieces (16 x 512 bytes) are in flight per
                                     // wavefront (measured on the 3B sweep, TB/s: 4 chunks 5.30, 6 5.48, 8 5.47, 12 5.41, 18 5.24)
#ifndef TQ_DOT_SETS
#define TQ_DOT_SETS 2
#endif
constexpr int kDotSets = TQ_DOT_SETS;   // register sets of the batch-1 kernel's chunk pipeline (operands read kDotSets - 1 chunks ahead)
constexpr uint32_t kLdsLimit = 160 * 1024;
constexpr int kPiece = 12;           // code chunks fetched together by a wavefront (units of 256-column segments are
                                     // 33..36 chunks long: three pieces with little repetition)
constexpr int kMaxMulti = 128;       // matrices one launch can serve (bounded by the 4 KB of kernel arguments)
constexpr int kInlineDescriptions = 4;

// What the kernels need to know about one matrix.
struct DevMat {
  const uint32_t* dict;    // the dictionary's byte image, as the batched kernels and the expansion keep it in LDS: 2 bytes per entry, zeros past the pad entry
  const uint32_t* dict_bf16;   // the same entries as two bf16 weights each (second one zero for a single byte): the form the
                               // batch-1 kernel keeps in LDS, made once when the dictionary is uploaded
  const uint32_t* uoff;    // n_units + 1 unit offsets, in chunks
  const uint2* codes;      // chunk c, lane l -> codes[c * 64 + l] (4 codes)
  const float* scales;     // n_bands * 16 row scales
  uint32_t rows, cols, seg_cols;
  uint32_t n_bands, n_quads;
  uint32_t dict_words;     // multiple of 4
  uint32_t x_span;         // dwords per panel in the LDS image of x: seg_cols plus a gap that spreads the 4 panels of a unit over the banks
  uint32_t x_dwords;       // size of that image, including the columns lanes can reach while they consume pad codes
  uint32_t seg_magic;      // floor(2^32 / seg_cols) + 1: col / seg_cols == mulhi(col, seg_magic) for every column index in use
  uint32_t ring;           // the lanes of every unit stay as close together as rings of 128 bytes (1), or of 64 bytes too (2), need; else 0 (ring_class)
  uint32_t packing;        // 1: every byte holds two 4-bit weights (columns 2j and 2j + 1 of a matrix of 2 * cols columns); rows,
                           // cols and seg_cols describe the byte matrix, and dict_bf16 holds four fp8 (e4m3) weights per entry
  uint32_t long_runs;      // 1: runs of 3 and 4 bytes exist (lmax > 2): the code space classes below apply, and dict / dict_bf16
                           // point to images with two slots for every entry from `class2` on (see long_slot)
  uint32_t class2, class3; // codes from class2 on are runs of at least 3 bytes, from class3 on of 4 (sorted code space)
  uint32_t dict16_bytes;   // size of the byte image at `dict` (a multiple of 16)
};
static_assert(sizeof(DevMat) % 8 == 0, "copied as whole dwords, kept 8-byte aligned in tables");

// Containers with runs of up to 4 bytes keep a dictionary image with one slot for an entry of up to 2 bytes and two
// slots for a longer one, the long ones starting on an even slot: slot index of a code.
__device__ __forceinline__ uint32_t long_slot(uint32_t code, uint32_t class2) {
  const uint32_t even = class2 & ~1u;
  return code + (code > even ? code - even : 0u);   // codes below class2 never exceed `even` by more than 0: class2 - 1 <= even
}
// Run length of a code by its place in the sorted code space (the pad code, past the last entry, counts as 4).
__device__ __forceinline__ uint32_t long_run_length(uint32_t code, uint32_t class2, uint32_t class3) {
  return 1u + (code >= 256u ? 1u : 0u) + (code >= class2 ? 1u : 0u) + (code >= class3 ? 1u : 0u);
}

struct Job {
  const DevMat* m;         // device copy of the matrix description
  const uint16_t* x;       // bf16 [batch][cols]
  float* y;                // fp32 [batch][rows]
};

// A job together with its matrix description, as a prepared step keeps them in device memory.
struct StepEntry {
  DevMat m;
  const uint16_t* x;
  float* y;
};
constexpr int kMaxStep = 896;        // matrices one launch can serve when the jobs come from a device table

// The launch's cost line: matrix i covers [cost[i], cost[i + 1]), one band of it costs its number of columns (by_workgroup:
// the line counts workgroups instead).
// The jobs travel in the kernel arguments (up to kMaxMulti of them) or, for a prepared step, sit in a table in device
// memory (up to kMaxStep); the cost line is in the arguments either way, at the same place.
struct MatvecArgs {
  int n, batch;
  uint32_t x_off, slot_off;   // byte offsets in LDS of the activation image (or of the tiles) and of the partial-sum slots
  uint32_t tile_area;         // bytes of LDS per wavefront in the tile kernels (the same for every matrix of the launch)
  uint16_t gate_up;           // 1: rows 2r and 2r + 1 are a gate and an up projection; y[b][r] = silu(row 2r) * (row 2r + 1)
  uint16_t by_workgroup;      // 1: the cost line counts workgroups (see share_of_bands); kBySharedBands: and workgroups may share bands (staged steps, see shared_share)
  uint32_t share, share_rest; // the cost line in even parts (even_part), one per workgroup; by_workgroup: share is the workgroups of a stage
  float parts_inverse;
  const StepEntry* table;     // device table of the n jobs, or null: then j and first below hold them
  // A staged step (one launch for products that depend on each other): the jobs come in n_stages groups, jobs
  // stage_first[s] .. stage_first[s + 1] - 1 form stage s, and no workgroup starts a stage before every workgroup has
  // stored the results of the one before (grid-wide hand-over through the words at sync, see stage_arrive).
  const uint32_t* stage_first;   // device, n_stages + 1 entries; null: not staged
  uint32_t* sync;                // device, sync_words(gridDim.x) words, zero at launch
  uint32_t* fault_host;          // host memory the device can write: set to 1 when a wait gave up
  uint32_t n_stages;
  uint32_t spin_limit;           // polls of the hand-over table before a workgroup gives up
  union {
    struct {
      uint32_t cost[kMaxMulti + 1];
      Job j[kMaxMulti];
      DevMat first[kInlineDescriptions];   // descriptions of the first matrices by value: a launch of one matrix (or of a
                                           // few) does not wait for a read of device memory before it can start loading
    } in;
    uint32_t cost_long[kMaxStep + 1];
  } u;
};
static_assert(sizeof(MatvecArgs) <= 4096, "kernel arguments");

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const uint32_t lds_cu32;
typedef __attribute__((address_space(3))) const uint64_t lds_cq64;
typedef __attribute__((address_space(3))) const uint16_t lds_cu16;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(4))) const uint32_t const_u32;

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// Unit offsets are wave-uniform and never written while a kernel runs: reading them through the constant address
// space makes them scalar loads, which do not share a counter with the vector loads of the code stream.
__device__ __forceinline__ uint32_t unit_offset(const DevMat& m, uint32_t u) { return ((const_u32*)m.uoff)[u]; }

// Loads and stores of device memory through the global address space.  Pointers that come out of a matrix description
// read from memory are generic to the compiler; a generic access is a flat instruction, which counts on the LDS counter
// as well as on the vector-memory one and so would make every LDS wait a wait for the code stream too.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Chunk `chunk` of the code stream, lane's 4 codes: a wave-uniform base in scalar registers plus the lane's offset, so
// that no vector arithmetic goes into the address.
__device__ __forceinline__ uint2 load_chunk(const uint2* codes, uint32_t chunk, int lane) {
  const uint64_t base = (uint64_t)codes + (uint64_t)chunk * (64 * sizeof(uint2));
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base), hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
  const u32x2 v = ((__attribute__((address_space(1))) const u32x2*)((uint64_t)hi << 32 | lo))[(uint32_t)lane];
  return make_uint2(v.x, v.y);
}

__device__ __forceinline__ uint2 global_load(const uint2* p) {
  const u32x2 v = *(__attribute__((address_space(1))) const u32x2*)p;
  return make_uint2(v.x, v.y);
}
__device__ __forceinline__ uint4 global_load(const uint4* p) {
  const u32x4 v = *(__attribute__((address_space(1))) const u32x4*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint32_t global_load(const uint32_t* p) { return *(__attribute__((address_space(1))) const uint32_t*)p; }
__device__ __forceinline__ uint32_t global_load(const uint8_t* p) { return *(__attribute__((address_space(1))) const uint8_t*)p; }
__device__ __forceinline__ uint32_t global_load(const uint16_t* p) { return *(__attribute__((address_space(1))) const uint16_t*)p; }
__device__ __forceinline__ float global_load(const float* p) { return *(__attribute__((address_space(1))) const float*)p; }
__device__ __forceinline__ void global_store(float* p, float v) { *(__attribute__((address_space(1))) float*)p = v; }

// The same accesses, coherent across the whole device without any cache maintenance: relaxed atomics at device scope
// are served at the level all compute units share.  A staged step stores its outputs and loads its activations this
// way, so that a hand-over between stages needs no write-back or invalidation of caches (those cost microseconds).
template <bool kCoherent>
__device__ __forceinline__ uint32_t x_load(const uint32_t* p) {
  if constexpr (kCoherent) return __hip_atomic_load((__attribute__((address_space(1))) const uint32_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return global_load(p);
}
template <bool kCoherent>
__device__ __forceinline__ uint32_t x_load(const uint16_t* p) {
  if constexpr (kCoherent) return __hip_atomic_load((__attribute__((address_space(1))) const uint16_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return global_load(p);
}
template <bool kCoherent>
__device__ __forceinline__ void y_store(float* p, float v) {
  if constexpr (kCoherent) __hip_atomic_store((__attribute__((address_space(1))) float*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else global_store(p, v);
}

__device__ __forceinline__ void y_add(float* p, float v) {   // at device scope, no return value
  (void)__builtin_amdgcn_global_atomic_fadd_f32((__attribute__((address_space(1))) float*)p, v);
}

// A matrix description from device memory, through scalar loads.
__device__ __forceinline__ DevMat load_description(const DevMat* p) {
  static_assert(sizeof(DevMat) % 4 == 0, "whole dwords");
  uint32_t w[sizeof(DevMat) / 4];
#pragma unroll
  for (size_t k = 0; k < sizeof(DevMat) / 4; ++k) w[k] = ((const_u32*)p)[k];
  DevMat m;
  __builtin_memcpy(&m, w, sizeof m);
  return m;
}

// Point i of the launch's cost line (the two forms of the arguments keep it at the same place).
__device__ __forceinline__ uint32_t cost_at(const MatvecArgs& a, int i) {
  const uint32_t v = a.u.cost_long[i];
  return a.by_workgroup ? v & kLineMask : v;
}

// A launch whose matrices have whole workgroups (kMaxAssign of them at most, one workgroup per compute unit) says in its arguments which
// matrix a workgroup serves, a byte each, behind the cost line: no search.
constexpr int kJobMapAt = kMaxAssign + 4, kJobMapWorkgroups = 256;   // (dwords of the cost line that such a launch does not use)
static_assert(kJobMapAt + kJobMapWorkgroups / 4 <= kMaxMulti + 1 && kMaxAssign <= 256, "the map lies in the unused part of the shorter line");
__device__ __forceinline__ int mapped_job(const MatvecArgs& a) {
  return (int)(a.u.cost_long[kJobMapAt + blockIdx.x / 4] >> (blockIdx.x % 4 * 8) & 255u);
}

// The workgroup's part of a cost line that counts weights.
__device__ __forceinline__ void even_share(const MatvecArgs& a, uint32_t& lo, uint32_t& hi) {
  lo = even_part(a.share, a.share_rest, a.parts_inverse, blockIdx.x);
  hi = even_part(a.share, a.share_rest, a.parts_inverse, blockIdx.x + 1);
  lo = __builtin_amdgcn_readfirstlane(lo);
  hi = __builtin_amdgcn_readfirstlane(hi);
}

// The lines of the kernel arguments a launch of few matrices looks at - head and cost line, first job, first description -
// requested together: taken as they are needed, each costs a round trip of its own (0.3 us) before the first load of
// the matrix can start.
__device__ __forceinline__ void touch_arguments() {
  const const_u32* k = (const const_u32*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr size_t line = offsetof(MatvecArgs, u.cost_long) / 4, job = offsetof(MatvecArgs, u.in.j) / 4, desc = offsetof(MatvecArgs, u.in.first) / 4;
  const uint32_t v0 = k[0], v1 = k[16], v2 = k[job], v3 = k[desc], v4 = k[desc + 16], v5 = k[desc + sizeof(DevMat) / 4 - 1];
  const uint32_t v6 = k[line + kJobMapAt + (blockIdx.x & (kJobMapWorkgroups - 1)) / 4];
  asm volatile("" ::"s"(v0), "s"(v1), "s"(v2), "s"(v3), "s"(v4), "s"(v5), "s"(v6));
}

// First job of [first, end) that ends behind point `lo` of the cost line.  A step has up to kMaxStep jobs: looking at
// them one after the other costs a scalar load's latency each (the last workgroups of a 113-matrix step began 3 us late),
// so the 64 lanes look at 64 of them at a time.
__device__ __forceinline__ int first_job(const MatvecArgs& a, int first, int end, uint32_t lo, int lane) {
  if (end - first <= 4) {
    while (first < end && cost_at(a, first + 1) <= lo) ++first;
    return first;
  }
  for (; first < end; first += 64) {
    const uint64_t behind = __builtin_amdgcn_ballot_w64(first + lane < end && cost_at(a, min(first + lane, end - 1) + 1) > lo);
    if (behind) return first + __builtin_ctzll(behind);
  }
  return end;
}

// The bands of matrix m, at [cb, ce) of the cost line, that belong to the share [lo, hi) of a workgroup.
// Cost line in weights: a band goes to the share that holds its middle; a workgroup may get the end of one matrix and the
// start of the next.  Cost line in workgroups (launches of few matrices, see assign_workgroups): [lo, hi) is one
// workgroup, inside one matrix (job i), which has its bands split evenly over its ce - cb workgroups.
__device__ __forceinline__ void share_of_bands(const MatvecArgs& a, bool by_workgroup, const DevMat& m, int i, uint32_t lo, uint32_t hi,
                                               uint32_t& band_lo, uint32_t& band_hi) {
  const uint32_t first = a.u.cost_long[i], next = a.u.cost_long[i + 1];
  if (by_workgroup) {
    const uint32_t cb = first & kLineMask, ce = next & kLineMask, bands = first >> kLineBits, rest = m.n_bands - bands * (ce - cb);
    band_lo = workgroup_band(bands, rest, lo - cb);
    band_hi = workgroup_band(bands, rest, hi - cb);
  } else {
    const uint32_t cb = first, ce = next;
    const uint32_t bc = m.cols;
    band_lo = lo <= cb ? 0u : (lo - cb + bc / 2) / bc;
    band_hi = hi >= ce ? m.n_bands : min(m.n_bands, (hi - cb + bc / 2) / bc);
  }
}

// Job i of the launch and the description of its matrix: from the kernel arguments, or from the step's device table
// (scalar loads, like the descriptions the arguments do not hold by value).
__device__ __forceinline__ void fetch_job(const MatvecArgs& a, int i, Job& job, DevMat& m) {
  if (a.table) {
    const StepEntry* e = a.table + i;
    static_assert(sizeof(StepEntry) % 4 == 0, "whole dwords");
    uint32_t w[sizeof(StepEntry) / 4];
#pragma unroll
    for (size_t k = 0; k < sizeof(StepEntry) / 4; ++k) w[k] = ((const_u32*)e)[k];
    StepEntry v;
    __builtin_memcpy(&v, w, sizeof v);
    m = v.m;
    job.m = &e->m;
    job.x = v.x;
    job.y = v.y;
  } else {
    job = a.u.in.j[i];
    m = i < kInlineDescriptions ? a.u.in.first[i] : load_description(job.m);
  }
}

// Grid-wide hand-over between two stages of a staged step.  The stage's outputs were stored with device-coherent
// stores (y_store<true>); every wavefront waits until its own stores have been acknowledged, the workgroup meets at a
// barrier and announces itself by writing the number of stages it has behind it to its word of the table at sync, and the
// first wavefront polls the table until no workgroup is behind (relaxed device-scope atomics throughout: the words
// and the data are coherent by the way they are accessed, so no cache is written back or invalidated).  The next stage
// loads its activations coherently too (x_load<true>).
// There are kSyncCopies copies of the table, each polled by 1 / kSyncCopies of the workgroups.  What this and the layout
// rest on: workgroups that poll one line keep its memory channel busy, and announcements queue behind them.  Four
// LLaMA-3.2-3B layers as 16 stages, us: one counter per stage that everybody adds to and polls 272, 2, 4, 8 such counters
// 250, 237, 231; a table of plain words 227, in 4, 8, 16, 32 copies 219, 216, 222, 223.
// All workgroups of the launch must be resident together (the host launches at most one per compute unit).  The wait is
// bounded: after spin_limit polls, or when another workgroup has given up, the workgroup sets the fault words and
// goes on without waiting - the launch then ends with results that must not be used, and the host reports it.
// The hand-over comes in two halves so that a workgroup can fetch what its next stage needs and what no other workgroup
// writes (matrix descriptions, unit offsets, the first code chunks) between the two, while the others still finish.
// stage_arrive: this workgroup's outputs of the stages are out.  stage_wait: every workgroup's are; it ends with a
// workgroup barrier.  A workgroup that has no share of a stage goes on to the next arrive without waiting: it reads
// and writes nothing there, and whatever it does later comes after a wait on a later stage.
// The words are zero when a launch starts: stage_end, the last thing a workgroup does, counts the workgroups out, and the
// last one clears them (nobody else looks at them any more) for the launch that follows on the stream.  The fault word is
// among them: the report to the host stays, but a captured launch that is replayed after it waits as it should.
constexpr uint32_t kSyncCopies = 8, kLineWords = 32;
__host__ __device__ constexpr uint32_t sync_stride(uint32_t grid) { return (grid + 127) / 128 * 128; }   // words of a copy
__host__ __device__ constexpr uint32_t fault_word(uint32_t grid) { return kSyncCopies * sync_stride(grid); }
__host__ __device__ constexpr uint32_t sync_words(uint32_t grid) { return fault_word(grid) + 2; }
typedef __attribute__((address_space(1))) uint32_t global_u32;
typedef __attribute__((address_space(1))) uint64_t global_u64;

__device__ __forceinline__ void wait_for_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void stage_arrive(const MatvecArgs& a, uint32_t stages) {   // this workgroup's outputs of stages 0 .. stages - 1
  __syncthreads();   // every wavefront's stores have reached the level the device shares
  if (threadIdx.x < kSyncCopies)
    __hip_atomic_store((global_u32*)a.sync + threadIdx.x * sync_stride(gridDim.x) + blockIdx.x, stages, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stage_wait(const MatvecArgs& a, uint32_t stages) {
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x;
    const global_u32* mine = (const global_u32*)a.sync + blockIdx.x % kSyncCopies * sync_stride(gridDim.x);
    global_u32* fault = (global_u32*)a.sync + fault_word(gridDim.x);
    uint32_t polls = 0;
    for (;;) {
      bool behind = false;
      for (uint32_t w = 2 * lane; w < gridDim.x; w += 128) {
        const uint64_t two = __hip_atomic_load((const global_u64*)(mine + w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        behind = behind || (uint32_t)two < stages || (w + 1 < gridDim.x && (uint32_t)(two >> 32) < stages);
      }
      if (__builtin_amdgcn_ballot_w64(behind) == 0) break;
      ++polls;   // (the fault word, one for all, is looked at now and then)
      if (polls > a.spin_limit || (polls % 32 == 0 && __hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        if (lane == 0) {
          __hip_atomic_store(fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(a.fault_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void stage_end(const MatvecArgs& a) {
  if (threadIdx.x < 64) {
    global_u32* sync = (global_u32*)a.sync;
    const uint32_t fault = fault_word(gridDim.x);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this workgroup's announcements (and its fault, if it gave up) are in
    uint32_t before = 0;
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(sync + fault + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) == gridDim.x - 1)
      for (uint32_t i = threadIdx.x; i < sync_words(gridDim.x); i += 64) __hip_atomic_store(sync + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// n16 pieces of 16 bytes from global memory to LDS by the loads that write LDS themselves: no registers, no store instructions, and all of
// a wavefront's requests on their way at once.  (120 KB into 8 wavefronts' workgroups on every compute unit, until the barrier: 1.05 us, through
// registers 1.45; the 64 bytes a clock that a compute unit takes are 0.85.)  In round r wavefront `wave` of n_waves takes kilobyte r * n_waves + wave.  lds_arrived(),
// then a barrier, before anyone reads.
__device__ __forceinline__ void request_to_lds(const void* src, uint32_t n16, int lane, int wave, int n_waves, void* lds, uint32_t first_round = 0,
                                               uint32_t end_round = 0x10000u) {
  typedef __attribute__((address_space(1))) const uint32_t global_cu32;
  typedef __attribute__((address_space(3))) uint32_t lds_mu32;
  // (whole rounds without a look at the lanes, the address a uniform base plus the lane's offset: four scalar instructions a request)
  const uint32_t step = (uint32_t)n_waves * 64, whole = min(n16 / 64, end_round * (uint32_t)n_waves);   // kilobytes that all lanes have
  uint32_t c = first_round * (uint32_t)n_waves + (uint32_t)wave;
  const uint64_t at = (uint64_t)src + (uint64_t)c * 1024;
  const uint32_t at_lo = __builtin_amdgcn_readfirstlane((uint32_t)at), at_hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
  uint64_t from = (uint64_t)at_hi << 32 | at_lo;
  uint32_t to = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)lds + c * 1024);
  for (; c < whole; c += (uint32_t)n_waves) {
    __builtin_amdgcn_global_load_lds((global_cu32*)from + 4 * lane, (lds_mu32*)(size_t)to, 16, 0, 0);
    from += step * 16;
    to += step * 16;
  }
  if (c == n16 / 64 && c < end_round * (uint32_t)n_waves && (uint32_t)lane < n16 % 64)
    __builtin_amdgcn_global_load_lds((global_cu32*)from + 4 * lane, (lds_mu32*)(size_t)to, 16, 0, 0);
}
// Where requests depend on a condition (a dictionary that is new) inside a loop over jobs, the wait belongs into the same branch: with a condition of its
// own the compiler takes the requests for unfinished on the way round it, and the barriers of the loop wait for all loads, those of the next
// activation tile or of the next codes among them (us, wait behind the tile or the image -> with the requests: eight LLaMA-3.2-3B layers batch 8 218.5 -> 217.0, packed
// 153.9 -> 151.5; four in 16 stages 192.6 -> 190.7, batch 2 200.0 -> 198.1).  k_matvec without stages keeps them apart: its workgroups have one job or two, and
// the first dictionary's first rounds ahead of the unit offsets are worth a little more (together -> apart: six LLaMA-3.2-1B layers 79.8 -> 79.4, eight 3B layers
// batch 2 173.4 -> 172.8, packed ones 82.5 -> 82.6).
__device__ __forceinline__ void lds_arrived() {
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0) alone.  (The builtin, not inline assembly: the compiler sees that these loads are done)
  asm volatile("" ::: "memory");
}

// Byte address inside LDS of a pointer into the workgroup's dynamic shared memory.
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(size_t)(const lds_u8*)p; }

// 16-bit halves of a packed code pair that are at least 256, as 0 / 1 in either half: the runs of two weights.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 count_pairs(u16x2 acc, uint32_t codes) {
  const u16x2 high = __builtin_bit_cast(u16x2, codes) >> 8;
  return acc + __builtin_elementwise_min(high, u16x2{1, 1});
}

// Where the lanes stand at chunk c0 of the unit that starts at chunk unit_start < c0: the mark before it, and the up to kMarkChunks - 1
// chunks between (requested together, and looked at when they have arrived).
struct Place {
  uint32_t mark;
  uint2 c[kMarkChunks - 1];
};
__device__ __forceinline__ void request_place(const DevMat& m, uint32_t unit_start, uint32_t c0, int lane, Place& p) {
  const uint32_t k = (c0 - unit_start) / kMarkChunks, from = unit_start + k * kMarkChunks;
  p.mark = 0;
  if (k) {
    const uint64_t at = (mark_index(unit_start) + k) * mark_bytes(m.seg_cols);
    const uint8_t* marks = (const uint8_t*)m.uoff + marks_at((uint64_t)m.n_bands * m.n_quads) + at;
    p.mark = m.seg_cols <= kMarkByteCols ? global_load(marks + lane) : global_load((const uint16_t*)marks + lane);
  }
#pragma unroll
  for (uint32_t j = 0; j < kMarkChunks - 1; ++j) p.c[j] = load_chunk(m.codes, min(from + j, c0 - 1), lane);
}
__device__ __forceinline__ uint32_t columns_passed(const Place& p, uint32_t unit_start, uint32_t c0) {
  const uint32_t n = (c0 - unit_start) % kMarkChunks;
  u16x2 pairs = {0, 0};
#pragma unroll
  for (uint32_t j = 0; j < kMarkChunks - 1; ++j)
    if (j < n) pairs = count_pairs(count_pairs(pairs, p.c[j].x), p.c[j].y);
  return kChunkCodes * (c0 - unit_start) + p.mark + pairs.x + pairs.y;
}

// One of n_waves equal runs of chunks of a share of n_units < 64 units: chunks [c0, c_end) of the units [u0, u1).
// uoff_lane: lane k holds the offset of the share's unit k, lanes from n_units on that of its end.
struct EvenRun {
  uint32_t u0, u1, c0, c_end;
  bool head, tail;       // the run starts / ends inside a unit
  uint32_t unit_start;   // of unit u0
};
__device__ __forceinline__ EvenRun even_run(uint32_t uoff_lane, uint32_t unit_lo, uint32_t n_units, int wave, int n_waves, uint32_t min_chunks) {
  EvenRun r;
  const uint32_t all_lo = __builtin_amdgcn_readlane(uoff_lane, 0), all_n = __builtin_amdgcn_readlane(uoff_lane, n_units) - all_lo;
  const uint32_t n_runs = min((uint32_t)n_waves, (all_n + min_chunks - 1) / min_chunks);   // the wavefronts behind that many have none
  r.c0 = all_lo + all_n * min((uint32_t)wave, n_runs) / n_runs;
  r.c_end = all_lo + all_n * min((uint32_t)wave + 1, n_runs) / n_runs;
  const uint64_t lanes = (2ull << n_units) - 1;   // lanes 0 .. n_units hold the offsets
  const uint32_t first = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(uoff_lane <= r.c0) & lanes) - 1;
  const uint32_t last = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(uoff_lane < max(r.c_end, r.c0 + 1)) & lanes) - 1;
  const uint32_t last_end = __builtin_amdgcn_readlane(uoff_lane, min(last + 1, 63u));
  const bool empty = r.c0 >= r.c_end;
  r.u0 = unit_lo + first;
  r.u1 = empty ? r.u0 : unit_lo + last + 1;
  r.unit_start = __builtin_amdgcn_readlane(uoff_lane, first);
  r.head = !empty && r.c0 > r.unit_start;
  r.tail = !empty && r.c_end < last_end;
  return r;
}

// Of the wavefronts of a SIMD that could go on the oldest is served, so that the first is done with its run when the last has a third of its own
// left, and works alone from then on.  A wavefront that has come further than half its run, three quarters, seven eighths takes a
// lower priority than those that have not: they end together.
__device__ __forceinline__ void pace(uint32_t done, uint32_t total) {
  if (2 * done < total) __builtin_amdgcn_s_setprio(3);
  else if (4 * done < 3 * total) __builtin_amdgcn_s_setprio(2);
  else if (8 * done < 7 * total) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// Pointer forms on purpose: the compiler tracks the outstanding LDS read and places the wait before the first use.
__device__ __forceinline__ uint32_t lds_read32(uint32_t addr) { return *(lds_cu32*)(size_t)addr; }
template <int kOff>
__device__ __forceinline__ uint32_t lds_read32_off(uint32_t addr) { return *(lds_cu32*)(size_t)(addr + kOff); }
template <int kOff>   // addr + kOff is 8-byte aligned
__device__ __forceinline__ uint64_t lds_read64_off(uint32_t addr) { return *(lds_cq64*)(size_t)(addr + kOff); }

// Byte offset of dictionary word `code` for the code in the low / high half of a packed code pair: one SDWA shift
// (selects the 16-bit half, zero-extends, multiplies by 4) instead of a mask and a shift.
__device__ __forceinline__ uint32_t word_offset_lo(uint32_t pair) {
  uint32_t a;
  const uint32_t two = 2;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(a) : "v"(two), "v"(pair));
  return a;
}
__device__ __forceinline__ uint32_t word_offset_hi(uint32_t pair) {
  uint32_t a;
  const uint32_t two = 2;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(a) : "v"(two), "v"(pair));
  return a;
}
// min(1, high byte of the low / high code): 1 for a two-weight entry (code >= 256), 0 for a single (a pad too, code 0)
__device__ __forceinline__ uint32_t is_pair_lo(uint32_t pair) {
  uint32_t a;
  const uint32_t one = 1;
  asm("v_min_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(a) : "v"(one), "v"(pair));
  return a;
}
__device__ __forceinline__ uint32_t is_pair_hi(uint32_t pair) {
  uint32_t a;
  const uint32_t one = 1;
  asm("v_min_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(a) : "v"(one), "v"(pair));
  return a;
}
__device__ __forceinline__ float dot2(uint32_t w, uint32_t x, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, x), acc, false);
}

}  // namespace tq
