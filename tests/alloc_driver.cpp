// Host-only: the validator with one allocation after the other refused, in the calling thread and in its own.  It has to come
// back with TQ_E_OOM every time (an exception that leaves a thread ends the process).
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>
#include "../include/tq.h"

static std::atomic<long> refuse{-1};   // allocations until one is refused

void* operator new(size_t n) {
  if (refuse.load() >= 0 && refuse.fetch_sub(1) == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
  // rows in turn all zeros (long runs of pairs) and all different: lanes far apart in every unit
  const uint32_t rows = 400, cols = 1024;
  std::vector<int8_t> q((size_t)rows * cols, 0);
  for (uint32_t r = 0; r < rows; r += 2)
    for (uint32_t c = 0; c < cols; ++c) q[(size_t)r * cols + c] = (int8_t)(std::rand() % 255 - 127);
  std::vector<float> scales(rows, 1.f);
  tq_encode_opts o;
  std::memset(&o, 0, sizeof o);
  o.max_entries = 300;
  void* blob = nullptr;
  size_t bytes = 0;
  if (tq_encode_quantized(q.data(), scales.data(), rows, cols, &o, &blob, &bytes) != TQ_OK) return std::printf("encode: %s\n", tq_last_error_string()), 1;
  int refused = 0;
  for (long k = 0;; ++k) {
    refuse = k;
    const int rc = tq_validate_blob(blob, bytes, nullptr);
    const bool reached = refuse.load() < 0;
    refuse = -1;
    if (!reached) {
      if (rc != TQ_OK) return std::printf("validate: %s\n", tq_last_error_string()), 1;
      break;
    }
    if (rc != TQ_E_OOM) return std::printf("allocation %ld refused: status %d\n", k, rc), 1;
    ++refused;
  }
  tq_free_blob(blob);
  std::printf("came back from %d refused allocations\n", refused);
  return refused > 1 ? 0 : 1;   // (the threads, and the list of units that each of them hands in)
}
