// Host-only: the encoder and the validator when the system does not start a thread.  pthread_create is replaced by one that
// refuses from the `allowed`-th call on; every call has to come back, with an error or with the same container.  And how many a
// short and wide matrix is given.
#include <dlfcn.h>
#include <errno.h>
#include <pthread.h>
#include <cstdio>
#include <cstring>
#include <vector>
#include "../include/tq.h"

static int calls = 0, allowed = 1 << 30;

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
  static auto real = (int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*))dlsym(RTLD_NEXT, "pthread_create");
  return calls++ < allowed ? real(t, a, f, arg) : EAGAIN;
}

int main() {
  const uint32_t rows = 512, cols = 1024;
  std::vector<float> w((size_t)rows * cols);
  uint32_t state = 1;
  for (auto& v : w) v = (float)(int)((state = state * 1664525u + 1013904223u) >> 24) - 128.f;
  tq_encode_opts o;
  std::memset(&o, 0, sizeof o);
  o.n_threads = 4;
  o.max_entries = 400;   // full after a few units: the rest is coded by the threads
  auto encode = [&](void** blob, size_t* bytes) { return tq_encode(w.data(), rows, cols, &o, blob, bytes); };
  void* want = nullptr;
  size_t want_bytes = 0;
  if (encode(&want, &want_bytes) != TQ_OK) return std::printf("encode: %s\n", tq_last_error_string()), 1;
  const int total = calls;
  int refused = 0;
  for (allowed = 0; allowed <= total; ++allowed) {
    calls = 0;
    void* blob = nullptr;
    size_t bytes = 0;
    const int rc = encode(&blob, &bytes);
    if (rc == TQ_OK ? bytes != want_bytes || std::memcmp(blob, want, bytes) != 0 : blob != nullptr) return std::printf("%d threads allowed: rc %d\n", allowed, rc), 1;
    refused += rc != TQ_OK;
    tq_free_blob(blob);
  }
  if (refused != total) return std::printf("%d of %d calls refused\n", refused, total), 1;
  for (allowed = 0; allowed < 3; ++allowed) {
    calls = 0;
    tq_validate_blob(want, want_bytes, nullptr);
  }
  allowed = 1 << 30;
  if (tq_validate_blob(want, want_bytes, nullptr) != TQ_OK) return std::printf("validate: %s\n", tq_last_error_string()), 1;
  tq_free_blob(want);
  // One band of many units, four threads asked for: its coding is work for every thread that was asked for, and so are its rows.
  std::vector<float> wide((size_t)16 * 16384);
  for (size_t i = 0; i < wide.size(); ++i) wide[i] = w[i % w.size()];
  const std::vector<int8_t> wide_q(wide.size(), 1);
  const std::vector<float> wide_s(16, 1.f);
  for (int quantized = 0; quantized < 2; ++quantized) {
    calls = 0;
    void* blob = nullptr;
    size_t bytes = 0;
    const int rc = quantized ? tq_encode_quantized(wide_q.data(), wide_s.data(), 16, 16384, &o, &blob, &bytes) : tq_encode(wide.data(), 16, 16384, &o, &blob, &bytes);
    tq_free_blob(blob);
    if (rc != TQ_OK || calls != 3) return std::printf("16 x 16384 (%s): rc %d, %d threads beside the caller's\n", quantized ? "quantized" : "fp32", rc, calls), 1;
  }
  // Two values to a byte: segments of half as many bytes, so 16 x 4096 weights are four units.
  calls = 0;
  o.bits = 4;
  o.packing = TQ_PACK_NIBBLES;
  void* packed = nullptr;
  size_t packed_bytes = 0;
  if (tq_encode(wide.data(), 16, 4096, &o, &packed, &packed_bytes) != TQ_OK || calls != 3) return std::printf("16 x 4096 (packed): %d threads beside the caller's\n", calls), 1;
  tq_free_blob(packed);
  o.bits = o.packing = 0;
  // Nobody asks, and all of it is less work than starting a thread.
  calls = 0;
  o.n_threads = 0;
  void* small = nullptr;
  size_t small_bytes = 0;
  if (tq_encode(w.data(), 256, 256, &o, &small, &small_bytes) != TQ_OK || calls != 0) return std::printf("256 x 256: %d threads started\n", calls), 1;
  tq_free_blob(small);
  std::printf("%d encodes came back without all of their threads\n", refused);
  return 0;
}
