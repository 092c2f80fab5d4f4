// Host-only: which of the ring kernels a container's matrix may take on the device, as it is decided when it is loaded (ring_class),
// and how far its lanes get in the activation image of the dot-product kernel (max_lane_reach).
#include <cstdio>
#include <vector>
#include "../include/tq.h"
#include "../paper_2509_22951_amd/csrc/tq_level.h"

int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    std::FILE* f = std::fopen(argv[i], "rb");
    if (!f) return std::printf("%s: cannot be opened\n", argv[i]), 1;
    std::vector<uint8_t> blob;
    uint8_t part[4096];
    for (size_t n; (n = std::fread(part, 1, sizeof part, f)) > 0;) blob.insert(blob.end(), part, part + n);
    std::fclose(f);
    tq::Header h;
    tq::BlobFacts facts;
    std::vector<uint32_t> wide;
    if (tq::validate_blob(blob.data(), blob.size(), &h, &facts, &wide, 4) != TQ_OK) return std::printf("%s\n", tq_last_error_string()), 1;
    std::unique_ptr<uint16_t[]> codes;
    std::printf("%u %u\n", tq::ring_class(blob.data(), h, wide, 4, codes), facts.max_lane_reach);
  }
  return 0;
}
