// Host build of the per-lane pieces of the lossless codec (csrc/zl_codec.h), for checking
// them on the CPU against the reference.  Test-only.
#include <cstring>

#include "../../paper_2409_02423_amd/csrc/zl_codec.h"

extern "C" void zl_host_to_planes(const uint32_t* words, size_t groups, uint32_t* references, uint32_t* bitmaps,
                                  uint32_t* planes) {
  for (size_t g = 0; g < groups; ++g) {
    uint32_t w[32];
    std::memcpy(w, words + 32 * g, sizeof w);
    bitmaps[g] = zl::to_residuals(w, references[g]);
    zl::transpose(w);
    std::memcpy(planes + 32 * g, w, sizeof w);
  }
}

// Groups of 32 16-bit words, as the kernel for such messages has them; planes 16..31 of each.
extern "C" void zl_host_halves_to_planes(const uint16_t* words, size_t groups, uint32_t* references, uint32_t* bitmaps,
                                         uint32_t* planes) {
  for (size_t g = 0; g < groups; ++g) {
    uint32_t w[16];
    for (int j = 0; j < 16; ++j) w[j] = words[32 * g + j] | (uint32_t)words[32 * g + j + 16] << 16;
    bitmaps[g] = zl::to_residuals_of_halves(w, references[g]);
    zl::transpose(w);
    std::memcpy(planes + 16 * g, w, sizeof w);
  }
}

extern "C" void zl_host_from_planes(const uint32_t* planes, const uint32_t* references, size_t groups, uint32_t* words) {
  for (size_t g = 0; g < groups; ++g) {
    uint32_t p[32];
    std::memcpy(p, planes + 32 * g, sizeof p);
    zl::from_planes(p, references[g]);
    std::memcpy(words + 32 * g, p, sizeof p);
  }
}

extern "C" void zl_host_planes_of_groups(const uint32_t* words, size_t groups, uint32_t* counts) {
  for (size_t g = 0; g < groups; ++g) counts[g] = zl::planes_of_group([&](int j) { return words[32 * g + j]; });
}

extern "C" uint32_t zl_host_counters() { return zl::kCounters; }
extern "C" uint32_t zl_host_counter_of(uint32_t workgroup) { return zl::counter_of(workgroup); }
