// Grids of the kernels that decode 4 x 4 blocks, in workgroups per CU, by the matrix, the rate and the type.
#pragma once
#include <stddef.h>

namespace zc2d {

// us of 8192 x 32768 values at rate 4: decompress2d 234, 222 and 222 at 16, 24 and 32, the 2-way reduce
// with fp32 output 384, 357, 362 and 386 at 24, 48, 64 and 96.  With fp32 rows that are aligned to
// their elements only, at rates 2 to 8 also with those that do not start at 64 bytes, decompress2d gains from more:
// neighbouring wavefronts write to the same cache lines and should do so at the same time (6144 x 43690 values at rate 4: 279
// at 48, 250 at 64; at rate 8 274 and 277; 6144 x 43688 at rate 4 309 at 24, 255 at 64).  At rate 8 those that do not start at 64
// bytes want no lane to take a second block (at 12, 24, 64 and at 1024, where none does: 5000 x 10004 values 56.4, 45.8, 45.6 and 45.2, 8192 x
// 12292 127, 115, 91.6 and 90.0, 10000 x 12292 157, 143, 109 and 110, 16384 x 12292 272, 254, 222 and 177, 6144 x 43688 326, 311, 268 and 236;
// when a step of the decoder took longer, 46.5, 89.6, 113, 189 and 229 with 12 up to 448 MiB of output and 64 from there), but for rows of
// five blocks at most, which share few lines (4000000 x 12 values 45.6 at 12 and 48.4 at 1024).
// Half-precision ones at rate 2 that do not start at cache lines gain from where the output is larger than the last-level
// cache (12288 x 12292 97 and 107, 8192 x 24580 141 and 134, 8192 x 28676 201 and 152; at rate 4 98 and 109, 132 and 139, 155 and 159).  The
// reduce with local values and fp32 output is like decompress2d (522 at 24, 457 at 64).  The reduces that write streams have
// 24: 469 at 16, 24 and 32.  Matrices of fewer than twice these many workgroups' blocks get fewer, unless they are to be
// decoded at once.
constexpr int kDecodeWorkgroupsPerCU = 24, kDecodeWorkgroupsPerCUWide = 64, kDecodeWorkgroupsPerCUMost = 1024, kDecodeWorkgroupsPerCULeast = 12;
constexpr size_t kDecodeBytesLarge = (size_t)448 << 20;   // of output

struct DecompressGrid {
  int per_cu;
  bool at_once;   // as many workgroups as there are blocks for, up to that
};
constexpr DecompressGrid decompress_grid(size_t blocks, size_t cols, bool half, int rate) {
  if (half) {
    if (rate == 2 && (cols & 31) != 0 && blocks * 32 >= kDecodeBytesLarge) return {kDecodeWorkgroupsPerCUWide, true};
    return {(cols & 3) != 0 ? kDecodeWorkgroupsPerCUWide : kDecodeWorkgroupsPerCU, false};
  }
  if ((cols & 3) != 0) return {kDecodeWorkgroupsPerCUWide, true};
  if ((cols & 15) != 0 && rate <= 4) return {kDecodeWorkgroupsPerCUWide, true};
  if ((cols & 15) != 0 && rate == 8) {
    if (cols > 20) return {kDecodeWorkgroupsPerCUMost, true};
    if (blocks * 64 >= kDecodeBytesLarge) return {kDecodeWorkgroupsPerCUWide, true};
  }
  return {kDecodeWorkgroupsPerCU, false};
}

}  // namespace zc2d
