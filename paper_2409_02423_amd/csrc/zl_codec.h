// zl_codec.h -- per-lane pieces of the lossless codec ("ZL-1"), as run by one GPU lane.
//
// The paper's first hybrid scheme sends model-parallel traffic through a lossless codec
// of the MPC kind (Sec. II-A, Sec. III-A); this is the format built for that role: a
// lane owns one group of 32 words of a chunk (four consecutive words from each of its
// eight 16-byte reads), describes each by its distance from the group's largest
// magnitude, bit-transposes the 32 residuals in registers and keeps the non-zero planes.
#ifndef ZL_CODEC_H
#define ZL_CODEC_H

#include <stdint.h>

#if defined(__HIPCC__)
#define ZL_DEV __host__ __device__ __forceinline__
#else
#define ZL_DEV inline
#endif

namespace zl {

constexpr uint32_t kMagic = 0x31304C5Au;   // "ZL01"
constexpr int kChunkWords = 8192;
constexpr int kGroups = 256;               // groups per chunk = lanes per workgroup
constexpr int kHeaderBytes = 32;
constexpr int kFixedChunkBytes = 8 * kGroups;   // references and bitmaps

// Table entry: two state bits above a 62-bit byte count.
constexpr uint64_t kValueMask = ((uint64_t)1 << 62) - 1;
constexpr uint64_t kOwnSize = (uint64_t)1 << 62;   // while compressing: the chunk's own size
constexpr uint64_t kEnd = (uint64_t)2 << 62;       // final: where the chunk ends in the payload
// While compressing, some entries also count (see the compress kernel), above the 43 bits that
// the byte count of 2^40 words can take and below the state bits.
constexpr int kTicketShift = 43;
constexpr uint64_t kTicketMask = kValueMask & ~(((uint64_t)1 << kTicketShift) - 1);
constexpr uint32_t kCounters = 8;      // of chunk numbers, in entries kCounterStride apart
constexpr uint32_t kCounterStride = 16;

// The counter that a workgroup of the compress kernel asks for chunk numbers; counter i hands out
// i, i + kCounters, ...  Workgroups go to the chip's eight dies in turn, so the remainder of a
// workgroup's number alone would tie every eighth chunk to one die, and all others would wait for
// the die that another kernel keeps busy.  With the quotient added, every eight workgroups in a row
// and every eight in a row on one die ask all eight counters.  (2^28 words while another kernel holds
// 16, 24, all 32 CUs of one die: 0.60 -> 0.41 ms, 1.09 -> 0.42 ms, done 356 -> 2 us after that kernel;
// alone 0.41 ms both.)
ZL_DEV constexpr uint32_t counter_of(uint32_t workgroup) { return (workgroup + workgroup / kCounters) % kCounters; }

// Byte j of the result is byte sel[j] of the eight bytes {hi, lo} (0..3 = lo, 4..7 = hi).
ZL_DEV constexpr uint32_t permute_bytes(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (!__builtin_is_constant_evaluated()) return __builtin_amdgcn_perm(hi, lo, sel);
#endif
  const uint64_t pool = ((uint64_t)hi << 32) | lo;
  uint32_t r = 0;
  for (int j = 0; j < 4; ++j) r |= (uint32_t)((pool >> (8 * ((sel >> (8 * j)) & 7u))) & 0xFFu) << (8 * j);
  return r;
}

// N = 32: the 32 x 32 bit transpose, out word k, bit j = in word j, bit k; its own inverse.
// N = 16: two 16 x 16 transposes side by side, out word k, bit j + 16*h = in word j, bit k + 16*h.
// The swaps of 16 and of 8 bits move whole bytes: one permute per word instead of a shift and a
// bit-field insert.
template <int N>
ZL_DEV constexpr void transpose(uint32_t (&a)[N]) {
  constexpr uint32_t mask[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
  int m = N == 32 ? 0 : 1;
#pragma unroll
  for (int s = N / 2; s >= 1; s >>= 1, ++m)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & s) == 0) {
        const uint32_t lo = a[i], hi = a[i + s];
        if (s >= 8) {
          a[i] = permute_bytes(hi, lo, s == 16 ? 0x05040100u : 0x06020400u);
          a[i + s] = permute_bytes(hi, lo, s == 16 ? 0x07060302u : 0x07030501u);
        } else {
          a[i] = (lo & mask[m]) | ((hi & mask[m]) << s);
          a[i + s] = ((lo >> s) & mask[m]) | (hi & ~mask[m]);
        }
      }
}

namespace selfcheck {
template <int N>
constexpr bool transpose_ok() {
  uint32_t a[N] = {}, ref[N] = {};
  uint32_t s = 0x2545F491u;
  for (int j = 0; j < N; ++j) { s = s * 1664525u + 1013904223u; a[j] = s; }
  for (int j = 0; j < N; ++j)
    for (int h = 0; h < 32; h += N)
      for (int k = 0; k < N; ++k) ref[k] |= ((a[j] >> (k + h)) & 1u) << (j + h);
  transpose<N>(a);
  for (int k = 0; k < N; ++k)
    if (a[k] != ref[k]) return false;
  return true;
}
static_assert(transpose_ok<32>() && transpose_ok<16>(), "bit transpose");
}  // namespace selfcheck

// Words of a group -> its reference (largest magnitude as a bit pattern), and in place the
// residuals sign | (reference - magnitude).  Returns the bitmap of the planes that are not empty,
// which is the residuals or-ed together: it is known before the transpose, after which register k
// is plane k.
ZL_DEV uint32_t to_residuals(uint32_t (&w)[32], uint32_t& reference) {
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    const uint32_t mag = w[j] & 0x7FFFFFFFu;
    m = mag > m ? mag : m;
  }
  uint32_t bitmap = 0;
#pragma unroll
  for (int j = 0; j < 32; ++j) {
    w[j] = (w[j] & 0x80000000u) | (m - (w[j] & 0x7FFFFFFFu));
    bitmap |= w[j];
  }
  reference = m;
  return bitmap;
}

// How many planes of a group are not empty, from its words one at a time (word(j), j = 0..31): two
// passes over them instead of 32 registers, for where a size is wanted without the group.
template <class Word>
ZL_DEV uint32_t planes_of_group(Word word) {
  uint32_t m = 0, bitmap = 0;
#pragma unroll 1
  for (int j = 0; j < 32; ++j) {
    const uint32_t mag = word(j) & 0x7FFFFFFFu;
    m = mag > m ? mag : m;
  }
#pragma unroll 1
  for (int j = 0; j < 32; ++j) {
    const uint32_t w = word(j);
    bitmap |= (w & 0x80000000u) | (m - (w & 0x7FFFFFFFu));
  }
  return (uint32_t)__builtin_popcount(bitmap);
}

// A group of 16-bit words v, coded as the 32-bit words v << 16: everything below bit 16 is zero, so
// the group is kept as 16 registers, word j in the lower and word j + 16 in the upper half of
// register j.  Reference and bitmap as the 32-bit form has them; after transpose<16> register k
// is plane 16 + k.
ZL_DEV uint32_t to_residuals_of_halves(uint32_t (&w)[16], uint32_t& reference) {
  typedef uint16_t Pair __attribute__((vector_size(4)));
  Pair m = __builtin_bit_cast(Pair, w[0] & 0x7FFF7FFFu);
#pragma unroll
  for (int j = 1; j < 16; ++j) {
    const Pair mag = __builtin_bit_cast(Pair, w[j] & 0x7FFF7FFFu);
    m = mag > m ? mag : m;
  }
  const uint16_t most = m[0] > m[1] ? m[0] : m[1];
  const Pair both = {most, most};
  uint32_t any = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const Pair distance = both - __builtin_bit_cast(Pair, w[j] & 0x7FFF7FFFu);
    w[j] = (w[j] & 0x80008000u) | __builtin_bit_cast(uint32_t, distance);
    any |= w[j];
  }
  reference = (uint32_t)most << 16;
  return (any | any << 16) & 0xFFFF0000u;
}

// Planes (absent ones as zero) and reference -> the words, in place.  The distance wraps
// within 31 bits, so residuals that no encoder produces still decode.
ZL_DEV void from_planes(uint32_t (&p)[32], uint32_t reference) {
  transpose(p);
#pragma unroll
  for (int j = 0; j < 32; ++j) p[j] = (p[j] & 0x80000000u) | ((reference - (p[j] & 0x7FFFFFFFu)) & 0x7FFFFFFFu);
}

}  // namespace zl
#endif  // ZL_CODEC_H
