// zc2d_codec.h -- per-block codec for 4 x 4 blocks ("ZC-2D"), as run by one GPU lane.
//
// Same codec family as zc_codec.h (the paper's lossy fixed-rate compressor of the ZFP
// kind, Sec. II-A, Sec. III-B) for matrix-shaped messages: shared exponent of the 16
// values, truncating conversion to 27 fraction bits, the reversible lifting transform
// along rows and then along columns, coefficients in order of total sequency,
// negabinary digits, and the embedded bit-plane code with 16 coefficients, cut at
// 16*RATE-8 bits behind a one-byte exponent header.
//
// How the bit-plane code is computed here:
//   * the words are aligned so that the first non-empty plane is bit 31, and their upper
//     halves are bit-transposed (a 16 x 16 transpose on eight registers that hold two
//     16-bit rows each), so that each of the first 16 planes is one 16-bit pattern in a
//     register; the lower halves are transposed only if some lane of the wavefront gets
//     that far within its budget, which low rates rarely do;
//   * the encoder's plane loop is unrolled, uniform over the wavefront, and ends when no
//     lane has budget left; the decoder's lanes go through their planes on their own,
//     one table look-up per step, and keep the patterns in LDS until they are
//     transposed;
//   * encoder: a plane is one code word, formed without a loop.  Past the coefficients
//     already significant, a zero is one bit 0 and a newly significant coefficient two
//     bits 1 (the end of its token and the next group bit), which two look-ups, one per
//     byte of the plane, write down in place; the topmost of these bits is a group bit 0;
//   * decoder: a table indexed by the next 9 stream bits and by how far the last
//     coefficient is (whose token has no closing one) decodes all the tokens that lie
//     whole within those bits.  The window is zero past the budget, which decodes to
//     what unseen bits are but for a run cut by the budget (its one goes to the lowest
//     index still possible); entries where that can matter are marked, and where it
//     does, one token is decoded by count-trailing-zeros with the limits applied;
//   * after the planes, the usual case (at most 16 planes read, starting within the top
//     16) turns each coefficient's 16-bit pattern into its word with one shift.
#ifndef ZC2D_CODEC_H
#define ZC2D_CODEC_H

#include <assert.h>
#include "zc_codec.h"

namespace zc2d {

using zc::alignbit;
using zc::umin;
using zc::umax;
using zc::count_leading_zeros;
using zc::count_leading_zeros_nonzero;
using zc::count_trailing_zeros;
using zc::count_trailing_zeros_nonzero;

constexpr int kFractionBits = 27;

template <int RATE>
struct Traits {
  static_assert(RATE == 2 || RATE == 4 || RATE == 8 || RATE == 16, "rate");
  static constexpr int kBlockBits = 16 * RATE;
  static constexpr int kBlockBytes = 2 * RATE;
  static constexpr int kPayloadBits = 16 * RATE - 8;
  static constexpr int kWords = RATE / 2;
};

// Position of coefficient c in the 4 x 4 array (4*i + j, i = row frequency, j = column
// frequency): ascending i + j, ties by ascending i.
struct Order { int v[16]; };
constexpr Order build_order() {
  Order o{};
  int c = 0;
  for (int s = 0; s <= 6; ++s)
    for (int i = 0; i < 4; ++i) {
      int j = s - i;
      if (j >= 0 && j < 4) o.v[c++] = 4 * i + j;
    }
  return o;
}
constexpr Order kOrder = build_order();

// bits of a where mask is set, of b elsewhere (bit operations of three operands take the GPU half as
// long as its bit-field insert, as long as all three are in vector registers)
ZC_DEV constexpr uint32_t select_bits(uint32_t mask, uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (!__builtin_is_constant_evaluated()) return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA);
#endif
  return (a & mask) | (b & ~mask);
}

// the same of a and ~b
ZC_DEV constexpr uint32_t select_bits_not(uint32_t mask, uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (!__builtin_is_constant_evaluated()) return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xC5);
#endif
  return (a & mask) | (~b & ~mask);
}

// ---- 16 x 16 bit transpose on eight words ----------------------------------------------
// Row r of a 16 x 16 bit matrix sits in half r >> 3 of word r & 7 (half 0 = bits 0..15).
// The transpose leaves the matrix in the same arrangement, so it is its own inverse.
// The encoder makes its words with the 8 x 8 quadrants in their places already (swap_quadrants),
// which is then one permute per word in all.
// (Cycles of the GPU: 38 for each of the three steps, one shift to the left for two words at a time, masks in
// vector registers.  A shift per word and masks in scalar registers took 67, the encoder's bit operations
// for the quadrants 50 in all.)

// Masks that operations of three operands take from vector registers: from scalar ones such an operation takes the
// GPU 4.2 cycles instead of 2.5.
struct SwapMasks { uint32_t v[3]; };
ZC_DEV constexpr SwapMasks swap_masks() {
  SwapMasks m = {{0x0F0F0F0Fu, 0x33333333u, 0x55555555u}};
  if (!__builtin_is_constant_evaluated())
    for (int i = 0; i < 3; ++i) zc::materialise(m.v[i]);
  return m;
}

// a and b shifted to the left by LG, the bits that a loses at b's lower end (one instruction, as long as one for a
// single word); with LG = 1 each by itself, as an addition.
template <int LG>
ZC_DEV void shift_left_two_here(uint32_t& a, uint32_t& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (LG == 1) {
    asm("v_add_u32 %0, %1, %1" : "=v"(a) : "v"(a));
    asm("v_add_u32 %0, %1, %1" : "=v"(b) : "v"(b));
  } else {
    uint64_t both = (uint64_t)b << 32 | a;
    asm("v_lshlrev_b64 %0, %1, %2" : "=v"(both) : "n"(LG), "v"(both));
    a = (uint32_t)both;
    b = (uint32_t)(both >> 32);
  }
#else
  b = b << LG | (LG == 1 ? 0u : a >> (32 - LG));
  a <<= LG;
#endif
}
template <int LG>
ZC_DEV constexpr void shift_left_two(uint32_t& a, uint32_t& b) {
  if (!__builtin_is_constant_evaluated()) {
    shift_left_two_here<LG>(a, b);
  } else {
    b = b << LG | (LG == 1 ? 0u : a >> (32 - LG));
    a <<= LG;
  }
}

ZC_DEV constexpr void swap_quadrants(uint32_t (&a)[8]) {
  // bits 8..15 of row r with bits 0..7 of row r + 8 (the two middle bytes of each word change places)
#pragma unroll
  for (int w = 0; w < 8; ++w) a[w] = zc::permute_bytes(a[w], a[w], 0x03010200u);
}

// JLG = 2, 1, 0: the 4 x 4, 2 x 2 and 1 x 1 blocks between words j = 2^JLG apart; each mask's complement is the
// mask shifted up by j, and so is what the words of a pair leave at each other's lower end.
template <int JLG>
ZC_DEV constexpr void swap_blocks(uint32_t (&a)[8], const SwapMasks& masks) {
  constexpr int j = 1 << JLG;
  const uint32_t mask = masks.v[2 - JLG];
#pragma unroll
  for (int w = 0; w < 8; ++w)
    if ((w & j) == 0 && (JLG == 0 ? (w & 2) == 0 : (w & 1) == 0)) {
      const int v = w + (JLG == 0 ? 2 : 1);   // two words at a time, w and v
      const uint32_t lo0 = a[w], lo1 = a[v], hi0 = a[w + j], hi1 = a[v + j];
      uint32_t up0 = hi0, up1 = hi1;
      shift_left_two<j>(up0, up1);
      a[w] = select_bits(mask, lo0, up0);
      a[v] = select_bits(mask, lo1, up1);
      a[w + j] = select_bits(mask, lo0 >> j, hi0);
      a[v + j] = select_bits(mask, lo1 >> j, hi1);
    }
}
ZC_DEV constexpr void swap_all_blocks(uint32_t (&a)[8]) {
  const SwapMasks masks = swap_masks();
  swap_blocks<2>(a, masks);
  swap_blocks<1>(a, masks);
  swap_blocks<0>(a, masks);
}
ZC_DEV constexpr void transpose_halves(uint32_t (&a)[8]) {
  swap_quadrants(a);
  swap_all_blocks(a);
}

// ---- tables --------------------------------------------------------------------------
// Encoder.  Behind a plane's first group bit, a coefficient that is still zero is one bit 0 and
// one that becomes significant is two bits 1: the end of its token and the next group bit; the last
// coefficient has neither, and is one bit 1 here, which only marks where the code ends.  Both tables hold
// that expansion X(c) of eight coefficients c, for the two bytes of a plane without the coefficients
// already significant.  These are zeros in it, one bit each, which is the room that their own bits take
// before the group bit: so a byte's place does not depend on how many they are.  v[c], the lower byte: X(c) from
// bit 1 up (the group bit lies below the first coefficient that is not yet significant), and in the
// upper half how far the upper byte's expansion moves up to follow it, 8 + (ones of c), from bit 20 up.
// v[256 + c], the upper byte: X(c) from bit 1 up.
constexpr int kExpandEntries = 512;
constexpr uint32_t kExpandBits = 0x1FFFFu;
constexpr int kExpandShift = 20;
struct ExpandTable { uint32_t v[kExpandEntries]; };
constexpr ExpandTable build_expand_table() {
  ExpandTable t{};
  for (int c = 0; c < 256; ++c) {
    uint32_t e = 0, at = 0;
    for (int p = 0; p < 8; ++p) {
      if ((c >> p) & 1) e |= 3u << at++;
      ++at;
    }
    t.v[c] = e << 1 | at << kExpandShift;
    t.v[256 + c] = (c & 0x80 ? e ^ 1u << (at - 1) : e) << 1;   // (the last coefficient's second bit)
  }
  return t;
}

// Decoder: entry for the next kLookahead stream bits at the start of a group test, by how far
// the last coefficient is.  With n the index of the first coefficient not yet known to be
// significant, the row is clamp(n, 6, 16) - 6: row 0 serves the indices up to 6, from where the
// last coefficient cannot be reached within the look-ahead; rows 1..9 are the indices 7..15 (8..0
// coefficients between the current one and the last); row 10 is that of a plane with nothing left
// to test, which it closes without reading anything.
// An entry holds all the tokens that lie whole within the look-ahead: group bit, zeros,
// closing one; a run that reaches the last coefficient needs no closing one, and the plane is
// closed after it; a group bit 0 closes the plane.
// Where these are a group bit 1 and zeros only, and the last coefficient is not among them, the entry passes the eight zeros and
// leaves the group bit to the next step, in the place of the last of them.
// Byte 0: how many bits of budget the entry must find; kTokenGoesOn, which is where the window has the last of the eight zeros, if a
// group bit has to be put there; from bit kIndexShift on, where n is kept: how many coefficients were passed; byte 2: the ones, as
// positions past the current coefficient; byte 3: how many stream bits were used, and bit 31 if the plane is closed (bits 29 and 30
// are zeros).
// (What lies below kIndexShift adds up in n's lower bits over a block, and must not reach kIndexShift: kTokenGoesOn occurs once
// at most, since it passes eight of sixteen coefficients and leaves the last, and each entry with a byte 0 passes one at least.)
// Bits past the budget are zeros in the decoder's window, and what they decode to there is right
// everywhere but in one place: zeros after a group bit 1 would put the one on the last
// coefficient, where a run cut by the budget has it at the lowest index still possible.  So
// byte 0 is the bits looked at if the entry holds a run that reaches the last coefficient without a closing one, or does not
// reach its end, and zero otherwise.
constexpr int kLookahead = 9;
constexpr int kTokenRows = 11;
constexpr uint32_t kTokenFirstRowIndex = 6;
constexpr uint32_t kTokenClosed = 0x80000000u, kTokenGoesOn = 4u << (kLookahead - 1);
constexpr int kIndexShift = kLookahead + 2;   // n, times the bytes of a row
static_assert(kTokenGoesOn + 16 * kLookahead < 1u << kIndexShift, "nothing is carried into n");
struct TokenTable { uint32_t v[kTokenRows << kLookahead]; };
constexpr TokenTable build_token_table() {
  TokenTable t{};
  for (uint32_t row = 0; row + 1 < (uint32_t)kTokenRows; ++row) {
    // coefficients between the current one and the last; row 0 stands for nine and more
    const uint32_t room = row == 0 ? 15u : 9u - row;
    for (uint32_t s = 0; s < (1u << kLookahead); ++s) {
      uint32_t ones = 0, passed = 0, used = 0, closed = 0, to_last = 0;
      for (;;) {
        if (passed > room) { closed = kTokenClosed; break; }   // the last coefficient has been dealt with
        if (used >= (uint32_t)kLookahead) break;
        if (((s >> used) & 1u) == 0u) { closed = kTokenClosed; ++used; break; }
        uint32_t z = 0;
        bool in_sight = true;
        while (passed + z < room) {
          if (used + 1 + z >= (uint32_t)kLookahead) { in_sight = false; break; }
          if ((s >> (used + 1 + z)) & 1u) break;
          ++z;
        }
        if (!in_sight || passed + z > 7u) break;
        ones |= 1u << (passed + z);
        if (passed + z == room) to_last = 1;
        used += 1 + z + (passed + z == room ? 0 : 1);       // no closing one at the last coefficient
        passed += z + 1;
      }
      uint32_t need = to_last ? used : 0u;
      if (used == 0u) {   // (s is 1)
        passed = used = kLookahead - 1;
        need = kLookahead | kTokenGoesOn;
      }
      t.v[(row << kLookahead) + s] = need | passed << kIndexShift | ones << 16 | used << 24 | closed;
    }
  }
  for (uint32_t s = 0; s < (1u << kLookahead); ++s) t.v[((kTokenRows - 1) << kLookahead) + s] = kTokenClosed;
  return t;
}

namespace selfcheck {
constexpr bool transpose_ok() {
  uint32_t a[8] = {}, ref[8] = {};
  uint32_t s = 0x9E3779B9u;
  for (int w = 0; w < 8; ++w) { s = s * 1664525u + 1013904223u; a[w] = s; }
  for (int r = 0; r < 16; ++r)
    for (int b = 0; b < 16; ++b)
      ref[b & 7] |= ((a[r & 7] >> (16 * (r >> 3) + b)) & 1u) << (16 * (b >> 3) + r);
  transpose_halves(a);
  for (int w = 0; w < 8; ++w)
    if (a[w] != ref[w]) return false;
  return true;
}
static_assert(transpose_ok(), "16 x 16 bit transpose");
}  // namespace selfcheck

// ---- forward ---------------------------------------------------------------------------

ZC_DEV void lift_forward(int32_t& a, int32_t& b, int32_t& c, int32_t& d) {
  d -= a; a += d >> 1;
  b -= c; c += b >> 1;
  c -= a; a += c >> 1;
  b -= d; d += b >> 1;
  d += b >> 2; b -= d;
}

// x: the block row-major as fp32 bit patterns.  Returns E and the negabinary words in
// coefficient order.  E is the exponent field of the largest magnitude plus one, also where that is zero.
// The result says whether some block of the wavefront is a tiny one, whose largest magnitude is below 2^-101 and not zero.
template <class AnyActive>
ZC_DEV bool forward_transform(const uint32_t (&x)[16], uint32_t& E, uint32_t (&u)[16], AnyActive any_lane_active) {
  // largest magnitude as a bit pattern (on the device a float maximum with |x| operands, as in
  // the 1-D codec: the same pattern for finite values, a third of the instructions)
#if defined(__HIP_DEVICE_COMPILE__)
  float mf = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; i += 2)
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(mf) : "v"(mf), "v"(zc::bits_to_float(x[i])), "v"(zc::bits_to_float(x[i + 1])));
  const uint32_t m = __builtin_bit_cast(uint32_t, mf);
#else
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) m = umax(m, x[i] & 0x7FFFFFFFu);
#endif
  E = (m >> 23) + 1u;
  int32_t q[16];
  const bool tiny = any_lane_active(m - 1u < (26u << 23) - 1u);
  if (tiny) {
    const int scale = 127 + kFractionBits - (int)E;
#pragma unroll
    for (int i = 0; i < 16; ++i) q[i] = (int32_t)__builtin_ldexpf(zc::bits_to_float(x[i]), scale);
  } else {
    // the power of two is a float (for a zero block some finite number), and a multiplication takes the GPU half
    // as long as its ldexp (us before and after: 2-way reduce of 8192 x 32768 values at rate 8 604.8 and 598, compress2d of
    // 8192 x 6144 bf16 values 53.9 and 52.1)
    const float scale = zc::bits_to_float(((253u + kFractionBits) << 23) - (m & 0x7F800000u));
#pragma unroll
    for (int i = 0; i < 16; ++i) q[i] = (int32_t)(zc::bits_to_float(x[i]) * scale);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) lift_forward(q[4 * r], q[4 * r + 1], q[4 * r + 2], q[4 * r + 3]);
#pragma unroll
  for (int c = 0; c < 4; ++c) lift_forward(q[c], q[4 + c], q[8 + c], q[12 + c]);
#pragma unroll
  for (int c = 0; c < 16; ++c) u[c] = ((uint32_t)q[kOrder.v[c]] + 0xAAAAAAAAu) ^ 0xAAAAAAAAu;
  return tiny;
}

// Constants of encode_plane that are wanted in vector registers (see SwapMasks).
struct PlaneConstants { uint32_t expand_bits, top, ones; };
ZC_DEV PlaneConstants plane_constants() {
  PlaneConstants k = {kExpandBits, 0x80000000u, 0xFFFFFFFFu};
  zc::materialise(k.expand_bits);
  zc::materialise(k.top);
  zc::materialise(k.ones);
  return k;
}

// One plane of the embedded code, appended to the window W as one code word: the bits of the
// coefficients already significant, then the group tests.  plane: the plane's bit of each
// coefficient, in its lower half or (UPPER) in its upper half; sig: ones for the leading coefficients that are significant;
// left: budget.
// The tokens' starts and ends come from two look-ups (see ExpandTable) without any case
// distinction: the topmost bit of the expansion is the group bit after the last one, or the
// plane's only one, and both are zeros in the code, which is as long as that bit's place tells.  With the last coefficient
// significant (its bit of sig, before or by this plane) that bit is no part of the code.  The length is at most 31.
// (Cycles of the GPU per plane at rate 4, at 2.3 for additions, shifts to the right, bit operations and 16-bit
// operations and 4.3 for anything else and whatever has an operand in a scalar register: 68.  With the pattern moved down by the
// significant coefficients and the code word up again, and the length counted where the last coefficient is
// reached, it was 93.  us before and after, with the transpose and the alignment as they are now: compress2d of 8192 x 32768
// values at rate 4 218 and 205, at rate 8 267 and 234, at rate 16 424 and 345, 8192 x 6144 bf16 values at rate 8 53.5 and 48.2, 64 x 256
// values at rate 16 4.25 and 3.65; 2-way reduce of 8192 x 32768 values at rate 4 430 and 414, at rate 8 593 and 562, at rate 16 1138 and
// 1050.)
template <bool UPPER, int NW>
ZC_DEV void encode_plane(uint32_t plane, const uint32_t* expand, const PlaneConstants& k, uint32_t (&W)[NW], uint32_t& sig, uint32_t& left) {
  const uint32_t pat = UPPER ? plane >> 16 : plane;
  const uint32_t rest = UPPER ? pat & ~sig : pat & ~sig & 0xFFFFu;
  const uint32_t lo = expand[rest & 0xFFu], hi = expand[256u + (rest >> 8)];
  const uint32_t tokens = zc::and_or(lo, k.expand_bits, sig + 1u) | hi << (lo >> kExpandShift);
  const uint32_t c = count_leading_zeros_nonzero(tokens);
  const uint32_t code = zc::and_or(pat, sig, tokens ^ (k.top >> c));
  sig = k.ones >> (count_leading_zeros_nonzero(sig | rest) & 31u);
  const uint32_t take = zc::umin16(32u - c - (sig >> 15), left);
  zc::shift_in<NW>(W, code, take);
  left -= take;
}

template <int RATE, class AnyActive>
ZC_DEV void encode_block(const uint32_t (&x)[16], const uint32_t* expand, uint32_t (&W)[Traits<RATE>::kWords],
                         AnyActive any_lane_active) {
  constexpr int NW = Traits<RATE>::kWords;
  constexpr int kPayload = Traits<RATE>::kPayloadBits;
  constexpr int kMaxPlanes = kPayload < 32 ? kPayload : 32;
  // in the first so many planes hardly a block of ordinary values spends its budget (on gradients, activations and parameters the first
  // of 64 blocks does in plane 3, 7 and 15 at rates 4, 8 and 16, the last in 6, 10 and 18), so it is asked from there on
  // (and at first, for wavefronts of zero blocks)
  constexpr int kUnasked = kPayload / 20;
  uint32_t E, u[16];
  const bool tiny = forward_transform(x, E, u, any_lane_active);
  uint32_t any = zc::or3(u[0], u[1], u[2]);
#pragma unroll
  for (int c = 3; c < 15; c += 2) any = zc::or3(any, u[c], u[c + 1]);
  const uint32_t raw = count_leading_zeros_nonzero(any | u[15]);
  E &= ~(uint32_t)((int32_t)raw >> 31);             // (the zero block)
  uint32_t lead = zc::umin16(raw, (uint32_t)kPayload);   // empty planes: one zero bit each
  uint32_t left = (uint32_t)kPayload - lead;
#pragma unroll
  for (int j = 0; j < NW; ++j) W[j] = 0;
  if (any_lane_active(left > 0)) {
    uint32_t h[8], sig = 0u;
    // the first non-empty plane to bit 31, or, where mostly sixteen planes or less are coded, to bit 15: shifts to the right take the
    // GPU half as long.  These need lead to be 16 at most, and but for tiny blocks (and zero ones) it is 8: the largest of the 16
    // numbers is 2^26 or more, the inverse transform makes no number larger than 2.25 times 2.25 times the largest coefficient (but for
    // what the halvings drop, less than 2^5), so that one coefficient is 2^23 or more, which takes a digit at bit 23 or above.
    constexpr bool kDown = RATE <= 8;
    if constexpr (kDown) {
#if !defined(__HIP_DEVICE_COMPILE__)
      assert(tiny || raw >= 32u || raw <= 8u);
#endif
      if (tiny) {
#pragma unroll
        for (int c = 0; c < 16; ++c) u[c] <<= umax(lead & 31u, 16u) - 16u;
        lead = umin(lead, 16u);
      }
      const uint32_t down = 16u - lead;
#pragma unroll
      for (int w = 0; w < 8; ++w) h[w] = zc::permute_bytes(u[w + 8] >> (down & 31u), u[w] >> (down & 31u), 0x05010400u);
    } else {
#pragma unroll
      for (int c = 0; c < 16; ++c) u[c] <<= (lead & 31u);
#pragma unroll
      for (int w = 0; w < 8; ++w) h[w] = zc::permute_bytes(u[w + 8], u[w], 0x07030602u);
    }
    const PlaneConstants k = plane_constants();
    swap_all_blocks(h);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      if (t >= kMaxPlanes || (t >= kUnasked && !any_lane_active(left > 0))) break;
      if (t < 8) encode_plane<true, NW>(h[7 - t], expand, k, W, sig, left);
      else encode_plane<false, NW>(h[15 - t], expand, k, W, sig, left);
    }
    if (kMaxPlanes > 16 && any_lane_active(left > 0)) {
      if constexpr (kDown) {
#pragma unroll
        for (int c = 0; c < 16; ++c) u[c] <<= (lead & 31u);
      }
#pragma unroll
      for (int w = 0; w < 8; ++w) h[w] = zc::permute_bytes(u[w + 8], u[w], 0x05010400u);
      swap_all_blocks(h);
#pragma unroll
      for (int t = 16; t < 32; ++t) {
        if (t >= kMaxPlanes || !any_lane_active(left > 0)) break;
        if (t < 24) encode_plane<true, NW>(h[23 - t], expand, k, W, sig, left);
        else encode_plane<false, NW>(h[31 - t], expand, k, W, sig, left);
      }
      static_assert(32 * NW == Traits<RATE>::kBlockBits, "the window is the block");
      if (any_lane_active(left > 0)) zc::shift_right<NW>(W, left);
    }
  }
  W[0] |= E;
}

// ---- inverse -----------------------------------------------------------------------------

// Negabinary words in coefficient order -> the block's fixed-point values, row-major.
ZC_DEV void inverse_transform(uint32_t (&u)[16], int32_t (&q)[16]) {
#pragma unroll
  for (int c = 0; c < 16; ++c) q[kOrder.v[c]] = zc::negabinary_to_int(u[c]);
#pragma unroll
  for (int c = 0; c < 4; ++c) zc::inverse_lift(q[c], q[4 + c], q[8 + c], q[12 + c]);
#pragma unroll
  for (int r = 0; r < 4; ++r) zc::inverse_lift(q[4 * r], q[4 * r + 1], q[4 * r + 2], q[4 * r + 3]);
}

// Fixed-point values -> fp32: int -> fp32 rounds to nearest even, the scaling by
// 2^(E - 127 - 27) is exact and rounds once more only for subnormal results.
ZC_DEV void scale_block(const int32_t (&q)[16], uint32_t E, float (&out)[16]) {
  const int ex = (int)E - 127 - kFractionBits;
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] = __builtin_ldexpf((float)q[i], ex);
}

// sum += the block's fp32 values, for exponent bytes where the scaling is exact and finite
// (see scaling_is_exact): the product of the rounded integer and the power of two is then the
// decoded value itself, and the fused multiply-add rounds the sum once, as the addition would.
ZC_DEV void accumulate_scaled(const int32_t (&q)[16], uint32_t E, float (&sum)[16]) {
  const float scale = __builtin_ldexpf(1.0f, (int)E - 127 - kFractionBits);
#pragma unroll
  for (int i = 0; i < 16; ++i) sum[i] = __builtin_fmaf((float)q[i], scale, sum[i]);
}

// Nonzero values have magnitude 1 .. 2^31 before scaling: from E = 28 on none of them becomes
// subnormal, up to E = 250 none overflows.  In the zero block (E = 0) all values are zero, and
// zero times anything finite added to the sum is the sum plus zero.
ZC_DEV bool scaling_is_exact(uint32_t E) { return E - 28u <= 222u || E == 0u; }

// Whether p or q holds in some lane (each comparison's own result is a set of lanes, and sets combine for
// free on the device).
template <class AnyActive>
ZC_DEV bool any_of(AnyActive any_lane_active, bool p, bool q) {
#if defined(__HIP_DEVICE_COMPILE__)
  (void)any_lane_active;
  return (__builtin_amdgcn_ballot_w64(p) | __builtin_amdgcn_ballot_w64(q)) != 0;
#else
  return any_lane_active(p || q);
#endif
}

// Where a lane's decoded planes go: sixteen 16-bit patterns, in the order they are read, that
// start as zeros.  Places are kPlaneStep apart, from begin() to end(), where a pattern may be put as
// well; word k is patterns 2k and, above it, 2k + 1.  This one is for the host.
constexpr uint32_t kPlaneStep = 2;   // (a closed token's two top bits)
struct LocalPlanes {
  uint16_t v[17];
  ZC_DEV void clear() { for (int t = 0; t < 16; ++t) v[t] = 0; }
  ZC_DEV uint32_t begin() const { return 0u; }
  ZC_DEV uint32_t end() const { return 16 * kPlaneStep; }
  ZC_DEV void put(uint32_t at, uint32_t pattern) { v[at / kPlaneStep] = (uint16_t)pattern; }
  ZC_DEV uint32_t word(int k) const { return v[2 * k] | (uint32_t)v[2 * k + 1] << 16; }
};

// `width` bits of v from bit `offset` on (offset below 32, width below 32; none for width 0).
ZC_DEV uint32_t bit_field(uint32_t v, uint32_t offset, uint32_t width) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ubfe(v, offset, width);
#else
  return (v >> (offset & 31u)) & ((1u << (width & 31u)) - 1u);
#endif
}

// Byte 2 of e, moved up by n.
ZC_DEV uint32_t shifted_byte2(uint32_t e, uint32_t n) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint32_t r;
  asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(n), "v"(e));
  return r;
#else
  return ((e >> 16) & 0xFFu) << n;
#endif
}

// Drops `len` bits (its lower six bits, below 32) at the bottom of the window; the two top words by one shift of 64
// bits, which takes the GPU as long as the one that joins two words.  (In the 1-D decoder it does not pay: 2-way reduce of 2^27
// values at rate 16 282 and 287 us.)
template <int NW>
ZC_DEV void drop_bits(uint32_t (&W)[NW], uint32_t len) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int j = 0; j < NW - 2; ++j) W[j] = alignbit(W[j + 1], W[j], len);
  if constexpr (NW == 1) {
    W[0] >>= len & 31u;
  } else {
    uint64_t top = (uint64_t)W[NW - 1] << 32 | W[NW - 2];
    asm("v_lshrrev_b64 %0, %1, %0" : "+v"(top) : "v"(len));   // (the compiler makes the lower word once more)
    W[NW - 2] = (uint32_t)top;
    W[NW - 1] = (uint32_t)(top >> 32);
  }
#else
  zc::shift_out<NW>(W, len & 31u);
#endif
}

// A lane's progress through its block's planes.
template <int NW>
struct PlaneReader {
  uint32_t (&W)[NW];   // the window: what is not yet read, from bit 2 on, zeros past the budget
  int32_t left;        // budget, which zeros read past its end make negative
  uint32_t n;          // how many leading coefficients are significant, from bit kIndexShift on (16 bits; what lies below has no meaning)
  uint32_t pattern;    // the ones of the current plane found so far
  uint32_t at;         // the current plane's place
};

// Reads planes, from the bottom of the window, until no lane has budget left or, in the plain
// form, some lane has read sixteen, or, in the CAREFUL one, all lanes with budget left have (a lane
// that has them then waits for the others, which the plain form does not provide for).
//
// Lanes go through their planes on their own: a step is one look-up in the token table and, in
// lanes that close a plane, the bits of the significant coefficients of the next one (9 + 16 bits are in
// the window's first word).  A lane out of budget goes on reading empty planes.  The current
// plane's pattern is put in its place in every step, whether it is whole or not: LDS writes are
// what this kernel has to spare, and it takes no test.  (What a lane has at the end of a plane begun by its last step
// is left to the caller.)  Only if some lane's entry asks for more
// budget than the lane has, an entry for one token is made for it by count-trailing-zeros with the
// limits applied.
// (What bounds the 4 x 4 kernels is their instruction count, and here the number of steps that
// the wavefront's slowest lane needs.  Plane by plane in step, the patterns in registers, that was
// 11.1 steps at rate 4 and 14.3 at rate 8 on the gradient matrix, as the sum over planes of the
// slowest lane's; this way, the slowest lane's sum, it is 6.7 and 10.4: 578 -> 529 instructions
// per block and 0.253 -> 0.233 ms for decompress2d of 8192 x 32768 values at rate 4 with the stream in
// the last-level cache, 0.278 -> 0.248 ms with streams from memory and with what else changed in the
// decoder, 0.623 -> 0.572 ms for the 2-way reduce.  A step of about 22 instructions instead of 28, without a vote on the places left and with a lane's
// planes on end in LDS: decompress2d at rate 16 120 -> 112 us for 8192 x 8192 values, 2-way reduce 328 ->
// 314 us, at rate 4 8192 x 32768 values 490 -> 469 us.  With the significant coefficients' bits taken when a plane closes
// and not when the next one starts, so that the look-up's bits are where the table wants them, a step is about
// 66 cycles instead of 87: 469 -> 457 us, at rate 8 641 -> 623, decompress2d of 8192 x 8192 values at rate 16 112 ->
// 108, the reduce of one chunk and local values there 222 -> 207.  With n kept where the row's offset has it, a mask in the place
// of comparisons and selections, 16-bit operations and the last two words moved by one shift, so that
// fewer of a step's instructions are slow ones, 58 cycles, and with no vote in the first steps: 2-way reduce of 8192 x 32768 values at
// rate 4 414 -> 400 us, at rate 8 561 -> 538, at rate 16 1050 -> 1003, decompress2d of 8192 x 6144 bf16 values at rate 8 46.1 -> 43.9,
// at rate 16 fp32 87.6 -> 82.7.)
template <bool CAREFUL, int NW, class AnyActive, class Planes>
ZC_DEV void read_planes(const uint32_t* token, PlaneReader<NW>& r, Planes& planes, AnyActive any_lane_active) {
  // byte offset of the entry: (clamped index - first row's index) rows, then the next bits
  uint32_t bits_mask = ((1u << kLookahead) - 1u) << 2, goes_on = kTokenGoesOn;   // (the next bit is bit 2 of the window)
  zc::materialise(bits_mask);   // (in vector registers, see SwapMasks)
  zc::materialise(goes_on);
  // Up to rate 8 (NW <= 4) few blocks take sixteen steps, and in as many no lane can pass its
  // sixteenth place: the plain form counts them.  At rate 16 it asks whether some lane has got there.
  constexpr bool kCounted = !CAREFUL && NW <= 4;
  // a step takes 25 bits at most and half as many mostly, so the first ones leave most lanes some: these are not asked
  constexpr uint32_t kUnasked = NW == 8 ? 9u : (NW == 4 ? 5u : (NW == 2 ? 3u : 1u));
  uint32_t n = r.n >> kIndexShift;
  auto step = [&]() {
    const bool reading = !CAREFUL || r.at != planes.end();
    uint32_t e = 0u;
    bool cut = false;
    if (reading) {
      const uint32_t row = zc::umax16<kTokenFirstRowIndex << kIndexShift>(r.n) & (0xFFFFu << kIndexShift);
      const uint32_t offset = select_bits(bits_mask, r.W[0], row) - (kTokenFirstRowIndex << kIndexShift);
      e = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(token) + offset);
      cut = (e & 0xFFu) > (uint32_t)r.left;   // (no budget at all: the window is empty, and so is byte 0)
    }
    if (any_lane_active(cut)) {
      // zeros up to the one; the run ends at the last coefficient or at the budget (of which some is
      // left: the group bit is a one).  The one may be too far on for an entry.  (Runs that are longer than the look-ahead did not
      // have entries: 2.2 of the 5.7 steps of a wavefront at rate 4, and of the 9.4 at rate 8, came here for such a
      // one, at 54 cycles; now it is 1.1 at rate 4 and hardly any at rate 8: 2-way reduce of 8192 x 32768 values at rate 4
      // 396 -> 380 us, at rate 8 524 -> 510, decompress2d of 8192 x 6144 bf16 values at rate 8 43.2 -> 42.4.)
      const uint32_t room = umin(15u - n, (uint32_t)r.left - 1u);
      const uint32_t z = umin(count_trailing_zeros(r.W[0] >> 3), room);
      const uint32_t made = (z + 1u) << kIndexShift | (1u + z + (z < room ? 1u : 0u)) << 24;
      e = cut ? made : e;
      r.pattern |= cut ? 1u << ((n + z) & 31u) : 0u;
    }
    if (reading) {
      r.pattern |= shifted_byte2(e, n);
      planes.put(r.at, r.pattern);
      r.n = zc::add16(r.n, e);
      n = r.n >> kIndexShift;
      // a closed plane: the next one's bits of the significant coefficients
      const uint32_t closed = (uint32_t)((int32_t)e >> 31), verbatim = n & closed;
      uint32_t used = e >> 24;   // (shifts and fields look at its lower five bits)
      zc::materialise(used);     // (a shift and two additions are faster than two additions of a byte)
      r.pattern = select_bits(closed, bit_field(r.W[0], used + 2u, n), r.pattern);
      zc::materialise(r.pattern);   // (before the window moves)
      r.at += e >> 30;
      const uint32_t taken = used + verbatim;
      r.W[0] = zc::and_or(e, goes_on, r.W[0]);   // (behind the shift it cost a wait for that: 64 x 256 constant values at rate 16 8.68 and 8.41 us)
      drop_bits<NW>(r.W, taken);
      r.left -= (int32_t)(taken & 31u);
    }
  };
  if (CAREFUL) {
#pragma unroll 1
    do step(); while (any_lane_active(r.left > 0 && r.at != planes.end()));
  } else {
#pragma unroll 1
    for (uint32_t steps = 0; steps < kUnasked; ++steps) step();
    uint32_t steps = 16u - kUnasked;
    if (kCounted) {
#pragma unroll 1
      do step(); while (any_lane_active(r.left > 0) && --steps != 0u);
    } else {
#pragma unroll 1
      do step(); while (any_lane_active(r.left > 0) && !any_lane_active(r.at == planes.end()));
    }
  }
}

// A block whose planes have been read: its exponent byte, the empty planes before the first one, and
// where reading stopped.  An empty block (a zero exponent byte, or 32 and more empty planes) has
// neither planes nor budget and counts as three empty planes under the exponent byte of 1.
template <int NW>
struct BlockReading {
  uint32_t E, lead;
  bool low_start;        // planes that start more than 16 below the top (and any to read)
  PlaneReader<NW> r;
};
constexpr uint32_t kEmptyLead = 3u, kEmptyExponent = 127u;

// After read_planes: a lane whose budget ended within the bits of significant coefficients has these in a
// plane that no step has put in its place.  If that is a seventeenth, it is marked as budget left.
template <int NW, class AnyActive, class Planes>
ZC_DEV void put_begun_plane(PlaneReader<NW>& r, Planes& planes, AnyActive any_lane_active) {
  planes.put(r.at, r.pattern);
  if (any_lane_active(r.at == planes.end()))
    r.left = r.at == planes.end() && r.pattern != 0u && r.left <= 0 ? 1 : r.left;
}

// Reads the first (up to sixteen) planes of the block in the window W.
template <int RATE, class AnyActive, class Planes>
ZC_DEV BlockReading<Traits<RATE>::kWords> read_block(uint32_t (&W)[Traits<RATE>::kWords], const uint32_t* token,
                                                     AnyActive any_lane_active, Planes& planes) {
  constexpr int NW = Traits<RATE>::kWords;
  constexpr int kPayload = Traits<RATE>::kPayloadBits;
  uint32_t E = W[0] & 0xFFu;
  // empty planes before the first one: zeros from bit 8 on, which seldom pass the first word
  const uint32_t top = W[0] & 0xFFFFFF00u;
  uint32_t lead = count_trailing_zeros_nonzero(top) - 8u;
  bool empty = false;
  if (any_of(any_lane_active, top == 0u, E == 0u)) {
    lead = 0;
    bool found = false;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      const uint32_t w = j == 0 ? top : W[j];
      const uint32_t z = count_trailing_zeros(w);
      lead = found ? lead : lead + z;
      found = found || (w != 0);
    }
    lead = umin(lead - 8u, (uint32_t)kPayload);
    empty = E == 0u || lead >= 32u;
  }
  int32_t left = (int32_t)kPayload - (int32_t)lead;
  // past the header byte and the leading zeros but for two bits: two shifts of less than 32 each (with 32 and
  // more leading zeros there is nothing to read, as in a zero block, whatever its payload)
  zc::shift_out<NW>(W, 6u);
  zc::shift_out<NW>(W, lead & 31u);
  if (any_lane_active(empty)) {
    if (empty) {
      left = 0;
      lead = kEmptyLead;
      E = kEmptyExponent;
#pragma unroll
      for (int j = 0; j < NW; ++j) W[j] = 0u;
    }
  }
  BlockReading<NW> b = {E, lead, lead > 16u && left > 0, {W, left, 0u, 0u, planes.begin()}};
  planes.clear();
  if (any_lane_active(left > 0)) read_planes<false>(token, b.r, planes, any_lane_active);   // (none in wavefronts of zero blocks)
  if (any_lane_active(b.r.left > 0)) {   // some lane may have read sixteen planes
    if (any_lane_active(b.r.left > 0 && b.r.at != planes.end())) read_planes<true>(token, b.r, planes, any_lane_active);
  }
  put_begun_plane(b.r, planes, any_lane_active);
  return b;
}

// Rows of the 16 x 16 transpose, the first plane the highest: plane 15 - w in the lower and 7 - w in the upper
// half of word w.
template <class Planes>
ZC_DEV void load_planes(const Planes& planes, uint32_t (&h)[8]) {
  uint32_t p[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) p[k] = planes.word(k);
#pragma unroll
  for (int w = 0; w < 8; ++w) h[w] = zc::permute_bytes(p[(7 - w) >> 1], p[(15 - w) >> 1], w & 1 ? 0x05040100u : 0x07060302u);
}

// The rest of the way to the fixed-point values, for any block.
template <int RATE, class AnyActive, class Planes>
ZC_DEV void finish_block(BlockReading<Traits<RATE>::kWords>& b, const uint32_t* token, int32_t (&q)[16],
                         AnyActive any_lane_active, Planes& planes) {
  constexpr int kPayload = Traits<RATE>::kPayloadBits;
  constexpr int kMaxPlanes = kPayload < 32 ? kPayload : 32;
  uint32_t h[8], u[16];
  load_planes(planes, h);
  transpose_halves(h);
#pragma unroll
  for (int w = 0; w < 8; ++w) zc::materialise(h[w]);   // one transpose, not one per half
  const bool deeper = kMaxPlanes > 16 && any_lane_active(b.r.left > 0);
  if (!deeper && !any_lane_active(b.low_start)) {
    // the usual case: at most 16 planes were read and they start within the top 16, so each
    // coefficient is its 16-bit pattern moved up (a lane that read nothing has zero patterns)
    const uint32_t up = (16u - b.lead) & 31u;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      u[w] = (h[w] & 0xFFFFu) << up;
      u[w + 8] = (h[w] >> 16) << up;
    }
  } else {
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      u[w] = h[w] << 16;
      u[w + 8] = h[w] & 0xFFFF0000u;
    }
    if (deeper) {
      b.r.at = planes.begin();
      b.r.pattern = b.r.left > 0 ? b.r.pattern : 0u;   // (a lane that ran out of budget within a plane has put it where it belongs)
      planes.clear();
      read_planes<true>(token, b.r, planes, any_lane_active);
      put_begun_plane(b.r, planes, any_lane_active);
      load_planes(planes, h);
      transpose_halves(h);
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        zc::materialise(h[w]);
        u[w] |= h[w] & 0xFFFFu;
        u[w + 8] |= h[w] >> 16;
      }
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) u[c] >>= b.lead;
  }
  inverse_transform(u, q);
}

// Whole block up to the fixed-point values; returns the exponent byte.
template <int RATE, class AnyActive, class Planes>
ZC_DEV uint32_t decode_block_fixed(uint32_t (&W)[Traits<RATE>::kWords], const uint32_t* token, int32_t (&q)[16],
                                   AnyActive any_lane_active, Planes& planes) {
  auto b = read_block<RATE>(W, token, any_lane_active, planes);
  finish_block<RATE>(b, token, q, any_lane_active, planes);
  return b.E;
}

// ---- the inverse transform as a matrix ----------------------------------------------------
// The inverse lifting halves with floors, but a halving that leaves no remainder is linear, and a
// coefficient that ends six digits above the lowest leaves none in either pass (the passes divide by
// 8 each in all).  Then the 16 values are a fixed 16 x 16 matrix times the coefficients, which the
// matrix cores work out, exactly: the digits that have been read, in bytes, are small whole
// numbers, and so are the sums.  What is needed for that to be the lifting's own result:
//   * digits end six or more above bit 0: lead + digits <= 26 (digits = 8 or 15, see below);
//   * no sum of the lifting wraps.  In the first pass a column's sums are at most 2.25 times its
//     largest coefficient.  With lead >= 2 coefficients are within -715827882..357913941 and
//     fit; with lead = 1 they are up to 1431655765 where the digit of bit 30 is set, and the
//     largest sum, a + c/2 - b/8 - 5d/8, is 2^31 - 1 if one of the four has it (and 1 if none has);
//     the block's first plane must then have a single one.  In the second pass every sum is a sum of
//     the values that come out, with weights of up to 4 in all: no value of 2^29 or more is allowed,
//     which is looked at afterwards, for lead <= 2 (from lead = 3 on coefficients are within
//     -178956970..357913941, and 2.25 * 2.25 times that fits).  Blocks that an encoder made have
//     values of about 2^27 at most;
//   * the scaling by the exponent byte is exact and finite.
constexpr int kInverse8[4][4] = {{8, 3, -4, -1}, {8, 1, 4, 5}, {8, -1, 4, -5}, {8, -3, -4, 1}};   // 8 x what inverse_lift does

// 64 x the weight of coefficient c in value p (row-major).
constexpr int inverse64(int p, int c) {
  return kInverse8[p >> 2][kOrder.v[c] >> 2] * kInverse8[p & 3][kOrder.v[c] & 3];
}

namespace selfcheck {
constexpr bool inverse64_ok() {
  for (int c = 0; c < 16; ++c)
    for (int sign = -1; sign <= 1; sign += 2) {
      int32_t q[16] = {};
      q[kOrder.v[c]] = sign * 64;
      for (int i = 0; i < 4; ++i) zc::inverse_lift(q[i], q[4 + i], q[8 + i], q[12 + i]);
      for (int i = 0; i < 4; ++i) zc::inverse_lift(q[4 * i], q[4 * i + 1], q[4 * i + 2], q[4 * i + 3]);
      for (int p = 0; p < 16; ++p)
        if (q[p] != sign * inverse64(p, c)) return false;
    }
  return true;
}
static_assert(inverse64_ok(), "the inverse transform as a matrix");
}  // namespace selfcheck

// Eight planes t = 0..7, plane 6 - 2w in the lower and 7 - 2w in the upper half of word w, to
// eight digits of each coefficient, plane 0 the highest: byte b of word w = coefficient
// digit_coefficient(w, b).  SIGNED: bytes 0 and 1 xor 0xAA, bytes 2 and 3 xor 0x55 (see kDigitSigns), which rides
// on the last step's operations.
template <bool SIGNED = false>
ZC_DEV constexpr void planes_to_digits(uint32_t (&x)[4]) {
  uint32_t mask[4] = {0x0F0F0F0Fu, 0x33333333u, 0xAAAA0000u, 0x00005555u};   // (in vector registers, see SwapMasks)
  if (!__builtin_is_constant_evaluated())
    for (int i = 0; i < 4; ++i) zc::materialise(mask[i]);
  uint32_t up[4] = {0, 0, x[2], x[3]};
  shift_left_two<4>(up[2], up[3]);
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const uint32_t lo = x[w], hi = x[w + 2];
    x[w] = select_bits(mask[0], lo, up[w + 2]);
    x[w + 2] = select_bits(mask[0], lo >> 4, hi);
  }
  up[1] = x[1];
  up[3] = x[3];
  shift_left_two<2>(up[1], up[3]);
#pragma unroll
  for (int w = 0; w < 4; w += 2) {
    const uint32_t lo = x[w], hi = x[w + 1];
    x[w] = select_bits(mask[1], lo, up[w + 1]);
    x[w + 1] = select_bits(mask[1], lo >> 2, hi);
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) up[w] = x[w];
  shift_left_two<17>(up[0], up[1]);
  shift_left_two<17>(up[2], up[3]);
#pragma unroll
  for (int w = 0; w < 4; ++w)
    x[w] = select_bits(mask[2], up[w], SIGNED ? select_bits_not(mask[3], x[w] >> 17, x[w]) : select_bits(mask[3], x[w] >> 17, x[w]));
}
constexpr int digit_coefficient(int w, int b) { return 8 * (b & 1) + 2 * w + 1 - (b >> 1); }

namespace selfcheck {
constexpr bool digits_ok() {
  uint32_t s = 0x1234567u, pattern[8] = {}, x[4] = {};
  for (int t = 0; t < 8; ++t) { s = s * 1664525u + 1013904223u; pattern[t] = s >> 16; }
  for (int w = 0; w < 4; ++w) x[w] = pattern[6 - 2 * w] | pattern[7 - 2 * w] << 16;
  uint32_t y[4] = {x[0], x[1], x[2], x[3]};
  planes_to_digits(x);
  planes_to_digits<true>(y);
  for (int w = 0; w < 4; ++w)
    for (int b = 0; b < 4; ++b)
      for (int t = 0; t < 8; ++t)
        if (((x[w] >> (8 * b + 7 - t)) & 1u) != ((pattern[t] >> digit_coefficient(w, b)) & 1u)) return false;
  for (int w = 0; w < 4; ++w)
    if (y[w] != (x[w] ^ 0x5555AAAAu)) return false;
  return true;
}
static_assert(digits_ok(), "digits of eight planes");
}  // namespace selfcheck

// A byte of digits d stands for (d ^ 0xAA) - 0xAA (negabinary, the lowest digit positive).
constexpr uint32_t kDigitSigns = 0xAAAAAAAAu;
constexpr int kDigitBias = 0xAA;
// That is y - 0xAA for y = d ^ 0xAA and 0x55 - y for y = d ^ 0x55: what the SIGNED bytes stand for.
constexpr int signed_digit_sign(int b) { return b < 2 ? 1 : -1; }
constexpr int signed_digit_bias(int b) { return b < 2 ? 0xAA : -0x55; }

// What each lane puts into the product.  A byte of digits goes in as the half-precision number of the same
// bits, digits * 2^-24 (the matrix instructions take subnormal halves as they are), and comes out
// as value * 2^(lead - 33) with the weights 64 * weight * 2^9 for the upper eight digits of 16 and 64 *
// weight * 2 for the lower eight.  The upper digits' bytes are SIGNED ones, the lower digits' all xor 0xAA, so that their
// lowest bit, of a sixteenth plane, is zero (with all of them xor 0xAA by operations of their own: 2-way reduce of 8192 x
// 32768 values at rate 8 612 instead of 598 us, with fp32 output 434 instead of 425).  bias: what takes the bytes' offset away, for the upper eight alone
// and for all.
struct MatrixOperands { uint32_t weight[64][4]; float bias[2][4][4]; };   // by lane, by lane / 16
constexpr uint32_t half_of_weight(int w, int lg) {   // w * 2^lg, |w| <= 64
  if (w == 0) return 0;
  const uint32_t m = (uint32_t)(w < 0 ? -w : w);
  int e = 0;
  while ((m >> (e + 1)) != 0) ++e;
  return (w < 0 ? 0x8000u : 0u) | (uint32_t)(15 + e + lg) << 10 | ((m << (10 - e)) & 0x3FFu);
}
constexpr MatrixOperands build_matrix_operands() {
  MatrixOperands t{};
  for (int l = 0; l < 64; ++l) {
    for (int b = 0; b < 4; ++b) {
      const int w = inverse64(l & 15, digit_coefficient(l >> 4, b));
      t.weight[l][b >> 1] |= half_of_weight(signed_digit_sign(b) * w, 9) << (16 * (b & 1));
      t.weight[l][2 + (b >> 1)] |= half_of_weight(w, 1) << (16 * (b & 1));
    }
  }
  for (int p = 0; p < 16; ++p) {
    int upper = 0, lower = 0;
    for (int w = 0; w < 4; ++w)
      for (int b = 0; b < 4; ++b) {
        const int weight = inverse64(p, digit_coefficient(w, b));
        upper += signed_digit_bias(b) * weight;
        lower += kDigitBias * weight;
      }
    t.bias[0][p >> 2][p & 3] = -(float)upper / 32768.0f;
    t.bias[1][p >> 2][p & 3] = -(float)(256 * upper + lower) / 8388608.0f;
  }
  return t;
}
namespace selfcheck {
// No sum of the product's terms and its bias, taken in any order, is longer than a float holds: in units of the lower
// eight digits', with bytes of 255 (the lower ones are even).
constexpr bool matrix_sums_ok() {
  for (int p = 0; p < 16; ++p) {
    int64_t up = 0, down = 0, bias = 0;
    for (int w = 0; w < 4; ++w)
      for (int b = 0; b < 4; ++b) {
        const int64_t weight = inverse64(p, digit_coefficient(w, b));
        const int64_t upper = 256 * 255 * signed_digit_sign(b) * weight, lower = 254 * weight;
        (upper > 0 ? up : down) += upper;
        (lower > 0 ? up : down) += lower;
        bias -= 256 * signed_digit_bias(b) * weight + kDigitBias * weight;
      }
    (bias > 0 ? up : down) += bias;
    if (up >= 1 << 24 || -down >= 1 << 24) return false;
  }
  return true;
}
static_assert(matrix_sums_ok(), "the matrix product's sums are exact");
}  // namespace selfcheck

// Whether the matrix covers a block, as far as that can be told from how it was read: first = the
// pattern of its first plane, digits = 8 or 15 of them.
ZC_DEV bool matrix_covers(uint32_t E, uint32_t lead, uint32_t first, uint32_t digits) {
  const bool place = lead - 1u <= 25u - digits;                      // 1 .. 26 - digits
  const bool crowded = lead < 2u && (first & (first - 1u)) != 0u;
  return place && !crowded && E - 28u <= 221u;
}
// ... and by its values, which come out as value * 2^(lead - 33): 2^29 for lead <= 2.
constexpr float kMatrixMost = 0.125f;

// What these numbers are multiplied with: 2^(33 - lead), the sign of the lowest digit, and the block's
// own scale, 2^(E - 154).
ZC_DEV float matrix_scale(uint32_t E, uint32_t lead) {
  return zc::bits_to_float(((E + 6u - lead) << 23) | lead << 31);
}

template <int RATE, class AnyActive, class Planes>
ZC_DEV void decode_block(uint32_t (&W)[Traits<RATE>::kWords], const uint32_t* token, float (&out)[16],
                         AnyActive any_lane_active, Planes& planes) {
  int32_t q[16];
  const uint32_t E = decode_block_fixed<RATE>(W, token, q, any_lane_active, planes);
  scale_block(q, E, out);
}

template <int RATE, class AnyActive>
ZC_DEV void decode_block(uint32_t (&W)[Traits<RATE>::kWords], const uint32_t* token, float (&out)[16],
                         AnyActive any_lane_active) {
  LocalPlanes planes;
  decode_block<RATE>(W, token, out, any_lane_active, planes);
}

}  // namespace zc2d
#endif  // ZC2D_CODEC_H
