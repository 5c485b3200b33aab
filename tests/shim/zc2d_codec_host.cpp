// Host build of the per-block 4 x 4 codec that the GPU kernels run (csrc/zc2d_codec.h),
// for checking its logic on the CPU against the reference.  Test-only.
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "../../paper_2409_02423_amd/csrc/zc2d_codec.h"

namespace {
// one lane alone: its own predicate is the vote
struct Alone {
  bool operator()(bool p) const { return p; }
};
const Alone always;
constexpr zc2d::ExpandTable kExpand = zc2d::build_expand_table();
constexpr zc2d::TokenTable kToken = zc2d::build_token_table();

template <int RATE>
void enc(const float* x, uint8_t* out) {
  uint32_t b[16], W[zc2d::Traits<RATE>::kWords];
  std::memcpy(b, x, 64);
  zc2d::encode_block<RATE>(b, kExpand.v, W, always);
  std::memcpy(out, W, zc2d::Traits<RATE>::kBlockBytes);
}
template <int RATE>
void dec(const uint8_t* in, float* x) {
  uint32_t W[zc2d::Traits<RATE>::kWords];
  std::memcpy(W, in, zc2d::Traits<RATE>::kBlockBytes);
  float o[16];
  zc2d::decode_block<RATE>(W, kToken.v, o, always);
  std::memcpy(x, o, 64);
}

// A wavefront on the host: `lanes` threads run the per-lane codec in lockstep and take the
// kernels' wavefront-wide votes among themselves (as in zc_codec_host.cpp).
struct Ballot {
  explicit Ballot(int n) : lanes(n) {}
  bool vote(bool p) {
    std::unique_lock<std::mutex> lock(mu);
    any = any || p;
    if (++arrived == lanes) {
      result = any;
      any = false;
      arrived = 0;
      ++round;
      cv.notify_all();
      return result;
    }
    const unsigned long mine = round;
    cv.wait(lock, [&] { return round != mine; });
    return result;
  }
  std::mutex mu;
  std::condition_variable cv;
  int lanes, arrived = 0;
  bool any = false, result = false;
  unsigned long round = 0;
};

template <int RATE>
void wave(bool encode, const uint8_t* in, size_t blocks, uint8_t* out, int lanes) {
  constexpr int B = zc2d::Traits<RATE>::kBlockBytes;
  Ballot ballot(lanes);
  struct Vote {
    Ballot* b;
    bool operator()(bool p) const { return b->vote(p); }
  };
  const Vote vote{&ballot};
  const size_t waves = (blocks + lanes - 1) / lanes;
  std::vector<std::thread> pool;
  for (int t = 0; t < lanes; ++t)
    pool.emplace_back([&, t] {
      for (size_t w = 0; w < waves; ++w) {
        const size_t j = w * lanes + t;
        const bool real = j < blocks;   // lanes past the end code a zero block and drop the result
        if (encode) {
          uint32_t b[16] = {}, W[zc2d::Traits<RATE>::kWords];
          if (real) std::memcpy(b, in + 64 * j, 64);
          zc2d::encode_block<RATE>(b, kExpand.v, W, vote);
          if (real) std::memcpy(out + j * B, W, B);
        } else {
          uint32_t W[zc2d::Traits<RATE>::kWords] = {};
          if (real) std::memcpy(W, in + j * B, B);
          float o[16];
          zc2d::decode_block<RATE>(W, kToken.v, o, vote);
          if (real) std::memcpy(out + 64 * j, o, 64);
        }
      }
    });
  for (auto& th : pool) th.join();
}
}  // namespace

extern "C" int zc2d_host_wave(int rate, int encode, const void* in, size_t blocks, void* out, int lanes) {
  const uint8_t* src = static_cast<const uint8_t*>(in);
  uint8_t* dst = static_cast<uint8_t*>(out);
  switch (rate) {
    case 2: wave<2>(encode != 0, src, blocks, dst, lanes); break;
    case 4: wave<4>(encode != 0, src, blocks, dst, lanes); break;
    case 8: wave<8>(encode != 0, src, blocks, dst, lanes); break;
    case 16: wave<16>(encode != 0, src, blocks, dst, lanes); break;
    default: return -2;
  }
  return 0;
}

// The matrix form of the decoder on one block, its products summed in whole numbers: false if the block
// is not covered.
namespace {
template <int RATE>
bool dec_matrix(const uint8_t* in, float* x) {
  uint32_t W[zc2d::Traits<RATE>::kWords];
  std::memcpy(W, in, zc2d::Traits<RATE>::kBlockBytes);
  zc2d::LocalPlanes planes;
  auto b = zc2d::read_block<RATE>(W, kToken.v, always, planes);
  uint32_t upper[4], lower[4];
  for (int w = 0; w < 4; ++w) {
    upper[w] = planes.word(3 - w);
    lower[w] = planes.word(7 - w);
  }
  const bool more = (lower[0] | lower[1] | lower[2] | lower[3]) != 0;
  if (b.r.left > 0 || (lower[0] >> 16) != 0) return false;
  if (!zc2d::matrix_covers(b.E, b.lead, upper[3] & 0xFFFFu, more ? 15u : 8u)) return false;
  zc2d::planes_to_digits(upper);
  zc2d::planes_to_digits(lower);
  int64_t n[16];
  for (int w = 0; w < 4; ++w)
    for (int c = 0; c < 4; ++c) {
      auto digits = [&](uint32_t word) { return (int64_t)(((word ^ zc2d::kDigitSigns) >> (8 * c)) & 0xFFu) - zc2d::kDigitBias; };
      n[zc2d::digit_coefficient(w, c)] = 256 * digits(upper[w]) + digits(lower[w]);
    }
  const float scale = zc2d::matrix_scale(b.E, b.lead);
  for (int p = 0; p < 16; ++p) {
    int64_t sum = 0;
    for (int c = 0; c < 16; ++c) sum += zc2d::inverse64(p, c) * n[c];
    const float v = (float)sum / 8388608.0f;
    if (sum != (int64_t)(v * 8388608.0f)) return false;   // (a sum that a float does not hold)
    if (b.lead <= 2u && (v < 0 ? -v : v) >= zc2d::kMatrixMost) return false;
    x[p] = __builtin_fmaf(v, scale, 0.0f);
  }
  return true;
}
}  // namespace

extern "C" int zc2d_host_decode_by_matrix(int rate, const uint8_t* in, size_t blocks, float* x, uint8_t* covered) {
  for (size_t j = 0; j < blocks; ++j) switch (rate) {
      case 2: covered[j] = dec_matrix<2>(in + j * 4, x + 16 * j); break;
      case 4: covered[j] = dec_matrix<4>(in + j * 8, x + 16 * j); break;
      case 8: covered[j] = dec_matrix<8>(in + j * 16, x + 16 * j); break;
      default: return -2;
    }
  return 0;
}

extern "C" int zc2d_host_encode_blocks(int rate, const float* x, size_t blocks, uint8_t* out) {
  for (size_t j = 0; j < blocks; ++j) switch (rate) {
      case 2: enc<2>(x + 16 * j, out + j * 4); break;
      case 4: enc<4>(x + 16 * j, out + j * 8); break;
      case 8: enc<8>(x + 16 * j, out + j * 16); break;
      case 16: enc<16>(x + 16 * j, out + j * 32); break;
      default: return -2;
    }
  return 0;
}

extern "C" int zc2d_host_decode_blocks(int rate, const uint8_t* in, size_t blocks, float* x) {
  for (size_t j = 0; j < blocks; ++j) switch (rate) {
      case 2: dec<2>(in + j * 4, x + 16 * j); break;
      case 4: dec<4>(in + j * 8, x + 16 * j); break;
      case 8: dec<8>(in + j * 16, x + 16 * j); break;
      case 16: dec<16>(in + j * 32, x + 16 * j); break;
      default: return -2;
    }
  return 0;
}
