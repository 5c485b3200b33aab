// Host build of the per-block 4 x 4 codec that the GPU kernels run (csrc/zc2d_codec.h),
// for checking its logic on the CPU against the reference.  Test-only.
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "../../paper_2409_02423_amd/csrc/zc2d_codec.h"
#include "../../paper_2409_02423_amd/csrc/zc2d_grid.h"

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

// The matrix form of the decoder on one block: the bytes, weights and biases that the kernels put into their matrix
// instructions, multiplied and summed in fp32 from either end, which has to give the same (every sum is exact).  False
// if the block is not covered.
namespace {
constexpr zc2d::MatrixOperands kMatrix = zc2d::build_matrix_operands();

float half_to_float(uint32_t h) {   // (exact; no infinities here)
  const int e = (int)((h >> 10) & 31u);
  const float m = e ? __builtin_ldexpf((float)(1024u + (h & 1023u)), e - 25) : __builtin_ldexpf((float)(h & 1023u), -24);
  return (h & 0x8000u) ? -m : m;
}

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
  zc2d::planes_to_digits<true>(upper);
  zc2d::planes_to_digits(lower);
  for (int w = 0; w < 4; ++w) lower[w] ^= zc2d::kDigitSigns;
  const float scale = zc2d::matrix_scale(b.E, b.lead);
  for (int p = 0; p < 16; ++p) {
    float term[32];
    int n = 0;
    for (int w = 0; w < 4; ++w)
      for (int c = 0; c < 4; ++c) {
        const uint32_t* weight = kMatrix.weight[16 * w + p];   // what lane 16 w + p has
        term[n++] = half_to_float((upper[w] >> (8 * c)) & 0xFFu) * half_to_float((weight[c >> 1] >> (16 * (c & 1))) & 0xFFFFu);
        if (more) term[n++] = half_to_float((lower[w] >> (8 * c)) & 0xFFu) * half_to_float((weight[2 + (c >> 1)] >> (16 * (c & 1))) & 0xFFFFu);
      }
    float v = kMatrix.bias[more][p >> 2][p & 3], back = 0.0f;
    for (int i = 0; i < n; ++i) v += term[i];
    for (int i = n; i-- > 0;) back += term[i];
    back += kMatrix.bias[more][p >> 2][p & 3];
    if (v != back) {
      for (int i = 0; i < 16; ++i) x[i] = -1e30f;   // (no block's values: the caller sees a difference)
      return true;
    }
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

// Workgroups per CU of decompress2d, negative if the grid may be made smaller for want of blocks per lane.
extern "C" int zc2d_host_decompress_grid(size_t rows, size_t cols, int half, int rate) {
  const zc2d::DecompressGrid g = zc2d::decompress_grid(((rows + 3) / 4) * ((cols + 3) / 4), cols, half != 0, rate);
  return g.at_once ? g.per_cu : -g.per_cu;
}
