// zc2d_kernels.hip -- gfx950 kernels and C ABI for the 4 x 4 block codec (see include/zc.h).
//
// One lane per block of 4 x 4 values, blocks taken in row-major block order with a grid
// stride, so that the 64 lanes of a wavefront read four contiguous 1 KiB spans (one per
// matrix row of the block row) and write one contiguous span of 64 * 2*RATE stream bytes.
// A block lives in registers from load to store; LDS holds the coder's look-up tables (2 KiB
// for the encoder, 22 KiB for the decoder) and, while a block is decoded, its planes (36 bytes per
// lane).  The decoder's inverse transform is a matrix product where its halvings leave no remainder,
// and then runs on the matrix cores (see "the decoder's values as a matrix product").
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "../../include/zc.h"
#include "zc2d_codec.h"
#include "zc2d_grid.h"
#include "zc_half.h"

namespace {

constexpr int kThreads = 256;
// Of the kernels that decode (see below): more wavefronts share one copy of the 22 KiB token table,
// but a small matrix occupies fewer CUs.
constexpr int kDecodeThreads = 512, kDecodeThreadsSmall = 256;

__device__ __align__(16) const zc2d::ExpandTable g_expand = zc2d::build_expand_table();
__device__ __align__(16) const zc2d::TokenTable g_token = zc2d::build_token_table();

// Copy a table of WORDS 32-bit words to LDS, 16 bytes per lane and step: a lane issues all of
// its loads back to back and then writes (one wait for the whole table, not one per step).
// In a last, partial step of several the lanes beyond the table's end copy its first entry
// once more.
template <int WORDS, int THREADS>
__device__ __forceinline__ void stage_table(const uint32_t* __restrict__ src, uint32_t* dst) {
  static_assert(WORDS % 4 == 0, "table size");
  constexpr int kVecs = WORDS / 4;
  constexpr int kSteps = (kVecs + THREADS - 1) / THREADS;
  if constexpr (kSteps == 1) {
    if (threadIdx.x < kVecs) reinterpret_cast<uint4*>(dst)[threadIdx.x] = reinterpret_cast<const uint4*>(src)[threadIdx.x];
  } else {
    uint4 v[kSteps];
    int idx[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
      idx[i] = threadIdx.x + i * THREADS;
      if ((i + 1) * THREADS > kVecs && idx[i] >= kVecs) idx[i] = 0;
      v[i] = reinterpret_cast<const uint4*>(src)[idx[i]];
    }
#pragma unroll
    for (int i = 0; i < kSteps; ++i) reinterpret_cast<uint4*>(dst)[idx[i]] = v[i];
    __builtin_amdgcn_sched_group_barrier(0x020, kSteps, 0);   // (for the instruction scheduler: the loads first,
    __builtin_amdgcn_sched_group_barrier(0x200, kSteps, 0);   // then the LDS writes)
  }
  __syncthreads();
}
// Workgroups per CU in the grid.  The kernels that decode have 512 lanes per workgroup (256 for small
// matrices, see decode_threads): 22 KiB of token table, 18 KiB of planes, 9 KiB for the matrix product and 2
// KiB for an encoder are 49 to 51 KiB, of which three fit a CU: six wavefronts per SIMD, for which 80 registers
// are left.  The forms with the matrix product are held to that (without being told the reduces took 88,
// four wavefronts: 0.530 against 0.496 ms for the 2-way reduce of 8192 x 32768 values at rate 4).  (256 lanes, as
// the kernels were before: 0.270 against 0.248 ms for decompress2d, 0.613 against 0.583 ms for the reduce;
// 1024: 0.599 ms.)
// Their grids and the figures behind them are in zc2d_grid.h.
// The compress kernel has 16, and 64 where that leaves a lane four blocks or more: with one block per lane a
// workgroup stages its table and asks for its values for nothing else (8192 x 32768 values at rate 4: 238 at 16, 224 at
// 64, 229 at 128; 8192 x 8192 at rate 2: 48.9 at 16, four blocks per lane, 55.8 at 64, one block; 6144 x 43690 at rate 8
// 296 and 265).
// Only a build with -DZC_TUNING_KNOBS lets ZC2D_WORKGROUPS_PER_CU override these; the shipped library reads
// no environment variable.
constexpr int kCompressWorkgroupsPerCU = 16, kCompressWorkgroupsPerCUMost = 64;
using zc2d::kDecodeWorkgroupsPerCU;
using zc2d::kDecodeWorkgroupsPerCULeast;
using zc2d::kDecodeWorkgroupsPerCUWide;

// The wavefront-wide vote of the codec: whether p holds in some lane.
struct AnyLane {
  __device__ bool operator()(bool p) const { return __builtin_amdgcn_ballot_w64(p) != 0; }
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A lane's sixteen decoded planes in LDS: 32 bytes on end, and a spare word between lanes so that lanes at
// the same plane are on different banks.  Places are byte offsets within the workgroup's planes.
constexpr int kPlaneBytes = 36;
struct WavePlanes {
  char* lds;
  uint32_t mine;
  __device__ __forceinline__ WavePlanes(char* planes, uint32_t tid) : lds(planes), mine(tid * kPlaneBytes) {}
  __device__ __forceinline__ uint32_t begin() const { return mine; }
  __device__ __forceinline__ uint32_t end() const { return mine + 16 * zc2d::kPlaneStep; }
  __device__ __forceinline__ void clear() {
    uint32_t* p = reinterpret_cast<uint32_t*>(lds + mine);
#pragma unroll
    for (int k = 0; k < 8; ++k) p[k] = 0u;
  }
  __device__ __forceinline__ void put(uint32_t at, uint32_t pattern) {
    asm volatile("" ::: "memory");   // (halves and words of the same memory)
    *reinterpret_cast<uint16_t*>(lds + at) = (uint16_t)pattern;
    asm volatile("" ::: "memory");
  }
  __device__ __forceinline__ uint32_t word(int k) const {
    asm volatile("" ::: "memory");   // (read where they are wanted, and not kept)
    return *reinterpret_cast<const uint32_t*>(lds + mine + 4 * k);
  }
  // the spare word, and the planes of the lane's wavefront
  __device__ __forceinline__ float& spare(uint32_t tid) const { return *reinterpret_cast<float*>(lds + tid * kPlaneBytes + 32); }
  __device__ __forceinline__ char* wave(uint32_t tid) const { return lds + (tid & ~63u) * kPlaneBytes; }
};

// Shape of the matrix and of the walk over its blocks; the same for every lane.
struct Walk {
  size_t rows, cols;
  size_t bc, blocks;        // blocks per block row, blocks in all
  size_t whole_br, whole_bc;   // block rows and block columns that lie inside the matrix
  size_t stride;            // lanes in the grid: a lane's next block is `stride` blocks on
  size_t step_bi, step_bj;  // stride / bc, stride % bc
  uint32_t narrow;          // 2^16 / bc, rounded up, if bc is less than 64, otherwise 0 (see WaveCursor::lane)
  uint32_t pieces;          // how values that come as rows are stored (see store_rows)
};
constexpr uint32_t kPieces = 1, kNarrowPieces = 2;

// A lane's place in the walk.  Advancing costs additions only: no division per block.
struct Cursor {
  size_t b, bi, bj;   // block index, block row, block column
  size_t first;       // index of the block's first value, (4 * bi) * cols + 4 * bj

  __device__ __forceinline__ void start(const Walk& w, size_t b0) {
    b = b0;
    bi = b0 / w.bc;
    bj = b0 - bi * w.bc;
    first = 4 * bi * w.cols + 4 * bj;
  }
  __device__ __forceinline__ void advance(const Walk& w) {
    b += w.stride;
    bi += w.step_bi;
    bj += w.step_bj;
    first += 4 * (w.step_bi * w.cols + w.step_bj);
    if (bj >= w.bc) {
      bj -= w.bc;
      bi += 1;
      first += 4 * w.cols - 4 * w.bc;
    }
  }
  // all 16 values inside the matrix
  __device__ __forceinline__ bool whole(const Walk& w) const { return bi < w.whole_br && bj < w.whole_bc; }
};

// A row of a block as one access.  Where the column count is not a multiple of 4 the rows are
// aligned to their elements only, which a global memory access of any width may be on this
// GPU; 16 single accesses per block took 0.334 ms to compress and 0.506 ms to decompress
// 6144 x 43690 fp32 values at rate 8, a row at a time takes 0.283 and 0.308 ms, as for 43688
// columns.  (With plain stores instead of non-temporal ones: 0.314 ms, and 0.278 against 0.262 ms
// at rate 4.)
typedef uint32_t Row32 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t Row16 __attribute__((ext_vector_type(2), aligned(2)));

// The block under the cursor as fp32 bit patterns; parts that stick out of the matrix
// repeat the last valid row / column.  DT: the matrix holds fp32, or bf16 / fp16 values
// that are widened (exactly) on the way in.
template <int DT>
__device__ __forceinline__ void load_block(const void* in, const Walk& w, const Cursor& c, uint32_t (&x)[16]) {
  if (c.whole(w)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (DT == kF32) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const Row32*>(static_cast<const float*>(in) + c.first + r * w.cols));
        x[4 * r] = v.x; x[4 * r + 1] = v.y; x[4 * r + 2] = v.z; x[4 * r + 3] = v.w;
      } else {
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const Row16*>(static_cast<const uint16_t*>(in) + c.first + r * w.cols));
        x[4 * r] = widen_half<DT>(v.x & 0xFFFFu); x[4 * r + 1] = widen_half<DT>(v.x >> 16);
        x[4 * r + 2] = widen_half<DT>(v.y & 0xFFFFu); x[4 * r + 3] = widen_half<DT>(v.y >> 16);
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        size_t rr = 4 * c.bi + r, cc = 4 * c.bj + q;
        rr = rr < w.rows ? rr : w.rows - 1;
        cc = cc < w.cols ? cc : w.cols - 1;
        if constexpr (DT == kF32) x[4 * r + q] = static_cast<const uint32_t*>(in)[rr * w.cols + cc];
        else x[4 * r + q] = widen_half<DT>(static_cast<const uint16_t*>(in)[rr * w.cols + cc]);
      }
  }
}

// The reverse; half-precision values are rounded to nearest, ties to even.
template <int DT>
__device__ __forceinline__ void store_block(void* out, const Walk& w, const Cursor& c, const float (&y)[16]) {
  if (c.whole(w)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (DT == kF32) {
        const Row32 v = {__float_as_uint(y[4 * r]), __float_as_uint(y[4 * r + 1]), __float_as_uint(y[4 * r + 2]),
                         __float_as_uint(y[4 * r + 3])};
        __builtin_nontemporal_store(v, reinterpret_cast<Row32*>(static_cast<float*>(out) + c.first + r * w.cols));
      } else {
        const Row16 v = {narrow_half<DT>(y[4 * r]) | narrow_half<DT>(y[4 * r + 1]) << 16,
                         narrow_half<DT>(y[4 * r + 2]) | narrow_half<DT>(y[4 * r + 3]) << 16};
        __builtin_nontemporal_store(v, reinterpret_cast<Row16*>(static_cast<uint16_t*>(out) + c.first + r * w.cols));
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const size_t rr = 4 * c.bi + r, cc = 4 * c.bj + q;
        if (rr < w.rows && cc < w.cols) {
          if constexpr (DT == kF32) static_cast<float*>(out)[rr * w.cols + cc] = y[4 * r + q];
          else static_cast<uint16_t*>(out)[rr * w.cols + cc] = (uint16_t)narrow_half<DT>(y[4 * r + q]);
        }
      }
  }
}

template <int NW>
__device__ __forceinline__ void load_words(const uint8_t* p, uint32_t (&W)[NW]) {
  if constexpr (NW == 1) {
    W[0] = *reinterpret_cast<const uint32_t*>(p);
  } else if constexpr (NW == 2) {
    const u32x2 v = *reinterpret_cast<const u32x2*>(p);
    W[0] = v.x; W[1] = v.y;
  } else {
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
      const u32x4 v = reinterpret_cast<const u32x4*>(p)[i];
      W[4 * i] = v.x; W[4 * i + 1] = v.y; W[4 * i + 2] = v.z; W[4 * i + 3] = v.w;
    }
  }
}

template <int NW>
__device__ __forceinline__ void store_words(uint8_t* p, const uint32_t (&W)[NW]) {
  if constexpr (NW == 1) {
    *reinterpret_cast<uint32_t*>(p) = W[0];
  } else if constexpr (NW == 2) {
    const u32x2 v = {W[0], W[1]};
    *reinterpret_cast<u32x2*>(p) = v;
  } else {
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
      const u32x4 v = {W[4 * i], W[4 * i + 1], W[4 * i + 2], W[4 * i + 3]};
      reinterpret_cast<u32x4*>(p)[i] = v;
    }
  }
}

template <int RATE, int DT>
__global__ __launch_bounds__(kThreads) void compress2d_kernel(const void* __restrict__ in, Walk w,
                                                              uint8_t* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint32_t expand[zc2d::kExpandEntries];
  stage_table<zc2d::kExpandEntries, kThreads>(g_expand.v, expand);
  constexpr int NW = zc2d::Traits<RATE>::kWords;
  const size_t b0 = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (b0 >= w.blocks) return;
  Cursor cur;
  cur.start(w, b0);
  uint32_t x[16];
  load_block<DT>(in, w, cur, x);
  // The first block has to have arrived before the loop starts: with loads still in flight
  // at its entry, every pass would wait for its own prefetch as well (loads return in order).
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  for (;;) {
    // The loads of the lane's next block, if it has one, are issued before its current
    // block is coded.
    Cursor next = cur;
    next.advance(w);
    const bool more = next.b < w.blocks;
    uint32_t xn[16], W[NW];
    if (more) load_block<DT>(in, w, next, xn);
    zc2d::encode_block<RATE>(x, expand, W, AnyLane());
    store_words<NW>(out + cur.b * zc2d::Traits<RATE>::kBlockBytes, W);
    if (!more) break;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = xn[i];
    cur = next;
  }
}

// ---- the decoder's values as a matrix product ------------------------------------------
// (See "the inverse transform as a matrix" in zc2d_codec.h.)  The wavefront's 64 blocks are four
// groups of 16, and a group is one matrix instruction: 16 x 16 weights times 16 coefficients of 16
// blocks.  Rows of lanes (lane / 16) and registers change places on the way in, so that lane 16*j + i
// has the digits of four coefficients (word j of planes_to_digits) of block i of each group; of the
// result it has row j of these blocks, four values that lie together in the matrix.  From there they
// are stored as they are, or change places back to a block per lane.  All of these changes go through LDS: it is
// idle three quarters of the time, and an instruction that swaps rows of two registers takes a SIMD 8 of the cycles
// that these kernels are bound by (with such instructions, 59 or 91 cycles per chunk and 130 for the way back, and now, us of a
// 2-way reduce of 8192 x 32768 values at rate 4 403 and 396, at rate 8 541 and 524).
// (What bounds these kernels is their VALU cycles.  The lifting's way, transpose of 16 planes, xor,
// shifts, lifting, conversions and scaling, takes about 250 instructions per block, this one about 100, 150
// with more than eight planes.  With the loop and the planes' layout as they are now, us before and after:
// 8192 x 32768 values, streams from memory, decompress2d at rate 4 244 and 220, at rate 8 275 and 242, 2-way
// reduce 577 and 469, 737 and 643; 8192 x 6144 values to bf16 at rate 8 59.3 and 49.5.  For the few wavefronts of
// a small matrix the product's latencies only add up: 1000 x 1003 values at rate 4 5.2 us to decompress
// with it, 4.9 without, so the kernels of 256 lanes do without.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __align__(16) const zc2d::MatrixOperands g_matrix = zc2d::build_matrix_operands();
constexpr int kMatrixWords = sizeof(zc2d::MatrixOperands) / 4;

// Values of a block per lane, row-major, from and to rows: rows[g] = row lane/16 of block lane%16 of
// group g.  `area` is the wavefront's own planes, which nobody needs any more; half of the values at a time take 2048 of
// its 2304 bytes.  Two values of row j of block b are at 512 * j + 8 * b, but with neighbouring groups exchanged in odd rows:
// then neither side's accesses meet in a bank.
typedef float f32x2 __attribute__((ext_vector_type(2)));
struct RowExchange {
  char *row, *row1, *block, *block1;   // of groups 0 and 1, of rows 0 and 1
  __device__ __forceinline__ RowExchange(char* area, uint32_t tid) {
    const uint32_t at = (tid & 15) * 8 + (tid & 48) * 32 + (tid & 16) * 8, mine = (tid & 63) * 8;
    row = area + at;
    row1 = area + (at ^ 128u);
    block = area + mine;
    block1 = area + (mine ^ 128u);
  }
  __device__ __forceinline__ f32x2& by_row(int g) const { return *reinterpret_cast<f32x2*>((g & 1 ? row1 : row) + 256 * (g >> 1)); }
  __device__ __forceinline__ f32x2& by_block(int r) const { return *reinterpret_cast<f32x2*>((r & 1 ? block1 : block) + 512 * r); }
};
// (what LDS holds changes places between a wavefront's lanes, in the order of the program)
__device__ __forceinline__ void lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void blocks_to_rows(const float (&y)[16], f32x4 (&rows)[4], char* area, uint32_t tid) {
  const RowExchange at(area, tid);
#pragma unroll
  for (int h = 0; h < 4; h += 2) {
    lds_order();
#pragma unroll
    for (int r = 0; r < 4; ++r) at.by_block(r) = f32x2{y[4 * r + h], y[4 * r + h + 1]};
    lds_order();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x2 v = at.by_row(g);
      rows[g][h] = v.x;
      rows[g][h + 1] = v.y;
    }
  }
  lds_order();
}
__device__ __forceinline__ void rows_to_blocks(const f32x4 (&rows)[4], float (&y)[16], char* area, uint32_t tid) {
  const RowExchange at(area, tid);
#pragma unroll
  for (int h = 0; h < 4; h += 2) {
    lds_order();
#pragma unroll
    for (int g = 0; g < 4; ++g) at.by_row(g) = f32x2{rows[g][h], rows[g][h + 1]};
    lds_order();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x2 v = at.by_block(r);
      y[4 * r + h] = v.x;
      y[4 * r + h + 1] = v.y;
    }
  }
  lds_order();
}

// Four words of a block per lane to the word lane/16 of block lane%16 of each group.  `area` has the words of the
// workgroup's blocks, word by word.
__device__ __forceinline__ void words_to_rows(uint32_t (&x)[4], char* area, uint32_t tid) {
  uint32_t* const mine = reinterpret_cast<uint32_t*>(area) + tid;
  const uint32_t* const theirs = reinterpret_cast<const uint32_t*>(area) + (tid & 48) * (kDecodeThreads / 16) + (tid & ~48u);
  lds_order();
#pragma unroll
  for (int w = 0; w < 4; ++w) mine[w * kDecodeThreads] = x[w];
  lds_order();
#pragma unroll
  for (int g = 0; g < 4; ++g) x[g] = theirs[16 * g];
  lds_order();
}

// The lane's number in the workgroup, anew in each pass of a loop: what is worked out from it, some dozen
// offsets, would otherwise be kept across the passes for want of registers.
__device__ __forceinline__ uint32_t fresh_tid() {
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  return tid;
}

// The wavefront's blocks as rows, unscaled, and each group's scale; false if some block is not covered.
// All 64 lanes take part.
__device__ __forceinline__ bool matrix_product(const WavePlanes& planes, uint32_t E, uint32_t lead, const uint32_t* matrix, char* digits, uint32_t tid,
                                               f32x4 (&d)[4], float (&scale)[4]) {
  uint32_t x[4], lower[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    x[w] = planes.word(3 - w);
    lower[w] = planes.word(7 - w);
  }
  const bool more = AnyLane()((lower[0] | lower[1] | lower[2] | lower[3]) != 0u);   // more than eight planes
  // (the sixteenth would make the sums too long for a float)
  if (AnyLane()(!zc2d::matrix_covers(E, lead, x[3] & 0xFFFFu, more ? 15u : 8u) || (lower[0] >> 16) != 0u)) return false;
  zc2d::planes_to_digits<true>(x);
  planes.spare(tid) = zc2d::matrix_scale(E, lead);
  words_to_rows(x, digits, tid);
#pragma unroll
  for (int g = 0; g < 4; ++g) scale[g] = planes.spare((tid & ~48u) + 16 * g);
  if (!more) {
    const f32x4 bias = *reinterpret_cast<const f32x4*>(matrix + 256 + ((tid & 48) >> 2));
    const f16x4 weight = __builtin_bit_cast(f16x4, *reinterpret_cast<const u32x2*>(matrix + 4 * (tid & 63)));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const u32x2 v = {zc::permute_bytes(0u, x[g], 0x0c010c00u), zc::permute_bytes(0u, x[g], 0x0c030c02u)};
      d[g] = __builtin_amdgcn_mfma_f32_16x16x16f16(weight, __builtin_bit_cast(f16x4, v), bias, 0, 0, 0);
    }
  } else {
    zc2d::planes_to_digits(lower);
#pragma unroll
    for (int w = 0; w < 4; ++w) lower[w] ^= zc2d::kDigitSigns;
    words_to_rows(lower, digits, tid);
    const f32x4 bias = *reinterpret_cast<const f32x4*>(matrix + 272 + ((tid & 48) >> 2));
    const f16x8 weight = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(matrix + 4 * (tid & 63)));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const u32x4 v = {zc::permute_bytes(0u, x[g], 0x0c010c00u), zc::permute_bytes(0u, x[g], 0x0c030c02u),
                       zc::permute_bytes(0u, lower[g], 0x0c010c00u), zc::permute_bytes(0u, lower[g], 0x0c030c02u)};
      d[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(weight, __builtin_bit_cast(f16x8, v), bias, 0, 0, 0);
    }
  }
  // values that the lifting's sums may not have room for, in blocks where they could be
  const uint64_t early = __builtin_amdgcn_ballot_w64(lead <= 2u);
  uint64_t bad = 0;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // (not as inline assembly: how long an instruction has to wait for a matrix instruction's result, the compiler
    // sees to for those that it knows.  These are two v_maximum3_f32.)
    const float v = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(d[g][0]), __builtin_fabsf(d[g][1])),
                                                  __builtin_elementwise_maximum(__builtin_fabsf(d[g][2]), __builtin_fabsf(d[g][3])));
    const uint64_t group = (early >> (16 * g)) & 0xFFFFu;
    bad |= __builtin_amdgcn_ballot_w64(v >= zc2d::kMatrixMost) & (group | group << 16 | group << 32 | group << 48);
  }
  return bad == 0;
}

// ---- the kernels that decode ----------------------------------------------------------
// A wavefront takes 64 consecutive blocks at a time, and all of its lanes stay together: lanes past the
// last block decode an empty one and store nothing.
// Whether a difference of two sizes is negative, from its upper half and on the scalar side (there are no
// scalar comparisons of 64 bits, and the vector ones would draw the cursor into vector registers).
__device__ __forceinline__ bool negative(size_t difference) {
  return __builtin_amdgcn_readfirstlane((int)(difference >> 32)) < 0;
}

struct WaveCursor {
  size_t b, bi, bj;   // the first of the 64 blocks, its block row and block column
  size_t first;       // index of its first value
  __device__ __forceinline__ void start(const Walk& w, size_t b0) {
    const size_t row = b0 / w.bc;   // (worked out in vector registers)
    b = b0;
    bi = (size_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(row >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)row);
    bj = b0 - bi * w.bc;
    first = 4 * bi * w.cols + 4 * bj;
  }
  __device__ __forceinline__ void advance(const Walk& w) {
    b += w.stride;
    bi += w.step_bi;
    bj += w.step_bj;
    first += 4 * (w.step_bi * w.cols + w.step_bj);
    const size_t past = bj - w.bc;
    if (!negative(past)) {
      bj = past;
      bi += 1;
      first += 4 * w.cols - 4 * w.bc;
    }
  }
  // how many of the 64 there are
  __device__ __forceinline__ uint32_t count(const Walk& w) const { return negative(w.blocks - b - 64) ? (uint32_t)(w.blocks - b) : 64u; }
  __device__ __forceinline__ bool inside(const Walk& w) const { return negative(b - w.blocks); }
  // all 64 in one block row and whole
  __device__ __forceinline__ bool whole(const Walk& w) const { return negative(bi - w.whole_br) && !negative(w.whole_bc - bj - 64); }
  // the lane's own block
  __device__ __forceinline__ Cursor lane(const Walk& w, uint32_t tid) const {
    Cursor c;
    const uint32_t l = tid & 63;
    c.b = b + l;
    if (w.narrow) {
      // many block rows: on = (bj + l) / bc, of numbers below 128 and 64, is the product's upper half, since (bj + l) *
      // (bc * narrow - 2^16) < 128 * 64 stays below 2^16.  (Subtracted in a loop: 2097152 x 4 values to bf16 at rate 4 15.4
      // instead of 12.9 us, 2-way reduce to a stream 23.5 and 19.3.)
      const uint32_t at = (uint32_t)bj + l, bc = (uint32_t)w.bc, on = at * w.narrow >> 16;
      c.bi = bi + on;
      c.bj = at - on * bc;
      c.first = first + (4 * l + on * (4 * (uint32_t)w.cols - 4 * bc));
    } else {
      // at most the end of one
      const uint32_t here = negative(w.bc - bj - 64) ? (uint32_t)(w.bc - bj) : 64u;
      const bool on = l >= here;
      c.bi = bi + (on ? 1 : 0);
      c.bj = (on ? bj - w.bc : bj) + l;
      c.first = (on ? first + 4 * w.cols - 4 * w.bc : first) + 4 * l;
    }
    return c;
  }
  // where the lane's four values of group 0 are if the wavefront's blocks are whole; group g is 64*g values on
  __device__ __forceinline__ size_t row(const Walk& w, uint32_t tid) const {
    const size_t l = tid & 63;
    return first + (l >> 4) * w.cols + 4 * (l & 15);
  }
};

// The wavefront's first block (the same in all its lanes).
template <int THREADS>
__device__ __forceinline__ size_t first_block() {
  return (size_t)blockIdx.x * THREADS + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u));
}

// The words of the lane's block, or of an empty one past the end.  (The wavefront's place is added up on the
// scalar side, the lane's is an offset.)
template <int RATE>
__device__ __forceinline__ void load_block_words(const uint8_t* in, const WaveCursor& cur, const Walk& w, uint32_t tid,
                                                 uint32_t (&W)[zc2d::Traits<RATE>::kWords]) {
#pragma unroll
  for (int i = 0; i < zc2d::Traits<RATE>::kWords; ++i) W[i] = 0u;
  const uint8_t* p = in + cur.b * zc2d::Traits<RATE>::kBlockBytes;
  const uint32_t lane = tid & 63u;
  if (lane < cur.count(w)) load_words<zc2d::Traits<RATE>::kWords>(p + lane * zc2d::Traits<RATE>::kBlockBytes, W);
}

template <int DT, bool PLAIN = false>
__device__ __forceinline__ void store_row(void* out, size_t at, const f32x4& y) {
  if constexpr (DT == kF32) {
    const Row32 v = {__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])};
    Row32* p = reinterpret_cast<Row32*>(static_cast<float*>(out) + at);
    if constexpr (PLAIN) *p = v;
    else __builtin_nontemporal_store(v, p);
  } else {
    const Row16 v = {narrow_half<DT>(y[0]) | narrow_half<DT>(y[1]) << 16, narrow_half<DT>(y[2]) | narrow_half<DT>(y[3]) << 16};
    Row16* p = reinterpret_cast<Row16*>(static_cast<uint16_t*>(out) + at);
    if constexpr (PLAIN) *p = v;
    else __builtin_nontemporal_store(v, p);
  }
}

// Stores the wavefront's blocks, given as rows: as they are, four pieces of 256 bytes (kPieces), or from a block per lane, 1
// KiB of a row at a time, or, where a block row is a few blocks long (kNarrowPieces), as they are with a place worked out for
// each.  Which, the host says (see store_form).
template <int DT>
__device__ __forceinline__ void store_rows(void* out, const Walk& w, const WaveCursor& cur, const WavePlanes& planes, uint32_t tid, const f32x4 (&rows)[4]) {
  if (cur.whole(w) && (w.pieces & kPieces)) {
    const size_t at = cur.row(w, tid);
#pragma unroll
    for (int g = 0; g < 4; ++g) store_row<DT>(out, at + 64 * g, rows[g]);
  } else if (w.pieces & kNarrowPieces) {
    // (as in WaveCursor::lane; the offsets are below 2^16, and blocks past the last one are past the last row)
    const uint32_t bc = (uint32_t)w.bc, cols = (uint32_t)w.cols, bj = (uint32_t)cur.bj, r = (tid >> 4) & 3;
    const uint32_t left = negative(w.rows - 4 * cur.bi - 256) ? (uint32_t)(w.rows - 4 * cur.bi) : 256u;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint32_t l = 16 * g + (tid & 15), on = (bj + l) * w.narrow >> 16, col = 4 * (bj + l - on * bc);
      const size_t at = cur.first + (4 * l + on * (4 * cols - 4 * bc) + r * cols);
      if (4 * on + r < left) {
        if (col + 4 <= cols) {
          if (cols & 3) {
            asm volatile("" ::: "memory");   // (either side: otherwise the two become one, a plain one)
            store_row<DT, true>(out, at, rows[g]);
            asm volatile("" ::: "memory");
          } else {
            store_row<DT>(out, at, rows[g]);
          }
        } else {
#pragma unroll
          for (uint32_t q = 0; q < 3; ++q)
            if (col + q < cols) {
              if constexpr (DT == kF32) static_cast<float*>(out)[at + q] = rows[g][q];
              else static_cast<uint16_t*>(out)[at + q] = (uint16_t)narrow_half<DT>(rows[g][q]);
            }
        }
      }
    }
  } else {
    float y[16];
    rows_to_blocks(rows, y, planes.wave(tid), tid);
    if ((tid & 63) < cur.count(w)) store_block<DT>(out, w, cur.lane(w, tid), y);
  }
}

// sum += the wavefront's blocks, as rows, that the lanes' windows W hold (or = for the first).
// Up to rate 8 nearly all blocks are covered by the matrix; at rate 16 they have too many planes, and
// only the lifting's way is there.  Told by the rate and by the width of the workgroups (see as_matrix).
// Returns kLiftedFirst if the first went the lifting's way, kByMatrix if they went the matrix's, otherwise 0.
//
// The sign of a sum that is zero: where all of a block's parts went the lifting's way it is as added here (tiny
// values round to - 0, and the sum of - 0 and - 0 is - 0).  From the matrix no value is - 0, but its zero times a negative scale
// is, and added to a sum of - 0, which only the lifting's first part leaves, that stays; added as + 0 it would not.
// So with both kinds among the parts no sum may be - 0, and + 0 added at the end sees to it.  (A stream has no sign for a zero.)
constexpr uint32_t kByMatrix = 1u, kLiftedFirst = 2u;
template <int RATE>
__device__ __forceinline__ uint32_t add_blocks(uint32_t (&W)[zc2d::Traits<RATE>::kWords], const uint32_t* token, WavePlanes& planes,
                                           const uint32_t* matrix, char* digits, uint32_t tid, bool first, f32x4 (&sum)[4]) {
  auto b = zc2d::read_block<RATE>(W, token, AnyLane(), planes);
  f32x4 d[4];
  float scale[4];
  uint32_t how = kByMatrix;
  if (AnyLane()(b.r.left > 0) || !matrix_product(planes, b.E, b.lead, matrix, digits, tid, d, scale)) {
    int32_t q[16];
    float y[16];
    zc2d::finish_block<RATE>(b, token, q, AnyLane(), planes);
    zc2d::scale_block(q, b.E, y);
    blocks_to_rows(y, d, planes.wave(tid), tid);
    how = first ? kLiftedFirst : 0u;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      scale[g] = 1.0f;
      if (first) sum[g] = f32x4{-0.0f, -0.0f, -0.0f, -0.0f};   // (what keeps the sign of a zero)
    }
  }
  // (onto + 0 the product of a zero and a negative scale is + 0, as the lifting has it)
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int q = 0; q < 4; ++q) sum[g][q] = __builtin_fmaf(d[g][q], scale[g], sum[g][q]);
  return how;
}
constexpr bool as_matrix(int rate, int threads) { return rate <= 8 && threads == kDecodeThreads; }

// LDS of a kernel that decodes.  The planes come first, so that a lane's are at its number times a constant, and the
// token table late enough for its place and what is taken off a row's index to make an offset that an instruction
// can have (in the decompress kernels of 256 lanes the room for that, 3 KiB, costs more than it gives: 64 x 256 values at rate
// 8 4.14 and 4.19 us; the reduce of 512 x 1024 values at rate 16 13.0 and 12.9).  us with the tables first and as it is: 2-way
// reduce of 8192 x 32768 values at rate 4 457 and 450, at rate 8 623 and 617, 8192 x 8192 at rate 16 303 and 298.
template <int THREADS, bool MATRIX, bool ENCODER>
struct DecodeLds {
  static constexpr int kExpand = ENCODER ? zc2d::kExpandEntries : 4;
  static constexpr int kBefore = THREADS * kPlaneBytes + 4 * kExpand;
  static constexpr int kTokenBias = (int)(zc2d::kTokenFirstRowIndex << zc2d::kIndexShift);
  char planes[THREADS * kPlaneBytes];
  uint32_t expand[kExpand];
  char unused[ENCODER && kBefore < kTokenBias ? kTokenBias - kBefore : 16];
  uint32_t token[zc2d::kTokenRows << zc2d::kLookahead];
  uint32_t matrix[MATRIX ? kMatrixWords : 4];
  char digits[MATRIX ? 16 * THREADS : 16];
};

// (Six wavefronts per SIMD for the forms with the matrix product, which at rate 8 would take 82 registers and leave five.  For the others 1
// says nothing: the compiler makes the same of them without.)
template <int RATE, int DT, int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(as_matrix(RATE, THREADS) ? 6 : 1)))
void decompress2d_kernel(const uint8_t* __restrict__ in, Walk w, void* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) DecodeLds<THREADS, as_matrix(RATE, THREADS), false> lds;
  char* const plane_lds = lds.planes;
  uint32_t *const token = lds.token, *const matrix = lds.matrix;
  if (as_matrix(RATE, THREADS) && threadIdx.x < kMatrixWords / 4)
    reinterpret_cast<uint4*>(matrix)[threadIdx.x] = reinterpret_cast<const uint4*>(&g_matrix)[threadIdx.x];
  stage_table<(zc2d::kTokenRows << zc2d::kLookahead), THREADS>(g_token.v, token);
  constexpr int NW = zc2d::Traits<RATE>::kWords;
  if constexpr (as_matrix(RATE, THREADS)) {
    const uint32_t tid = threadIdx.x;
    WavePlanes planes(plane_lds, tid);
    WaveCursor cur;
    const size_t b0 = first_block<THREADS>();
    if (b0 >= w.blocks) return;
    cur.start(w, b0);
    uint32_t W[NW];
    load_block_words<RATE>(in, cur, w, tid, W);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), for the same reason as in the compress kernel
    for (;;) {
      WaveCursor next = cur;
      next.advance(w);
      const bool more = next.inside(w);
      uint32_t Wn[NW];
      if (more) load_block_words<RATE>(in, next, w, tid, Wn);   // the next blocks' stream, ahead of time
      f32x4 y[4] = {};
      add_blocks<RATE>(W, token, planes, matrix, lds.digits, tid, true, y);
      store_rows<DT>(out, w, cur, planes, tid, y);
      if (!more) break;
#pragma unroll
      for (int i = 0; i < NW; ++i) W[i] = Wn[i];
      cur = next;
    }
  } else {
    const size_t b0 = (size_t)blockIdx.x * THREADS + threadIdx.x;
    if (b0 >= w.blocks) return;
    WavePlanes planes(plane_lds, threadIdx.x);
    Cursor cur;
    cur.start(w, b0);
    uint32_t W[NW];
    load_words<NW>(in + cur.b * zc2d::Traits<RATE>::kBlockBytes, W);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), for the same reason as in the compress kernel
    for (;;) {
      Cursor next = cur;
      next.advance(w);
      const bool more = next.b < w.blocks;
      uint32_t Wn[NW];
      if (more) load_words<NW>(in + next.b * zc2d::Traits<RATE>::kBlockBytes, Wn);   // the next block's stream, ahead of time
      float y[16];
      zc2d::decode_block<RATE>(W, token, y, AnyLane(), planes);
      store_block<DT>(out, w, cur, y);
      if (!more) break;
#pragma unroll
      for (int i = 0; i < NW; ++i) W[i] = Wn[i];
      cur = next;
    }
  }
}

struct ChunkPointers2d {
  const uint8_t* p[16];
};

// What is encoded of a lane's block: where it sticks out of the matrix its fill is taken from the sum's
// last valid row / column.
__device__ __forceinline__ void fill_block(const Walk& w, const Cursor& cur, const float (&sum)[16], uint32_t (&x)[16]) {
  if (cur.whole(w)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = __float_as_uint(sum[i]);
  } else {
    const uint32_t rv = (uint32_t)(w.rows - 4 * cur.bi < 4 ? w.rows - 4 * cur.bi : 4);
    const uint32_t cv = (uint32_t)(w.cols - 4 * cur.bj < 4 ? w.cols - 4 * cur.bj : 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // value at (min(r, rv-1), min(q, cv-1)), picked without indexing registers by a variable
        float v = sum[0];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
#pragma unroll
          for (int qq = 0; qq < 4; ++qq) {
            const bool pick = (uint32_t)rr == ((uint32_t)r < rv ? (uint32_t)r : rv - 1) &&
                              (uint32_t)qq == ((uint32_t)q < cv ? (uint32_t)q : cv - 1);
            v = pick ? sum[4 * rr + qq] : v;
          }
        x[4 * r + q] = __float_as_uint(v);
      }
  }
}

// The reduce-scatter step on matrix-shaped messages: block b of the k chunks is decoded,
// the 16 values are added in registers in chunk order, and the sum is encoded; where the
// block sticks out of the matrix its fill is taken from the sum's last valid row / column.
// LOCAL: a raw fp32 matrix is added last (a ring hop's own contribution); RAW_OUT: the sum
// is stored as an fp32 matrix instead of being encoded (the last hop).
// (Where local values are added the lifting's way is kept: a block per lane is what they are added to, and
// the matrix product, the rows' way back and the local values together took 88 registers and four
// wavefronts per SIMD: 23.8 against 22.4 us for one chunk and fp32 output, 2048 x 6144 values at rate 4.)
// (Six wavefronts per SIMD also for one that adds local values and encodes, which at rate 4 took 82 registers and five: one chunk and local
// values to a stream, 8192 x 8192 values at rate 4, 99.5 and 91.9 us.)
template <int RATE, bool LOCAL, bool RAW_OUT, int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(as_matrix(RATE, THREADS) && !(LOCAL && RAW_OUT) ? 6 : 1)))
void reduce2d_kernel(ChunkPointers2d chunks, int k, const float* local, Walk w, uint8_t* out, float* out_raw) {
  constexpr bool kMatrix = as_matrix(RATE, THREADS) && !LOCAL;
  __shared__ __attribute__((aligned(16))) DecodeLds<THREADS, kMatrix, !RAW_OUT> lds;
  char* const plane_lds = lds.planes;
  uint32_t *const token = lds.token, *const matrix = lds.matrix, *const expand = lds.expand;
  if (kMatrix && threadIdx.x < kMatrixWords / 4)
    reinterpret_cast<uint4*>(matrix)[threadIdx.x] = reinterpret_cast<const uint4*>(&g_matrix)[threadIdx.x];
  if constexpr (!RAW_OUT) {
    for (int i = threadIdx.x; i < zc2d::kExpandEntries / 4; i += THREADS)
      reinterpret_cast<uint4*>(expand)[i] = reinterpret_cast<const uint4*>(g_expand.v)[i];
  }
  stage_table<(zc2d::kTokenRows << zc2d::kLookahead), THREADS>(g_token.v, token);   // (its barrier covers all tables)
  constexpr int NW = zc2d::Traits<RATE>::kWords;
  if constexpr (kMatrix) {
    WaveCursor cur;
    const size_t b0 = first_block<THREADS>();
    if (b0 >= w.blocks) return;
    cur.start(w, b0);
    // The next words, ahead of time: the next chunk's, or the next blocks' of the first.  (us without and with, 2 chunks of
    // 8192 x 32768 values at rate 4: to a stream 438 and 431, to fp32 359 and 324; 6144 x 43690 at rate 8 601 and 595, 447 and 421.)
    uint32_t Wn[NW];
    load_block_words<RATE>(chunks.p[0], cur, w, threadIdx.x, Wn);
    for (;;) {
      WaveCursor next = cur;
      next.advance(w);
      f32x4 rows[4] = {};
      uint32_t how = 0u;
      int j = 0;
#pragma unroll 1
      do {   // (one copy of the decoder, a few hundred instructions, is enough)
        const uint32_t tid = fresh_tid();
        WavePlanes planes(plane_lds, tid);
        uint32_t W[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) W[i] = Wn[i];
        if (j + 1 < k) load_block_words<RATE>(chunks.p[j + 1], cur, w, tid, Wn);
        else if (next.inside(w)) load_block_words<RATE>(chunks.p[0], next, w, tid, Wn);
        how |= add_blocks<RATE>(W, token, planes, matrix, lds.digits, tid, j == 0, rows);
      } while (++j < k);
      const uint32_t tid = fresh_tid();
      const WavePlanes planes(plane_lds, tid);
      if constexpr (RAW_OUT) {
        if (how == (kByMatrix | kLiftedFirst)) {
#pragma unroll
          for (int g = 0; g < 4; ++g) rows[g] += 0.0f;
        }
        store_rows<kF32>(out_raw, w, cur, planes, tid, rows);
      } else {
        float sum[16];
        rows_to_blocks(rows, sum, planes.wave(tid), tid);
        uint32_t x[16], W[NW];
        if (cur.whole(w)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) x[i] = __float_as_uint(sum[i]);
        } else {
          fill_block(w, cur.lane(w, tid), sum, x);
        }
        zc2d::encode_block<RATE>(x, expand, W, AnyLane());
        uint8_t* p = out + cur.b * zc2d::Traits<RATE>::kBlockBytes;
        if ((tid & 63u) < cur.count(w)) store_words<NW>(p + (tid & 63u) * zc2d::Traits<RATE>::kBlockBytes, W);
      }
      cur = next;
      if (!cur.inside(w)) break;
    }
  } else {
    WavePlanes planes(plane_lds, threadIdx.x);
    const size_t b0 = (size_t)blockIdx.x * THREADS + threadIdx.x;
    if (b0 >= w.blocks) return;
    Cursor cur;
    cur.start(w, b0);
    for (;;) {
      const size_t at = cur.b * zc2d::Traits<RATE>::kBlockBytes;
      float sum[16];
#pragma unroll 1
      for (int j = 0; j < k; ++j) {   // (the first chunk in the same loop: the decoder is a few hundred instructions long, one copy of it is enough)
        uint32_t W[NW];
        int32_t q[16];
        load_words<NW>(chunks.p[j] + at, W);
        const uint32_t E = zc2d::decode_block_fixed<RATE>(W, token, q, AnyLane(), planes);
        // scale and add in one fused step, unless some lane's exponent byte is one where the
        // scaling may round or overflow (tiny or huge blocks, arbitrary bytes)
        if (j == 0) {
          zc2d::scale_block(q, E, sum);
        } else if (AnyLane()(!zc2d::scaling_is_exact(E))) {
          float y[16];
          zc2d::scale_block(q, E, y);
#pragma unroll
          for (int i = 0; i < 16; ++i) sum[i] += y[i];
        } else {
          zc2d::accumulate_scaled(q, E, sum);
        }
      }
      if constexpr (LOCAL) {
        // (where the block sticks out of the matrix the clamped loads add copies of edge values;
        // those positions are refilled from the sum or dropped below)
        uint32_t mine[16];
        load_block<kF32>(local, w, cur, mine);
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[i] += __uint_as_float(mine[i]);
      }
      if constexpr (RAW_OUT) {
        store_block<kF32>(out_raw, w, cur, sum);
        cur.advance(w);
        if (cur.b >= w.blocks) break;
        continue;
      }
      uint32_t x[16];
      fill_block(w, cur, sum, x);
      uint32_t W[NW];
      zc2d::encode_block<RATE>(x, expand, W, AnyLane());
      store_words<NW>(out + at, W);
      cur.advance(w);
      if (cur.b >= w.blocks) break;
    }
  }
}

int compute_units() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  return cus;
}

int workgroups_per_cu(int preset) {
#ifdef ZC_TUNING_KNOBS
  if (const char* e = getenv("ZC2D_WORKGROUPS_PER_CU")) {
    const int v = atoi(e);
    if (v >= 1 && v <= 4096) return v;
  }
#endif
  return preset;
}

// preset: workgroups per CU of so many lanes.
unsigned grid_for(size_t blocks, int preset, int threads, int cus) {
  const size_t groups = (blocks + threads - 1) / threads;
  const size_t cap = (size_t)cus * (size_t)workgroups_per_cu(preset);
  return (unsigned)(groups < cap ? groups : cap);
}

// The same for the decoding kernels, whose workgroups stage 22 KiB of token table for 8 to 32 KiB of values per block and
// lane: one workgroup per 512 blocks up to 12 per CU, 12 per CU while that leaves a lane at most two blocks (up to 24 per CU), then
// two blocks per lane up to the preset.  (us at 24 per CU, one block per lane, and at 12: decompress2d of 8192 x
// 6144 bf16 values at rate 8 46.8 and 43.9, at rate 16 86.4 and 84.3; 8192 x 8192 fp32 values, one or two at 24 and two or three at 12, at
// rate 4 47.7 and 45.5, 2-way reduce 115.8 and 113.2; one chunk and local values of 8192 x 6144 at rate 8 99.0 and 94.1.  decompress2d with fp32 rows
// that take the wide grid keeps one: 5000 x 10003 values at rate 4 41.0 and 52.4, 5000 x 10004 41.2 and 56.0.)
unsigned decode_grid_for(size_t blocks, int preset, int threads, int cus) {
  const size_t groups = (blocks + threads - 1) / threads, least = (size_t)cus * kDecodeWorkgroupsPerCULeast;
  const unsigned most = grid_for(blocks, preset, threads, cus);
  if (groups <= least) return most;
  const size_t two = groups / 2 > least ? groups / 2 : least;
  return (unsigned)(two < most ? two : most);
}

// Lanes per workgroup of a decoding kernel: the fewer where the wide ones would not be one per CU.
// (us with 512 and 256 lanes, 2-way reduce at rates 4 and 16: 64 x 256 values 8.6 and 7.3, 16.7 and
// 13.3; 512 x 1024 8.9 and 7.5, 17.0 and 14.0; 700 x 2500, just below the line, 9.1 and 8.9, 17.4
// and 17.2; 1024 x 2048, on it, 9.1 both, 17.4 and 17.3; 2048 x 4096 23.1 and 24.1, 49.1 and 50.3.  On the line at rate 2, where the
// wide form's product gives least, 1024 x 2048 values 5.1 and 4.6 to decompress, 10.5 and 10.0 to reduce three chunks, but with local
// values 5.9 and 6.3.)
int decode_threads(size_t blocks, int rate, bool local, int cus) {
  const size_t line = (size_t)cus * kDecodeThreads;
  return blocks < line || (rate == 2 && !local && blocks == line) ? kDecodeThreadsSmall : kDecodeThreads;
}

// How the wide decoding kernels store values that come as rows.  fp32 rows aligned to their elements only go from a
// block per lane: four pieces of 256 bytes that share cache lines with their neighbours took 0.312 instead of 0.281 ms, 6144 x
// 43690 values at rate 4; of half-precision rows the pieces are better, 40 against 44 us for 8192 x 6145 values.  So it is with rows of
// `per_piece` values' alignment: decompress2d at rates 2 and 4, which wait for memory most, wants the pieces' ends on 64 bytes (us in
// pieces and from a block per lane, the grid being kDecodeWorkgroupsPerCUWide: 5000 x 10004 values 53.5 and 41.2 at rate 2, 52.0 and
// 41.4 at rate 4, but 46.5 and 50.6 at rate 8; 2-way reduce to fp32 at rate 4 59.5 and 63.5).
// With few blocks per block row, a wavefront's 64 blocks span many of these, and a row at a time would write a quarter of each
// cache line, four times: 16 blocks at a time fill whole lines but for both ends (us, decompress2d at rate 4 from a block per lane and
// in pieces: 2097152 x 4 values 43.8 and 10.2, to bf16 15.4 and 10.0, 2-way reduce to fp32 42.7 and 14.9; 400000 x 13 13.6 and
// 11.7, 400001 x 23 18.6 and 17.0; 300001 x 31 16.1 and 15.2; but 262144 x 32 9.4 and 9.8, 65536 x 100 9.4 and 14.1).  Of rows aligned to their
// elements only the ends then meet in the second-level cache (plain stores; without, 400001 x 26 21.6 instead of 16.1; of
// others with them, 1048576 x 8 at rate 8 13.0 instead of 11.6).
uint32_t store_form(size_t cols, bool half, size_t per_piece) {
  const size_t bc = (cols + 3) / 4;
  return (half || cols % per_piece == 0 ? kPieces : 0u) | (bc <= 5 || (bc <= 8 && (cols & 3) != 0) ? kNarrowPieces : 0u);
}

Walk walk_for(size_t rows, size_t cols, unsigned grid, int threads, uint32_t pieces = 0) {
  Walk w;
  w.rows = rows;
  w.cols = cols;
  w.bc = (cols + 3) / 4;
  w.blocks = ((rows + 3) / 4) * w.bc;
  w.whole_br = rows / 4;
  w.whole_bc = cols / 4;
  w.stride = (size_t)grid * threads;
  w.step_bi = w.stride / w.bc;
  w.step_bj = w.stride % w.bc;
  w.pieces = pieces;
  w.narrow = w.bc < 64 ? (uint32_t)((65535 + w.bc) / w.bc) : 0u;
  return w;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
constexpr size_t kMaxValues = (size_t)1 << 40;

}  // namespace

#define ZC2D_DISPATCH_RATE(rate, CALL) \
  switch (rate) {                      \
    case 2: CALL(2); break;            \
    case 4: CALL(4); break;            \
    case 8: CALL(8); break;            \
    case 16: CALL(16); break;          \
    default: return ZC_ERR_RATE;       \
  }

namespace {

template <int DT>
int launch_compress2d(const void* d_in, size_t rows, size_t cols, int rate, void* d_out, size_t out_cap, void* stream) {
  if (!zc2d_rate_supported(rate)) return ZC_ERR_RATE;
  if (rows == 0 || cols == 0) return ZC_OK;
  if (!d_in || !d_out) return ZC_ERR_NULL;
  if (!aligned16(d_in) || !aligned16(d_out)) return ZC_ERR_ALIGN;
  if (rows > kMaxValues || cols > kMaxValues || rows > kMaxValues / cols) return ZC_ERR_SIZE;
  if (out_cap < zc2d_compressed_size(rows, cols, rate)) return ZC_ERR_CAPACITY;
  const size_t blocks = ((rows + 3) / 4) * ((cols + 3) / 4);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int cus = compute_units();
  const unsigned few = grid_for(blocks, kCompressWorkgroupsPerCU, kThreads, cus);
  const unsigned many = grid_for(blocks / 4, kCompressWorkgroupsPerCUMost, kThreads, cus);   // four blocks per lane
  const unsigned grid = few > many ? few : many;
  const Walk w = walk_for(rows, cols, grid, kThreads);
#define CALL(R) hipLaunchKernelGGL((compress2d_kernel<R, DT>), dim3(grid), dim3(kThreads), 0, s, d_in, w, static_cast<uint8_t*>(d_out))
  ZC2D_DISPATCH_RATE(rate, CALL)
#undef CALL
  return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
}

template <int DT>
int launch_decompress2d(const void* d_in, size_t rows, size_t cols, int rate, void* d_out, void* stream) {
  if (!zc2d_rate_supported(rate)) return ZC_ERR_RATE;
  if (rows == 0 || cols == 0) return ZC_OK;
  if (!d_in || !d_out) return ZC_ERR_NULL;
  if (!aligned16(d_in) || !aligned16(d_out)) return ZC_ERR_ALIGN;
  if (rows > kMaxValues || cols > kMaxValues || rows > kMaxValues / cols) return ZC_ERR_SIZE;
  const size_t blocks = ((rows + 3) / 4) * ((cols + 3) / 4);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int cus = compute_units(), threads = decode_threads(blocks, rate, false, cus);
  const zc2d::DecompressGrid g = zc2d::decompress_grid(blocks, cols, DT != kF32, rate);
  const unsigned grid = g.at_once ? grid_for(blocks, g.per_cu, threads, cus) : decode_grid_for(blocks, g.per_cu, threads, cus);
  const Walk w = walk_for(rows, cols, grid, threads, store_form(cols, DT != kF32, rate <= 4 ? 16 : 4));
#define LAUNCH(R, T) hipLaunchKernelGGL((decompress2d_kernel<R, DT, T>), dim3(grid), dim3(T), 0, s, static_cast<const uint8_t*>(d_in), w, d_out)
#define CALL(R)                                                                \
  do {                                                                         \
    if (threads == kDecodeThreadsSmall) LAUNCH(R, kDecodeThreadsSmall);        \
    else LAUNCH(R, kDecodeThreads);                                            \
  } while (0)
  ZC2D_DISPATCH_RATE(rate, CALL)
#undef CALL
#undef LAUNCH
  return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
}

int launch_reduce2d(const void* const* d_in, int k, const float* d_local, size_t rows, size_t cols, int rate, void* d_out,
                    size_t out_cap, float* d_out_raw, void* stream) {
  const bool raw_out = d_out_raw != nullptr;
  if (!zc2d_rate_supported(rate)) return ZC_ERR_RATE;
  if (k < 1 || k > 16) return ZC_ERR_K;
  if (rows == 0 || cols == 0) return ZC_OK;
  if (!d_in || (!raw_out && !d_out)) return ZC_ERR_NULL;
  ChunkPointers2d chunks;
  for (int j = 0; j < 16; ++j) chunks.p[j] = nullptr;
  for (int j = 0; j < k; ++j) {
    if (!d_in[j]) return ZC_ERR_NULL;
    if (!aligned16(d_in[j])) return ZC_ERR_ALIGN;
    chunks.p[j] = static_cast<const uint8_t*>(d_in[j]);
  }
  if (!aligned16(d_out) || !aligned16(d_out_raw) || !aligned16(d_local)) return ZC_ERR_ALIGN;
  if (rows > kMaxValues || cols > kMaxValues || rows > kMaxValues / cols) return ZC_ERR_SIZE;
  if (!raw_out && out_cap < zc2d_compressed_size(rows, cols, rate)) return ZC_ERR_CAPACITY;
  const size_t blocks = ((rows + 3) / 4) * ((cols + 3) / 4);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int cus = compute_units(), threads = decode_threads(blocks, rate, d_local != nullptr, cus);
  // One chunk, local values and fp32 output at rates 2 and 4 wait for memory, and workgroups of one pass of each lane, of which three
  // fit a CU, leave the last ones by themselves: up to six per CU, those that fit take several passes (us with a workgroup per 512
  // blocks and with three per CU, at rate 4: 1100 x 6144 values, 3.2 per CU, 14.8 and 12.8, 1536 x 6144 17.5 and 16.4, 2048 x 6144 20.9 and
  // 19.6, constant values 27.9 and 28.2, with two per CU 31.2; but 3072 x 6144, 9 per CU, 29.6 and 31.0, three chunks of 2048 x 6144 35.4 and
  // 40.1 with two per CU, 2097152 x 4 33.6 and 35.5, 2000 x 5003 19.7 and 20.0).
  const size_t groups = (blocks + threads - 1) / threads;
  const bool few = k == 1 && d_local && raw_out && rate <= 4 && (cols & 3) == 0 && cols >= 32 &&
                   groups > (size_t)cus * 3 && groups <= (size_t)cus * 6;
  const unsigned grid = few ? grid_for(blocks, 3, threads, cus)
                            : decode_grid_for(blocks, raw_out ? kDecodeWorkgroupsPerCUWide : kDecodeWorkgroupsPerCU, threads, cus);
  const Walk w = walk_for(rows, cols, grid, threads, store_form(cols, false, 4));
  uint8_t* out = static_cast<uint8_t*>(d_out);
#define LAUNCH(R, LOCAL, RAW, T) \
  hipLaunchKernelGGL((reduce2d_kernel<R, LOCAL, RAW, T>), dim3(grid), dim3(T), 0, s, chunks, k, d_local, w, out, d_out_raw)
#define FORMS(R, T)                                   \
  do {                                                \
    if (d_local && raw_out) LAUNCH(R, true, true, T); \
    else if (d_local) LAUNCH(R, true, false, T);      \
    else if (raw_out) LAUNCH(R, false, true, T);      \
    else LAUNCH(R, false, false, T);                  \
  } while (0)
#define CALL(R)                                                        \
  do {                                                                 \
    if (threads == kDecodeThreadsSmall) FORMS(R, kDecodeThreadsSmall); \
    else FORMS(R, kDecodeThreads);                                     \
  } while (0)
  ZC2D_DISPATCH_RATE(rate, CALL)
#undef CALL
#undef FORMS
#undef LAUNCH
  return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int zc2d_rate_supported(int rate) { return rate == 2 || rate == 4 || rate == 8 || rate == 16; }

size_t zc2d_compressed_size(size_t rows, size_t cols, int rate) {
  if (!zc2d_rate_supported(rate)) return 0;
  return ((rows + 3) / 4) * ((cols + 3) / 4) * (size_t)(2 * rate);
}

int zc2d_compress(const float* d_in, size_t rows, size_t cols, int rate, void* d_out, size_t out_cap, void* stream) {
  return launch_compress2d<kF32>(d_in, rows, cols, rate, d_out, out_cap, stream);
}

int zc2d_decompress(const void* d_in, size_t rows, size_t cols, int rate, float* d_out, void* stream) {
  return launch_decompress2d<kF32>(d_in, rows, cols, rate, d_out, stream);
}

int zc2d_compress_half(const void* d_in, int dtype, size_t rows, size_t cols, int rate, void* d_out, size_t out_cap,
                       void* stream) {
  if (dtype == ZC_BF16) return launch_compress2d<kBF16>(d_in, rows, cols, rate, d_out, out_cap, stream);
  if (dtype == ZC_F16) return launch_compress2d<kF16>(d_in, rows, cols, rate, d_out, out_cap, stream);
  return ZC_ERR_DTYPE;
}

int zc2d_decompress_half(const void* d_in, size_t rows, size_t cols, int rate, int dtype, void* d_out, void* stream) {
  if (dtype == ZC_BF16) return launch_decompress2d<kBF16>(d_in, rows, cols, rate, d_out, stream);
  if (dtype == ZC_F16) return launch_decompress2d<kF16>(d_in, rows, cols, rate, d_out, stream);
  return ZC_ERR_DTYPE;
}

int zc2d_reduce_compressed(const void* const* d_in, int k, size_t rows, size_t cols, int rate, void* d_out,
                           size_t out_cap, void* stream) {
  return launch_reduce2d(d_in, k, nullptr, rows, cols, rate, d_out, out_cap, nullptr, stream);
}

int zc2d_reduce_mixed(const void* const* d_in, int k, const float* d_local, size_t rows, size_t cols, int rate, void* d_out,
                      size_t out_cap, void* stream) {
  return launch_reduce2d(d_in, k, d_local, rows, cols, rate, d_out, out_cap, nullptr, stream);
}

int zc2d_reduce_decompress(const void* const* d_in, int k, const float* d_local, size_t rows, size_t cols, int rate,
                           float* d_out, void* stream) {
  if (zc2d_rate_supported(rate) && k >= 1 && k <= 16 && rows != 0 && cols != 0 && !d_out) return ZC_ERR_NULL;
  return launch_reduce2d(d_in, k, d_local, rows, cols, rate, nullptr, 0, d_out, stream);
}

}  // extern "C"
