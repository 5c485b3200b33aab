// zl_kernels.hip -- gfx950 kernels and C ABI for the lossless codec (see include/zc.h).
//
// One workgroup of 256 lanes per chunk of 8192 words; a lane owns one group of 32 words
// (its eight 16-byte reads), so residuals, the bit transpose and the test for empty
// planes all stay in registers.  A workgroup-wide prefix sum of the per-lane plane counts
// gives every lane its place in the chunk; each wavefront then moves its planes between
// registers and its contiguous span of the stream through 4 KiB of LDS of its own, half
// of its lanes at a time, with no further barrier (16 KiB of LDS per workgroup, so that
// seven workgroups fit on a CU and hide each other's waits).
//
// Chunks have data-dependent sizes, so a chunk's place in the stream is the sum of the
// sizes before it.  That sum is formed in the same launch.  A workgroup publishes a chunk's own
// size in the stream's table as soon as that is known, which is before its planes are formed;
// later it adds up the entries of the chunks before it, 64 at a time, back to the nearest
// entry that already holds a running total, replaces the chunk's entry by its own running total
// and writes the chunk.
// Messages of up to two and a half times as many chunks as workgroups fit on the chip have a
// workgroup per chunk.  For longer ones about as many workgroups run as fit, and each asks for chunk numbers,
// one after the other.  A coded chunk then waits in registers while its workgroup codes the next
// one, and only after that looks for its place: by then most of what the sum needs has arrived,
// so the look-back rarely has to poll.  (Chunks b, b + G, b + 2G, ... for workgroup b of G need no
// asking, but all wait for the slowest: 2^28 fp32 words took 0.466 instead of 0.403 ms.)
// A counter serves one request in about 11.5 ns, however many workgroups ask, so there are
// eight, one for each remainder of the chunk number: each is a field of 19 bits in the table
// entry of an early chunk, between its byte count and its state bits, on a cache line of its
// own, and the last to ask clears it.  (A single one takes 0.38 ms for the 32768 chunks of 2^28
// words; with it the kernel took 0.457 ms.)
// A workgroup that is waited for may not run yet: its number may be one that no workgroup has asked
// for, and a workgroup per chunk has to wait for its place on its die (with 24 of one die's 32 CUs
// held by another kernel 2048 x 6144 words take 0.068 instead of 0.036 ms).  Nobody waits for good
// all the same: a workgroup that has polled for a while in vain works out the missing chunks' sizes
// itself (a size depends on the message alone) and goes on.
// With all this, the residuals' or as the bitmap, byte permutes in the transpose and 16-bit
// groups kept as 16 registers: 2^28 fp32 words 0.452 -> 0.390 ms (5.2 TB/s of message and
// stream), as 16-bit words 0.332 -> 0.253 ms; 2048 x 6144 words 0.056 -> 0.031 ms, as 16-bit words
// 0.036 -> 0.020 ms.
// The table is part of the stream (the decoder needs it): no memory beyond input and output
// is used.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "../../include/zc.h"
#include "zl_codec.h"

namespace {

constexpr int kThreads = zl::kGroups;
using zl::kCounters;
using zl::kCounterStride;
constexpr uint32_t kPatience = 256;     // polls of the table (about 1 us each) before a workgroup helps itself
template <bool HALF> constexpr int kMinWavesPerSimd = HALF ? 7 : 4;   // registers per lane: 72 and 128, of which the kernels use 72 and 113
constexpr int kWaveStageWords = 32 * 33;   // planes of 32 lanes: a wavefront's LDS, one spare word per 32

// Where plane word i of a half-wavefront sits in its LDS.  Lanes reach their planes with a
// stride of their plane count (32 if nothing is dropped): the spare word per 32 keeps such
// strides off a single bank, and consecutive words stay consecutive for the copy.
__device__ __forceinline__ uint32_t staged(uint32_t i) { return i + (i >> 5); }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t Word4 __attribute__((ext_vector_type(4), aligned(4)));   // four words of the stream

struct Header {
  uint32_t magic;
  uint32_t chunks;
  uint64_t n;
  uint64_t total;
  uint64_t reserved;   // zero
};
static_assert(sizeof(Header) == zl::kHeaderBytes, "header layout");

__global__ __launch_bounds__(256) void zero_words_kernel(uint64_t* p, size_t count) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) p[i] = 0;
}

// The stream of an empty message: the header alone.
__global__ void empty_stream_kernel(Header* header) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    header->magic = zl::kMagic;
    header->chunks = 0;
    header->n = 0;
    header->total = zl::kHeaderBytes;
    header->reserved = 0;
  }
}

// Inclusive prefix sum over the wavefront.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)v, d);
    v += lane >= d ? up : 0u;
  }
  return v;
}

__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d);
    v += (uint64_t)hi << 32 | lo;
  }
  return v;
}

// Places of the planes within a chunk, from the per-lane counts.
struct Places {
  uint32_t in_wave;      // planes of lower lanes of the same wavefront
  uint32_t wave_total;   // planes of the whole wavefront
  uint32_t wave_start;   // planes of lower wavefronts
  uint32_t total;        // planes of the chunk
};

// The 256 lanes of a chunk are four consecutive wavefronts of the workgroup (which may hold
// more than one chunk).
__device__ __forceinline__ Places workgroup_places(uint32_t count, uint32_t* wave_totals) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_sum(count, lane);
  if (lane == 63) wave_totals[wave] = incl;
  __syncthreads();
  Places p;
  p.in_wave = incl - count;
  // (the same in every lane of the wavefront: these go to scalar registers)
  const uint32_t first_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave) & ~3u;
  p.wave_total = 0;
  p.wave_start = 0;
  p.total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_totals[first_wave + w]);
    const uint32_t ahead = (uint32_t)__builtin_amdgcn_readfirstlane(wave & 3);
    p.wave_start += (uint32_t)w < ahead ? t : 0u;
    p.wave_total = (uint32_t)w == ahead ? t : p.wave_total;
    p.total += t;
  }
  return p;
}

// Span, within the wavefront's planes, of the half of its lanes that starts at lane 32*half.
__device__ __forceinline__ void half_span(const Places& p, int half, uint32_t& start, uint32_t& end) {
  const uint32_t middle = (uint32_t)__shfl((int)p.in_wave, 32);
  start = half ? middle : 0u;
  end = half ? p.wave_total : middle;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The lane's group of chunk c: words 1024*t + 4*tid .. +3 of the chunk, t = 0..7; words
// past the end of the message read as zero.
__device__ __forceinline__ void load_group(const void* __restrict__ message, size_t n, uint32_t c, int tid, uint32_t (&w)[32]) {
  const size_t base = (size_t)c * zl::kChunkWords;
  const uint32_t* in = static_cast<const uint32_t*>(message);
  if (base + zl::kChunkWords <= n) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(in + base + 1024 * t + 4 * tid));
      w[4 * t] = v.x; w[4 * t + 1] = v.y; w[4 * t + 2] = v.z; w[4 * t + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const size_t i = base + 1024 * (j >> 2) + 4 * tid + (j & 3);
      w[j] = i < n ? in[i] : 0u;
    }
  }
}

// The same for 16-bit words, two to a register: word j in the lower, word j + 16 in the upper half
// of register j.
__device__ __forceinline__ void load_group_of_halves(const void* __restrict__ message, size_t n, uint32_t c, int tid, uint32_t (&w)[16]) {
  const size_t base = (size_t)c * zl::kChunkWords;
  const uint16_t* in = static_cast<const uint16_t*>(message);
  if (base + zl::kChunkWords <= n) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x2 a = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(in + base + 1024 * t + 4 * tid));
      const u32x2 b = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(in + base + 1024 * (t + 4) + 4 * tid));
      w[4 * t] = zl::permute_bytes(b.x, a.x, 0x05040100u);
      w[4 * t + 1] = zl::permute_bytes(b.x, a.x, 0x07060302u);
      w[4 * t + 2] = zl::permute_bytes(b.y, a.y, 0x05040100u);
      w[4 * t + 3] = zl::permute_bytes(b.y, a.y, 0x07060302u);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const size_t i = base + 1024 * (j >> 2) + 4 * tid + (j & 3), k = i + 4 * 1024;
      w[j] = (i < n ? in[i] : 0u) | (k < n ? (uint32_t)in[k] << 16 : 0u);
    }
  }
}

// The reverse; HALF keeps the upper halves of the words.
template <bool HALF>
__device__ __forceinline__ void store_group(void* __restrict__ message, size_t n, uint32_t c, int tid, const uint32_t (&w)[32]) {
  const size_t base = (size_t)c * zl::kChunkWords;
  if constexpr (HALF) {
    uint16_t* out = static_cast<uint16_t*>(message);
    if (base + zl::kChunkWords <= n) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const u32x2 v = {w[4 * t] >> 16 | (w[4 * t + 1] & 0xFFFF0000u), w[4 * t + 2] >> 16 | (w[4 * t + 3] & 0xFFFF0000u)};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x2*>(out + base + 1024 * t + 4 * tid));
      }
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const size_t i = base + 1024 * (j >> 2) + 4 * tid + (j & 3);
        if (i < n) out[i] = (uint16_t)(w[j] >> 16);
      }
    }
  } else {
    uint32_t* out = static_cast<uint32_t*>(message);
    if (base + zl::kChunkWords <= n) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const u32x4 v = {w[4 * t], w[4 * t + 1], w[4 * t + 2], w[4 * t + 3]};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + base + 1024 * t + 4 * tid));
      }
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) {
        const size_t i = base + 1024 * (j >> 2) + 4 * tid + (j & 3);
        if (i < n) out[i] = w[j];
      }
    }
  }
}

// Sets entry c of the table, to the chunk's own size or to its running total.  In an entry that
// counts, the counter's field is left alone.
__device__ __forceinline__ void publish(uint64_t* table, uint32_t c, uint64_t entry) {
  if (c % kCounterStride != 0 || c >= kCounters * kCounterStride) {
    __hip_atomic_store(&table[c], entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    uint64_t old = __hip_atomic_load(&table[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (!__hip_atomic_compare_exchange_strong(&table[c], &old, (old & zl::kTicketMask) | entry, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    }
  }
}

// Whether workgroups publish the sizes of the chunks they code.  They do; only with the tuning knobs,
// ZL_PATIENCE=0 keeps them from it, so that every size has to be worked out by those that wait for it.
__device__ __forceinline__ bool sizes_are_published(uint32_t patience) {
#ifdef ZC_TUNING_KNOBS
  return patience != 0;
#else
  return true;
#endif
}

// The workgroup's next chunk number, or `chunks` if there is none.  It asks its counter until it
// gets a number past the end, so a counter's last request is known by its number, and clears the
// field: the grid is a multiple of kCounters, and so as many workgroups ask each counter.
__device__ __forceinline__ uint32_t next_chunk(uint64_t* table, uint32_t chunks) {
  const uint32_t i = zl::counter_of(blockIdx.x);
  uint64_t* entry = &table[kCounterStride * i];
  const uint64_t old = __hip_atomic_fetch_add(entry, (uint64_t)1 << zl::kTicketShift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t ticket = (uint32_t)((old & zl::kTicketMask) >> zl::kTicketShift);
  const uint32_t tickets = (chunks - i + kCounters - 1) / kCounters;
  // (what was added is taken away again; a mask for the field, a constant of 64 bits, would be kept in
  // memory throughout the 16-bit kernel for want of registers)
  if (ticket + 1 == tickets + gridDim.x / kCounters)
    __hip_atomic_fetch_add(entry, 0 - ((uint64_t)(ticket + 1) << zl::kTicketShift), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return ticket < tickets ? i + kCounters * ticket : chunks;
}

// Bytes that chunk c takes in the payload, worked out from the message by one whole wavefront (two
// passes over the chunk, few registers: this is the exception).
template <bool HALF>
__device__ uint64_t size_of_chunk(const void* __restrict__ message, size_t n, uint32_t c, int lane) {
  const size_t base = (size_t)c * zl::kChunkWords;
  auto word = [&](int tid, int j) {
    const size_t i = base + 1024 * (j >> 2) + 4 * tid + (j & 3);
    if constexpr (HALF) return i < n ? (uint32_t)static_cast<const uint16_t*>(message)[i] << 16 : 0u;
    else return i < n ? static_cast<const uint32_t*>(message)[i] : 0u;
  };
  uint32_t planes = 0;
#pragma unroll 1
  for (int tid = lane; tid < kThreads; tid += 64) planes += zl::planes_of_group([&](int j) { return word(tid, j); });
  return zl::kFixedChunkBytes + 4 * wave_sum64(planes);
}

// Sum of the sizes of chunks 0..c-1, read from the table (run by one whole wavefront):
// 64 entries per pass, the lane's being the chunk at distance lane + 1 before c.  (Wider
// passes were slower: the polls of all workgroups in flight fall on the same few hundred
// table entries, and it is the number of these loads that costs.)  Where entries stay empty,
// the wavefront works one of them out after the other, its pick among the empty ones
// depending on c, so that several wavefronts in want of the same entries share the work; the
// chunk's own workgroup may publish the same size at any time.
template <bool HALF>
__device__ uint64_t bytes_before(uint64_t* table, const void* __restrict__ message, size_t n, uint32_t c, int lane,
                                 uint32_t patience) {
  uint64_t sum = 0;
  int64_t base = (int64_t)c - 1;
  uint32_t polls = 0;
  while (base >= 0) {
    const int64_t idx = base - lane;
    uint64_t s = 0;
    uint32_t first = 64;
    for (;;) {
      s = idx >= 0 ? __hip_atomic_load(&table[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : zl::kEnd;
      const uint64_t totals = __builtin_amdgcn_ballot_w64((s >> 62) == 2u);
      const uint64_t empty = __builtin_amdgcn_ballot_w64((s >> 62) == 0u);
      first = totals ? (uint32_t)__builtin_ctzll(totals) : 64u;
      const uint64_t needed = first >= 63u ? ~0ull : ((2ull << first) - 1ull);
      uint64_t missing = empty & needed;
      if (missing == 0) break;
      if (++polls > patience) {
        for (uint32_t skip = c % (uint32_t)__builtin_popcountll(missing); skip != 0; --skip) missing &= missing - 1;
        const uint32_t other = (uint32_t)(base - __builtin_ctzll(missing));
        const uint64_t size = size_of_chunk<HALF>(message, n, other, lane);
        if (lane == 0) {   // (unless the entry has changed meanwhile; if only its counter has, this is done again)
          uint64_t old = __hip_atomic_load(&table[other], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((old >> 62) == 0u)
            __hip_atomic_compare_exchange_strong(&table[other], &old, old | zl::kOwnSize | size, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        }
      } else {
        __builtin_amdgcn_s_sleep(2);
      }
    }
    sum += wave_sum64((uint32_t)lane <= first ? (s & zl::kValueMask & ~zl::kTicketMask) : 0ull);
    if (first != 64u) break;
    base -= 64;
  }
  return sum;
}

// A coded chunk that waits, in registers, for its place in the stream.
// A group of 16-bit words has planes 16 and up only.
template <bool HALF>
struct Coded {
  static constexpr int kPlanes = HALF ? 16 : 32;
  uint32_t planes[kPlanes];
  uint32_t reference, bitmap, chunk;
  Places at;
};

template <bool HALF>
__global__ __launch_bounds__(kThreads, kMinWavesPerSimd<HALF>) void zl_compress_kernel(const void* __restrict__ in, size_t n, uint8_t* out,
                                                                  uint32_t chunks, bool counted, uint32_t patience) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t stage[kWaveStageWords * kWaves];
  __shared__ uint32_t wave_totals[kWaves];
  __shared__ uint64_t my_start;
  __shared__ uint32_t next;
  Header* header = reinterpret_cast<Header*>(out);
  uint64_t* table = reinterpret_cast<uint64_t*>(out + zl::kHeaderBytes);
  uint8_t* payload = out + zl::kHeaderBytes + 8 * (size_t)chunks;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // A workgroup codes chunk after chunk.  A chunk's size is published as soon as it is known;
  // its place is worked out, and it is written, only after the next chunk has been coded in turn,
  // by which time most of what its place depends on has arrived.
  Coded<HALF> held;
  bool holding = false;
  uint32_t c = blockIdx.x;
  if (counted) {
    if (threadIdx.x == 0) next = next_chunk(table, chunks);
    __syncthreads();
    c = next;
    __syncthreads();
  }
  for (;;) {
    // (The lane's number anew in every pass: what is worked out from it, three dozen offsets, would
    // otherwise be kept across the passes, in memory, for want of registers.)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const bool coding = c < chunks;
    Coded<HALF> now;
    if (coding) {
      if constexpr (HALF) {
        load_group_of_halves(in, n, c, tid, now.planes);
        now.bitmap = zl::to_residuals_of_halves(now.planes, now.reference);
      } else {
        load_group(in, n, c, tid, now.planes);
        now.bitmap = zl::to_residuals(now.planes, now.reference);
      }
      now.chunk = c;
      now.at = workgroup_places((uint32_t)__builtin_popcount(now.bitmap), wave_totals);
      if (tid == 0 && (c == 0 || sizes_are_published(patience))) publish(table, c, (c == 0 ? zl::kEnd : zl::kOwnSize) | (zl::kFixedChunkBytes + 4ull * now.at.total));
      zl::transpose(now.planes);
    }
    if (holding) {
      if (wave == 0) {
        const uint64_t bytes = zl::kFixedChunkBytes + 4ull * held.at.total;
        const uint64_t before = held.chunk == 0 ? 0 : bytes_before<HALF>(table, in, n, held.chunk, lane, patience);
        if (lane == 0) {
          if (held.chunk != 0) publish(table, held.chunk, zl::kEnd | (before + bytes));
          my_start = before;
          if (held.chunk == chunks - 1) {   // the last chunk's end is the stream's
            header->magic = zl::kMagic;
            header->chunks = chunks;
            header->n = n;
            header->total = zl::kHeaderBytes + 8ull * chunks + before + bytes;
          }
        }
      }
      __syncthreads();
    }
    // the next chunk number travels while the held chunk is written
    uint32_t asked = chunks;
    if (coding && counted && tid == 0) asked = next_chunk(table, chunks);
    if (holding) {
      uint32_t* dst = reinterpret_cast<uint32_t*>(payload + my_start);
      dst[tid] = held.reference;
      dst[kThreads + tid] = held.bitmap;
      dst += 2 * kThreads + held.at.wave_start;
      // the wavefront's planes, as many lanes at a time as the LDS holds: into it by lane, out of it
      // by address, four words per lane and step (LDS operations of one wavefront take effect in
      // program order; the stream is aligned to words only, which a global store of any width may be)
      constexpr int kPlanes = Coded<HALF>::kPlanes, kParts = HALF ? 1 : 2;
      uint32_t* mine = stage + kWaveStageWords * wave;
#pragma unroll 1
      for (int part = 0; part < kParts; ++part) {
        uint32_t start = 0, end = held.at.wave_total;
        if (kParts == 2) half_span(held.at, part, start, end);
        if (kParts == 1 || (lane >> 5) == part) {
          uint32_t pos = held.at.in_wave - start;
#pragma unroll
          for (int k = 0; k < kPlanes; ++k)
            if ((held.bitmap >> (32 - kPlanes + k)) & 1u) mine[staged(pos++)] = held.planes[k];
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t count = end - start, whole = count & ~3u;
        for (uint32_t i = 4 * lane; i < whole; i += 256) {
          const uint32_t* p = mine + staged(i);   // (four words from a multiple of 4 on lie together)
          const Word4 v = {p[0], p[1], p[2], p[3]};
          *reinterpret_cast<Word4*>(dst + start + i) = v;
        }
        if ((uint32_t)lane < count - whole) dst[start + whole + lane] = mine[staged(whole + lane)];
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (!coding) break;
    held = now;
    holding = true;
    if (tid == 0) next = asked;
    __syncthreads();   // (also: the totals and the start are used again)
    c = next;
  }
}

// in_bytes: size of the buffer that holds the stream; every read stays below it.
template <bool HALF>
__global__ __launch_bounds__(kThreads) void zl_decompress_kernel(const uint8_t* __restrict__ in, size_t in_bytes, size_t n,
                                                                 void* __restrict__ out, uint32_t chunks) {
  __shared__ uint32_t stage[zl::kChunkWords + zl::kChunkWords / 32 + 64];   // spare words as in staged(); a lane may look one past its last plane
  __shared__ uint32_t wave_totals[kThreads / 64];
  const uint64_t* table = reinterpret_cast<const uint64_t*>(in + zl::kHeaderBytes);
  const uint64_t room = in_bytes - zl::kHeaderBytes - 8 * (uint64_t)chunks;   // the host checked that this is not negative
  const uint32_t* payload = reinterpret_cast<const uint32_t*>(in + zl::kHeaderBytes + 8 * (size_t)chunks);
  const int tid = threadIdx.x;
  const uint32_t c = blockIdx.x;

  // the chunk's span, clamped to the buffer and to whole words
  uint64_t end = table[c] & zl::kValueMask, start = c ? table[c - 1] & zl::kValueMask : 0;
  end = end < room ? end : room;
  start = start < end ? start : end;
  const uint64_t first_word = (start + 3) / 4, words = end / 4 > first_word ? end / 4 - first_word : 0;
  const uint32_t* src = payload + first_word;

  const uint32_t reference = (uint64_t)tid < words ? src[tid] : 0u;
  const uint32_t bitmap = (uint64_t)(kThreads + tid) < words ? src[kThreads + tid] : 0u;
  // the chunk's plane words, as many as the span really holds: fetched by address before
  // anything is known about them, 32 loads in flight per lane
  const uint64_t held = words > 2 * kThreads ? words - 2 * kThreads : 0;
  const uint32_t stored = held < (uint64_t)zl::kChunkWords ? (uint32_t)held : (uint32_t)zl::kChunkWords;
  src += 2 * kThreads;
  // (a chunk that holds 16 planes per group or fewer, as every chunk of a 16-bit message does,
  // needs the first half of these loads and of the staging only; what a malformed stream then
  // picks up beyond its span is whatever the staging area held, which is as unspecified as
  // zeros would be)
  const bool upper_half = stored > 16u * kThreads;
  uint32_t p[32];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const uint32_t i = tid + kThreads * q;
    p[q] = i < stored ? src[i] : 0u;
  }
  if (upper_half) {
#pragma unroll
    for (int q = 16; q < 32; ++q) {
      const uint32_t i = tid + kThreads * q;
      p[q] = i < stored ? src[i] : 0u;
    }
  }
  const Places at = workgroup_places((uint32_t)__builtin_popcount(bitmap), wave_totals);
#pragma unroll
  for (int q = 0; q < 16; ++q) stage[staged(tid + kThreads * q)] = p[q];
  if (upper_half) {
#pragma unroll
    for (int q = 16; q < 32; ++q) stage[staged(tid + kThreads * q)] = p[q];
  }
  __syncthreads();
  uint32_t pos = at.wave_start + at.in_wave;
  if constexpr (HALF) {
    // A stream made from 16-bit words has no planes below 16 and references with empty lower
    // halves.  Where that holds for every lane of the wavefront, only the upper 16 planes are
    // picked up and the lower ones are zeros the compiler can see, which takes a third off the
    // transpose as well; any other stream (arbitrary bytes) goes the general way below.
    const bool as_made = ((bitmap | reference) & 0xFFFFu) == 0u;
    if (__builtin_amdgcn_ballot_w64(!as_made) == 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) p[k] = 0u;
#pragma unroll
      for (int k = 16; k < 32; ++k) {
        const bool present = (bitmap >> k) & 1u;
        p[k] = present ? stage[staged(pos)] : 0u;
        pos += present ? 1u : 0u;
      }
      zl::from_planes(p, reference);
      store_group<HALF>(out, n, c, tid, p);
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const bool present = (bitmap >> k) & 1u;
    p[k] = present ? stage[staged(pos)] : 0u;
    pos += present ? 1u : 0u;
  }
  zl::from_planes(p, reference);
  store_group<HALF>(out, n, c, tid, p);
}

int compute_units() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  return cus;
}

// Workgroups of the compress kernel per CU: as many as the registers allow.
// (Only a build with -DZC_TUNING_KNOBS lets ZL_WORKGROUPS_PER_CU override it, and ZL_PATIENCE the
// number of polls before a workgroup works out missing sizes itself; with 0, see sizes_are_published.)
int workgroups_per_cu(int preset) {
#ifdef ZC_TUNING_KNOBS
  if (const char* e = getenv("ZL_WORKGROUPS_PER_CU")) {
    const int v = atoi(e);
    if (v >= 1 && v <= 64) return v;
  }
#endif
  return preset;
}

uint32_t patience() {
#ifdef ZC_TUNING_KNOBS
  if (const char* e = getenv("ZL_PATIENCE")) return (uint32_t)atoi(e);
#endif
  return kPatience;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
constexpr size_t kMaxWords = (size_t)1 << 40;

size_t chunks_of(size_t n) { return (n + zl::kChunkWords - 1) / zl::kChunkWords; }

}  // namespace

namespace {
template <bool HALF>
int launch_zl_compress(const void* d_in, size_t n, void* d_out, size_t out_cap, void* stream) {
  if (!d_out || (n && !d_in)) return ZC_ERR_NULL;
  if (!aligned16(d_in) || !aligned16(d_out)) return ZC_ERR_ALIGN;
  if (n > kMaxWords) return ZC_ERR_SIZE;
  if (out_cap < zl_max_compressed_size(n)) return ZC_ERR_CAPACITY;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t chunks = chunks_of(n);
  if (chunks == 0) {
    hipLaunchKernelGGL(empty_stream_kernel, dim3(1), dim3(64), 0, s, static_cast<Header*>(d_out));
    return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
  }
  // header and table start as zeros: the empty table entries, the reserved word
  // (a fill kernel rather than a memset node, so that the call can be captured in a graph)
  const size_t clear = (zl::kHeaderBytes + 8 * chunks) / 8;
  const unsigned zgrid = (unsigned)((clear + 255) / 256 < 1024 ? (clear + 255) / 256 : 1024);
  hipLaunchKernelGGL(zero_words_kernel, dim3(zgrid), dim3(256), 0, s, static_cast<uint64_t*>(d_out), clear);
  if (hipGetLastError() != hipSuccess) return ZC_ERR_LAUNCH;
  const size_t resident = (size_t)compute_units() * workgroups_per_cu(kMinWavesPerSimd<HALF>);
  // a workgroup per chunk up to two and a half times as many as run at a time (us, a workgroup per
  // chunk against asking for numbers: 2048 chunks of 32-bit words 37.7 and 41.6, 2320 44.6 and 46.7,
  // 2930 51.9 and 51.2, 3418 61.9 and 56.8; of 16-bit words 3589 41.0 and 43.1, 4395 49.9 and 48.8),
  // and where a counter's field of 19 bits is too small: beyond 2^22 chunks, 2^35 words
  const bool countable = chunks / kCounters + resident < ((size_t)1 << (62 - zl::kTicketShift));
  const unsigned grid = (unsigned)(chunks <= 5 * resident / 2 || !countable ? chunks : resident / kCounters * kCounters);
  hipLaunchKernelGGL((zl_compress_kernel<HALF>), dim3(grid), dim3(kThreads), 0, s, d_in, n,
                     static_cast<uint8_t*>(d_out), (uint32_t)chunks, grid < chunks, patience());
  return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
}

template <bool HALF>
int launch_zl_decompress(const void* d_in, size_t in_bytes, size_t n, void* d_out, void* stream) {
  if (!d_in || (n && !d_out)) return ZC_ERR_NULL;
  if (!aligned16(d_in) || !aligned16(d_out)) return ZC_ERR_ALIGN;
  if (n > kMaxWords) return ZC_ERR_SIZE;
  const size_t chunks = chunks_of(n);
  if (in_bytes < zl::kHeaderBytes + 8 * chunks) return ZC_ERR_CAPACITY;
  if (chunks == 0) return ZC_OK;
  hipLaunchKernelGGL(zl_decompress_kernel<HALF>, dim3((unsigned)chunks), dim3(kThreads), 0, static_cast<hipStream_t>(stream),
                     static_cast<const uint8_t*>(d_in), in_bytes, n, d_out, (uint32_t)chunks);
  return hipGetLastError() == hipSuccess ? ZC_OK : ZC_ERR_LAUNCH;
}
}  // namespace

extern "C" {

size_t zl_max_compressed_size(size_t n) {
  if (n > kMaxWords) return 0;
  return zl::kHeaderBytes + chunks_of(n) * (size_t)(8 + zl::kFixedChunkBytes + 4 * zl::kChunkWords);
}

int zl_compress(const void* d_in, size_t n, void* d_out, size_t out_cap, void* stream) {
  return launch_zl_compress<false>(d_in, n, d_out, out_cap, stream);
}

int zl_compress16(const void* d_in, size_t n, void* d_out, size_t out_cap, void* stream) {
  return launch_zl_compress<true>(d_in, n, d_out, out_cap, stream);
}

int zl_stream_bytes(const void* d_stream, size_t* h_bytes, void* stream) {
  if (!d_stream || !h_bytes) return ZC_ERR_NULL;
  Header h;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(&h, d_stream, sizeof h, hipMemcpyDeviceToHost, s) != hipSuccess) return ZC_ERR_LAUNCH;
  if (hipStreamSynchronize(s) != hipSuccess) return ZC_ERR_LAUNCH;
  if (h.magic != zl::kMagic || h.reserved != 0) return ZC_ERR_STREAM;
  *h_bytes = (size_t)h.total;
  return ZC_OK;
}

int zl_decompress(const void* d_in, size_t in_bytes, size_t n, void* d_out, void* stream) {
  return launch_zl_decompress<false>(d_in, in_bytes, n, d_out, stream);
}

int zl_decompress16(const void* d_in, size_t in_bytes, size_t n, void* d_out, void* stream) {
  return launch_zl_decompress<true>(d_in, in_bytes, n, d_out, stream);
}

}  // extern "C"
