// k_container.hip -- gfx950 kernels for the container operations of a
// particle set: removal by overwriting with the last particle (Section 2),
// and the zero fill used when a set grows.
//
// Removal is the sequential algorithm "while particle i is flagged, copy the
// last particle over it and shrink the set", computed in parallel from its
// closed form: with m flagged particles and n' = n - m survivors, the flagged
// slots below n' (ascending) receive the unflagged particles at or above n'
// taken from the end (descending).  Four passes: per-tile flag counts, their
// exclusive sums (one workgroup, which also hands m to the host), per-element
// ranks into two lists (holes and movers), and the moves themselves.
//
// What bounds it is the moves' writes: a hole is a few bytes in a line of its
// own, and this memory takes a write of part of 64 bytes as slowly as a read
// and a write of all of them (8e6 scattered 8-byte stores 320-370 us, whole
// 64-byte stores to the same places 104 us, with the read that would need
// 397 us).  Removing 1% of 1e8 particles from both copies, with the resize
// before it: 633 us when the host summed the counts and every array had its
// own zero fill, 487 us now, of which the moves take 320 to 355; from a set of
// 1000 particles 150 us before, 45 us now.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "launch.h"

namespace soax {

namespace {

constexpr int kBlock = 256;
// A thread takes kItems consecutive flags of a tile as kLoads 16-byte loads,
// all in flight at once.
constexpr int kItems = 64;
constexpr int kLoads = kItems / 16;
constexpr int64_t kTile = int64_t(kBlock) * kItems;

// Bit j (0..3) set iff byte j of w is nonzero: adding 0x7F to the low seven
// bits of a byte carries into its bit 7 iff they are not all zero, and no
// carry leaves the byte.
__device__ __forceinline__ uint32_t nonzero_bytes4(uint32_t w) {
  const uint32_t hi = (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
  return ((hi >> 7) & 1u) | ((hi >> 14) & 2u) | ((hi >> 21) & 4u) | ((hi >> 28) & 8u);
}

// Bit j set iff element base + j (j < kItems) is in range and flagged.  A
// whole in-range run of 16-byte aligned flags goes as 16-byte loads; the last
// run of the array, or unaligned flags, byte by byte so nothing past n is
// read.
__device__ __forceinline__ uint64_t flag_bits(const uint8_t* __restrict__ flags, int64_t base,
                                              int64_t n, bool vec) {
  uint64_t f = 0;
  if (vec && base + kItems <= n) {
    uint4 w[kLoads];
#pragma unroll
    for (int l = 0; l < kLoads; ++l) w[l] = reinterpret_cast<const uint4*>(flags + base)[l];
#pragma unroll
    for (int l = 0; l < kLoads; ++l) {
      const uint32_t b = nonzero_bytes4(w[l].x) | (nonzero_bytes4(w[l].y) << 4) |
                         (nonzero_bytes4(w[l].z) << 8) | (nonzero_bytes4(w[l].w) << 12);
      f |= static_cast<uint64_t>(b) << (16 * l);
    }
    return f;
  }
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = base + j;
    if (i < n && flags[i]) f |= uint64_t(1) << j;
  }
  return f;
}

// The low j bits (0 <= j <= 64).
__device__ __forceinline__ uint64_t low_bits(int64_t j) {
  return j >= 64 ? ~uint64_t(0) : (uint64_t(1) << j) - 1;
}

// Inclusive scan of v over one 64-lane wave.
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v) {
  const int lane = static_cast<int>(threadIdx.x) & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t u = __shfl_up(v, off, 64);
    if (lane >= off) v += u;
  }
  return v;
}

// Exclusive scan of v over the workgroup (called once by a kernel): wave
// scans, then the wave totals through LDS.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v) {
  constexpr int kWaves = kBlock / 64;
  __shared__ int32_t wave_sum[kWaves];
  const int wid = static_cast<int>(threadIdx.x) >> 6;
  const int32_t incl = wave_inclusive_scan(v);
  if ((threadIdx.x & 63) == 63) wave_sum[wid] = incl;
  __syncthreads();
  int32_t before = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) before += w < wid ? wave_sum[w] : 0;
  return before + incl - v;
}

__global__ __launch_bounds__(kBlock) void count_flags_kernel(const uint8_t* __restrict__ flags,
                                                             int64_t n, int vec,
                                                             int32_t* __restrict__ counts) {
  constexpr int kWaves = kBlock / 64;
  __shared__ int32_t sums[kWaves];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kTile + threadIdx.x * kItems;
  int32_t v = __popcll(flag_bits(flags, base, n, vec));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) all += sums[w];
    counts[blockIdx.x] = all;
  }
}

// One workgroup: before[b] = counts in tiles before b; the total goes to
// *total, which the host reads (pinned host memory) once the stream has
// passed this kernel.  Runs of kScanBlock tiles with the next run's counts
// already asked for.
constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void scan_counts_kernel(const int32_t* __restrict__ counts,
                                                                 int64_t tiles,
                                                                 int32_t* __restrict__ before,
                                                                 int32_t* __restrict__ total) {
  constexpr int kWaves = kScanBlock / 64;
  constexpr int kPer = 4;  // tiles per thread and run
  __shared__ int32_t wave_sum[kWaves];
  const int wid = static_cast<int>(threadIdx.x) >> 6;
  int32_t carry = 0;
  int32_t next[kPer];
  const auto fetch = [&](int64_t run) {
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int64_t b = run + threadIdx.x * kPer + j;
      next[j] = b < tiles ? counts[b] : 0;
    }
  };
  fetch(0);
  for (int64_t run = 0; run < tiles; run += kScanBlock * kPer) {
    int32_t c[kPer];
    int32_t v = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      c[j] = next[j];
      v += c[j];
    }
    fetch(run + kScanBlock * kPer);
    const int32_t incl = wave_inclusive_scan(v);
    if ((threadIdx.x & 63) == 63) wave_sum[wid] = incl;
    __syncthreads();
    int32_t at = carry + incl - v, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int32_t t = wave_sum[w];
      at += w < wid ? t : 0;
      all += t;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int64_t b = run + threadIdx.x * kPer + j;
      if (b < tiles) before[b] = at;
      at += c[j];
    }
    carry += all;
    __syncthreads();  // wave_sum is reused by the next run
  }
  if (threadIdx.x == 0) __hip_atomic_store(total, carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// before[b]: flagged slots in tiles before b; m: flagged in all.  A thread
// visits only the set bits of its kItems flags, and their complement in the
// tiles that reach past n_new; one workgroup scan of the flagged counts gives
// the ranks of both, because every thread before this one holds kItems
// in-range elements or the tile's last.
__global__ __launch_bounds__(kBlock) void rank_kernel(const uint8_t* __restrict__ flags, int64_t n,
                                                      int vec, int64_t n_new,
                                                      const int32_t* __restrict__ before,
                                                      int32_t* __restrict__ hole_at,
                                                      int32_t* __restrict__ mover_at,
                                                      int32_t* __restrict__ nmoves) {
  const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kTile;
  const int64_t base = tile0 + threadIdx.x * kItems;
  const uint64_t f = flag_bits(flags, base, n, vec);
  const int32_t pre_f = block_exclusive_scan(__popcll(f));
  const int32_t hole0 = before[blockIdx.x] + pre_f;  // flagged slots before this thread's
  if (base >= n) return;
  // bits of this thread's elements that lie below n_new
  const uint64_t low = base >= n_new ? 0 : low_bits(n_new - base);
  int32_t k = hole0;
  for (uint64_t h = f & low; h != 0; h &= h - 1)
    hole_at[k++] = static_cast<int32_t>(base) + __ffsll(static_cast<unsigned long long>(h)) - 1;
  // the flagged slots below n_new are those before the thread that holds
  // element n_new - 1, and its own
  if (base < n_new && n_new - base <= kItems) *nmoves = hole0 + __popcll(f & low);
  if (~low == 0) return;
  // the unflagged elements from n_new on; after element j come all elements
  // after it less the flagged ones among them, m - (flagged up to it)
  const int32_t m = static_cast<int32_t>(n - n_new);
  for (uint64_t h = ~f & ~low & low_bits(n - base); h != 0; h &= h - 1) {
    const int j = __ffsll(static_cast<unsigned long long>(h)) - 1;
    const int32_t flagged_to = hole0 + __popcll(f & low_bits(j));
    const int32_t after = static_cast<int32_t>(n - 1 - (base + j)) - (m - flagged_to);
    mover_at[after] = static_cast<int32_t>(base) + j;
  }
}

struct alignas(16) Word16 {
  uint32_t v[4];
};

template <int W>
struct WordOf;
template <>
struct WordOf<1> {
  using T = uint8_t;
};
template <>
struct WordOf<4> {
  using T = uint32_t;
};
template <>
struct WordOf<8> {
  using T = uint64_t;
};
template <>
struct WordOf<16> {
  using T = Word16;
};

// Thread k moves particle mover_at[k] to hole_at[k] in every array, kGroup
// arrays of one word size at a time: their loads, then their stores.  Holes
// lie below the new size and movers at or above it, so no thread reads what
// another writes.  Array by array (a
// row of workgroups each) the moves take the same time; this way the lists
// are read once.
constexpr int kMoveGroup = 4;

template <int W>
__device__ __forceinline__ void move_words(const MoveArgs& a, int b, int e, int64_t h, int64_t m) {
  using T = typename WordOf<W>::T;
  int y = b;
  for (; y + kMoveGroup <= e; y += kMoveGroup) {
    T v[kMoveGroup];
#pragma unroll
    for (int j = 0; j < kMoveGroup; ++j) v[j] = reinterpret_cast<const T*>(a.base[y + j])[m];
#pragma unroll
    for (int j = 0; j < kMoveGroup; ++j) reinterpret_cast<T*>(a.base[y + j])[h] = v[j];
  }
  for (; y < e; ++y) reinterpret_cast<T*>(a.base[y])[h] = reinterpret_cast<const T*>(a.base[y])[m];
}

// The AoS record, W bytes at a time.
template <int W>
__device__ __forceinline__ void move_record(char* base, int32_t stride, int64_t h, int64_t m) {
  using T = typename WordOf<W>::T;
  T* dst = reinterpret_cast<T*>(base + h * stride);
  const T* src = reinterpret_cast<const T*>(base + m * stride);
  const int words = stride / W;
  int w = 0;
  for (; w + kMoveGroup <= words; w += kMoveGroup) {
    T v[kMoveGroup];
#pragma unroll
    for (int j = 0; j < kMoveGroup; ++j) v[j] = src[w + j];
#pragma unroll
    for (int j = 0; j < kMoveGroup; ++j) dst[w + j] = v[j];
  }
  for (; w < words; ++w) dst[w] = src[w];
}

__global__ __launch_bounds__(kBlock) void move_all_kernel(MoveArgs a,
                                                          const int32_t* __restrict__ hole_at,
                                                          const int32_t* __restrict__ mover_at,
                                                          const int32_t* __restrict__ nmoves) {
  const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= *nmoves) return;
  const int64_t h = hole_at[k], m = mover_at[k];
  if (a.record) {
    switch (a.record_word) {
      case 16: move_record<16>(a.record, a.record_stride, h, m); break;
      case 8: move_record<8>(a.record, a.record_stride, h, m); break;
      case 4: move_record<4>(a.record, a.record_stride, h, m); break;
      default: move_record<1>(a.record, a.record_stride, h, m); break;
    }
  }
  move_words<8>(a, 0, a.group_end[0], h, m);
  move_words<4>(a, a.group_end[0], a.group_end[1], h, m);
  move_words<1>(a, a.group_end[1], a.group_end[2], h, m);
}

// Row y of the grid zeroes part y: single bytes up to the first 16-byte
// boundary, kZeroChunks 16-byte stores per thread for the aligned body, single
// bytes for the rest.  One launch for all parts: eight launches of 1e6
// elements each took 48 us, this takes 22 us.
constexpr int kZeroChunks = 4;

__global__ __launch_bounds__(256) void zero_kernel(ZeroArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x * kZeroChunks + threadIdx.x;
  char* p = a.base[blockIdx.y];
  const int64_t bytes = a.bytes[blockIdx.y];
  const int64_t lead = static_cast<int64_t>((16 - (reinterpret_cast<uintptr_t>(p) & 15u)) & 15u);
  const int64_t head = min(bytes, lead);
  const int64_t nbody = (bytes - head) >> 4;
  const int64_t tail0 = head + (nbody << 4);
  if (i < head) p[i] = 0;
  if (i < bytes - tail0) p[tail0 + i] = 0;
#pragma unroll
  for (int j = 0; j < kZeroChunks; ++j) {
    const int64_t c = i + j * static_cast<int64_t>(blockDim.x);
    if (c < nbody) reinterpret_cast<uint4*>(p + head)[c] = make_uint4(0u, 0u, 0u, 0u);
  }
}

}  // namespace

int64_t container_tiles(int64_t n) { return (n + kTile - 1) / kTile; }

// 16-byte loads of the flags need a 16-byte aligned array.
static int flags_vec(const uint8_t* flags) { return (reinterpret_cast<uintptr_t>(flags) & 15u) == 0; }

hipError_t launch_count_flags(const uint8_t* flags, int64_t n, int32_t* counts, int32_t* before,
                              int32_t* total, hipStream_t s) {
  const int64_t tiles = container_tiles(n);
  if (tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(count_flags_kernel, dim3(tiles), dim3(kBlock), 0, s, flags, n,
                     flags_vec(flags), counts);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(kScanBlock), 0, s, counts, tiles, before,
                     total);
  return hipGetLastError();
}

hipError_t launch_rank_flags(const uint8_t* flags, int64_t n, int64_t n_new, const int32_t* before,
                             int32_t* hole_at, int32_t* mover_at, int32_t* nmoves, hipStream_t s) {
  const int64_t grid = container_tiles(n);
  if (grid > 0)
    hipLaunchKernelGGL(rank_kernel, dim3(grid), dim3(kBlock), 0, s, flags, n, flags_vec(flags),
                       n_new, before, hole_at, mover_at, nmoves);
  return hipGetLastError();
}

hipError_t launch_move_all(const MoveArgs& m, const int32_t* hole_at, const int32_t* mover_at,
                           const int32_t* nmoves, int64_t max_moves, hipStream_t s) {
  if (max_moves <= 0) return hipSuccess;
  if (m.record) {
    const int w = m.record_word;
    if ((w != 1 && w != 4 && w != 8 && w != 16) || m.record_stride % w) return hipErrorInvalidValue;
  }
  const int64_t grid = (max_moves + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(move_all_kernel, dim3(grid), dim3(kBlock), 0, s, m, hole_at, mover_at,
                     nmoves);
  return hipGetLastError();
}

hipError_t launch_zero(const ZeroArgs& z, hipStream_t s) {
  int64_t most = 0;
  for (int y = 0; y < z.parts; ++y) most = std::max(most, z.bytes[y]);
  if (most <= 0) return hipSuccess;
  // a part has at most bytes / 16 body chunks and fewer than 16 head or tail
  // bytes, which the first workgroup's threads write
  const int64_t per_block = 256 * kZeroChunks;
  const int64_t grid = std::max<int64_t>(((most >> 4) + per_block - 1) / per_block, 1);
  hipLaunchKernelGGL(zero_kernel, dim3(grid, z.parts), dim3(256), 0, s, z);
  return hipGetLastError();
}

}  // namespace soax
