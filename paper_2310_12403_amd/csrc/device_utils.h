// Wave64 helpers for gfx950.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "coop_internal.h"

namespace coop {

constexpr int kWave = 64;
constexpr int kBlock = 256;              // 4 waves per workgroup
constexpr int kWavesPerBlock = kBlock / kWave;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_in_block() { return threadIdx.x >> 6; }
// the same value, but known to the compiler to be wave-uniform: addresses and loop bounds derived from it stay scalar
__device__ __forceinline__ int uniform_wave_in_block() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// number of set bits of `mask` strictly below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }
// the same of a plain comparison: the compare instruction's result as it is.  (Of a condition that combines several, the
// compiler spends a select and a second comparison; combine the masks instead.)
__device__ __forceinline__ uint64_t compare_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// is this lane's bit set in a wave-uniform mask?  (no instruction of its own: the mask becomes the execution mask)
__device__ __forceinline__ bool lane_in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }
// the lowest n lanes (n <= 64)
__device__ __forceinline__ uint64_t low_lanes(uint32_t n) { return n >= 64u ? ~0ull : (1ull << n) - 1ull; }
// lanes_below plus `base`, the addition being part of the two counting instructions
__device__ __forceinline__ uint32_t lanes_below_plus(uint64_t mask, uint32_t base) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
}

// wave-wide inclusive sum of a uint32 (all lanes get their prefix)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    uint32_t o = __shfl_up(v, off, kWave);
    if (lane_id() >= off) v += o;
  }
  return v;
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// One thread per block: counts the block, with `add`, in the tally; true in the block that is the last of gridDim.x, where
// *total is the sum of all blocks' `add` (below 2^32).  Each atomic is performed before the next one that depends on it is
// sent.  The words are zero again afterwards.
__device__ __forceinline__ bool tally_last(Tally* tally, uint32_t add, uint32_t* total) {
  unsigned long long* word = tally->word;
  const uint32_t line = blockIdx.x % kTallyLines;
  const uint32_t in_line = (gridDim.x - line + kTallyLines - 1) / kTallyLines;  // blocks line, line + kTallyLines, ...
  uint32_t sum = add, counts = gridDim.x;
  if (gridDim.x > (uint32_t)kTallyLines) {  // (fewer blocks count themselves in the one word)
    const unsigned long long a = atomicAdd(&word[(line + 1) * 16], ((unsigned long long)1 << 32) | add);
    if ((uint32_t)(a >> 32) != in_line - 1) return false;
    __hip_atomic_store(&word[(line + 1) * 16], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sum = (uint32_t)a + add;
    counts = kTallyLines;
  }
  const unsigned long long b = atomicAdd(&word[0], ((unsigned long long)1 << 32) | sum);
  if ((uint32_t)(b >> 32) != counts - 1) return false;
  __hip_atomic_store(&word[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *total = (uint32_t)b + sum;
  return true;
}

__device__ __forceinline__ bool tally_last(Ctl* ctl, uint32_t add, uint32_t* total) {
  return tally_last(&reinterpret_cast<DeviceCtl*>(ctl)->tally, add, total);
}

// ---- rows moved as items of up to 16 bytes --------------------------------------------------------------------------
// Feature rows have any even number of bytes (an odd number of fp16 columns, 602 fp32 columns, ...), and the tables any
// 2-byte aligned base.  A row is cut into vecs = ceil(row_bytes / VB) items of VB bytes, VB the largest power of two up to
// 16 that the row is long enough for; the last item is anchored at the row's end, so it may overlap the one before it
// (both copies of the shared bytes are the same).  Items are read and written at the alignment they have: global memory
// instructions take any.  The (row, item) pairs are dealt to the threads without gaps, so a row of 10 or 151 items leaves
// no lane idle.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int VB> struct RowVec;
template <> struct RowVec<16> { typedef u32x4 T; typedef u32x4 U __attribute__((aligned(2))); };
template <> struct RowVec<8> { typedef u32x2 T; typedef u32x2 U __attribute__((aligned(2))); };
template <> struct RowVec<4> { typedef uint32_t T; typedef uint32_t U __attribute__((aligned(2))); };
template <> struct RowVec<2> { typedef uint16_t T; typedef uint16_t U; };

template <int VB>
__device__ __forceinline__ typename RowVec<VB>::T row_load_nt(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const typename RowVec<VB>::U*>(p));
}
template <int VB>
__device__ __forceinline__ void row_store_nt(char* p, typename RowVec<VB>::T x) {
  __builtin_nontemporal_store(x, reinterpret_cast<typename RowVec<VB>::U*>(p));
}

struct RowShape {
  int64_t row_bytes;
  uint32_t vecs;   // items per row
  uint32_t magic;  // ceil(2^32 / vecs)
  int vec_bytes;
};
inline RowShape row_shape(int64_t row_bytes) {
  const int vb = row_bytes >= 16 ? 16 : row_bytes >= 8 ? 8 : row_bytes >= 4 ? 4 : 2;
  const uint32_t vecs = (uint32_t)((row_bytes + vb - 1) / vb);
  return RowShape{row_bytes, vecs, (uint32_t)((((uint64_t)1 << 32) + vecs - 1) / vecs), vb};
}

// A launch has fewer than 2^32 threads (one that asks for more runs with what is left of the number modulo 2^32, without an
// error), which is 64 GB of rows at an item per thread: kernels of that kind are launched in slices of blocks.
constexpr int64_t kSliceBlocks = ((int64_t)1 << 32) / kBlock - 1;

// The items [first, first + count) of a block, count <= 1024: thread items are given as offsets below count.
struct BlockItems {
  int64_t row0;  // row of the block's first item
  uint32_t rem;  // ... and that item's number in the row
  __device__ __forceinline__ BlockItems(int64_t first, uint32_t vecs) : row0(first / vecs), rem((uint32_t)(first - row0 * vecs)) {}
  // (the multiplication is exact for vecs < 1024: the dividend stays below 2048 and the excess of magic * vecs over 2^32
  // below vecs)
  __device__ __forceinline__ int64_t row_of(uint32_t at, const RowShape& sh, uint32_t* item) const {
    const uint32_t i = rem + at;
    const uint32_t q = sh.vecs >= 1024u ? (i >= sh.vecs ? 1u : 0u) : sh.vecs == 1u ? i : __umulhi(i, sh.magic);
    *item = i - q * sh.vecs;
    return row0 + q;
  }
  template <int VB>
  static __device__ __forceinline__ int64_t byte_of(uint32_t item, const RowShape& sh) {
    const int64_t o = (int64_t)item * VB, last = sh.row_bytes - VB;
    return o < last ? o : last;
  }
};

}  // namespace coop
