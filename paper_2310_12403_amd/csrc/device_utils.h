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

// A source's tag: the highest byte of the hash by which the dedup of a short list deals the vertices to buckets (unique.hip).
constexpr uint32_t kSourceHash = 0x9E3779B9u;
__device__ __forceinline__ uint32_t source_tag(uint32_t key) { return key * kSourceHash >> 24; }

// wave-wide inclusive sum of a uint32 (all lanes get their prefix)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    uint32_t o = __shfl_up(v, off, kWave);
    if (lane_id() >= off) v += o;
  }
  return v;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
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

// inclusive scan over the block of one int64 per thread, WAVES waves; *total = the block's sum
template <int WAVES>
__device__ __forceinline__ int64_t block_incl_scan_i64(int64_t v, int64_t* total, int64_t* lds /* [WAVES] */) {
  const int lane = lane_id(), w = wave_in_block();
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int64_t o = __shfl_up(v, off, kWave);
    if (lane >= off) v += o;
  }
  if (lane == kWave - 1) lds[w] = v;
  __syncthreads();
  int64_t base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    const int64_t x = lds[i];
    if (i < w) base += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return v + base;
}

// what a one-thread publishing kernel would do, done by a thread that has just stored what the host waits for
__device__ __forceinline__ void publish_ctl(const Publish& pub) {
  if (pub.h == nullptr) return;
  send_ctl(pub.h, pub.ticket, *pub.d_ctl);
}

// Tile by tile: out holds, for the first element of every tile of 2^log2 elements, the tile's sum (stored by tile_sum_done), and
// the last block turns these sums into offsets.  The whole block calls it.
template <int WAVES>
__device__ __forceinline__ int64_t scan_tile_sums(int64_t n, int log2, int64_t* out, int64_t* lds) {
  const int64_t tiles = (n + ((int64_t)1 << log2) - 1) >> log2;
  int64_t carry = 0;
  for (int64_t first = 0; first < tiles; first += WAVES * kWave) {
    const int64_t t = first + threadIdx.x;
    const int64_t v = t < tiles ? __hip_atomic_load(&out[t << log2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    int64_t all;
    const int64_t upto = block_incl_scan_i64<WAVES>(v, &all, lds);
    if (t < tiles) out[t << log2] = carry + upto - v;
    carry += all;
  }
  return carry;
}
// One thread per block: leaves the tile's sum where its first element's offset belongs; true in the block that is last.
// No fence stands between the sum and the count: an atomic that returns a value has been performed in memory when the value is
// here (the asm waits for it), and the count is sent behind that; the reader of the sums (scan_tile_sums, k_scan_tiled) uses
// agent-scope loads, which pass the caches that are not shared.  That is how gfx950 carries these instructions out, not a promise
// of the language's memory model for relaxed accesses.
__device__ __forceinline__ bool tile_sum_done(int64_t sum, int64_t* first, Ctl* ctl) {
  // the exchange has been performed when its result is here; the block counts itself behind it
  const unsigned long long old = atomicExch(reinterpret_cast<unsigned long long*>(first), (unsigned long long)sum);
  asm volatile("" : : "v"(old) : "memory");
  uint32_t unused;
  return tally_last(ctl, 0u, &unused);
}

// Where a destination's entries go, found by the kernel that puts them there: 1 << LOG2 neighbouring lanes for a destination,
// blocks of BLOCK threads, destinations dealt to the blocks in order from `first` on.  OWN: from the counts alone, every block adding
// up those in front of it (at most kScanOwn: 128 KB out of L2); 16 thousand 3 us more in this kernel in the place of two launches of
// 5.  Else what scan_in_tiles left, every wave adding up the tiles in front of its own, or, where those are many, what scan_tiles
// left.  Either way the offsets leave in indptr.
// Where element i of counts in pieces lies.  The pieces' addresses are chosen among, not looked up by the piece's number: an argument
// indexed by a lane's number is read from memory by the lane, a wait ahead of the load that needs it.
__device__ __forceinline__ const int32_t* chunk_at(const ChunkedI32& c, int64_t i) {
  const int32_t* from = c.ptr[0] - c.start[0];
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (q < c.n_chunks && i >= c.start[q]) from = c.ptr[q] - c.start[q];
  return from + i;
}
struct CountOffsets {
  ChunkedI32 cnt;
  int64_t* indptr;
  int64_t* total_out;
  const int64_t* sums;  // the tiles' sums, when they have not been turned into offsets (scan_in_tiles)
};
template <bool OWN, int BLOCK, int LOG2>
__device__ __forceinline__ int64_t offset_of(const CountOffsets& co, int64_t w, int64_t n_dst, int32_t* count) {
  const bool live = w < n_dst, speaks = live && (threadIdx.x & ((1 << LOG2) - 1)) == 0;
  *count = live ? *chunk_at(co.cnt, w) : 0;
  if constexpr (OWN) {
    constexpr int kWaves = BLOCK / kWave;
    __shared__ int64_t lds[2 * kWaves];
    const int64_t w0 = (int64_t)blockIdx.x * (BLOCK >> LOG2);
    int64_t part = 0;
    for (int q = 0; q < co.cnt.n_chunks; ++q) {
      const int64_t hi = q + 1 < co.cnt.n_chunks && co.cnt.start[q + 1] < w0 ? co.cnt.start[q + 1] : w0;
#pragma unroll 4
      for (int64_t i = co.cnt.start[q] + threadIdx.x; i < hi; i += BLOCK) part += co.cnt.ptr[q][i - co.cnt.start[q]];
    }
    part = wave_sum_i64(part);
    const int64_t mine = speaks ? *count : 0;
    int64_t upto = mine;
#pragma unroll
    for (int off = 1 << LOG2; off < kWave; off <<= 1) {
      const int64_t o = __shfl_up(upto, off, kWave);
      if (lane_id() >= off) upto += o;
    }
    if (lane_id() == 0) lds[wave_in_block()] = part;
    if (lane_id() == kWave - (1 << LOG2)) lds[kWaves + wave_in_block()] = upto;
    __syncthreads();
    int64_t o = __shfl(upto - mine, lane_id() & ~((1 << LOG2) - 1), kWave);
#pragma unroll
    for (int q = 0; q < kWaves; ++q) o += lds[q] + (q < wave_in_block() ? lds[kWaves + q] : 0);
    if (speaks) {
      co.indptr[w] = o;
      if (w == n_dst - 1) {
        co.indptr[n_dst] = o + *count;
        *co.total_out = o + *count;
      }
    }
    return o;
  } else {
    const int64_t tile = w >> kOffsetTileLog2 << kOffsetTileLog2;
    if (co.sums != nullptr) {
      const int64_t in_tile = live && w != tile ? co.indptr[w] : 0;
      // (a wave's destinations are neighbours of one tile)
      const int in_front = __builtin_amdgcn_readfirstlane((int)(w >> kOffsetTileLog2));
      int64_t part = 0;
#pragma unroll
      for (int q = 0; q < (int)kTilesAhead / kWave; ++q) {
        const int t = q * kWave + lane_id();
        if (t < in_front) part += co.sums[t];
      }
      const int64_t o = wave_sum_i64(part) + in_tile;
      if (speaks) {
        co.indptr[w] = o;
        if (w == n_dst - 1) {
          co.indptr[n_dst] = o + *count;
          *co.total_out = o + *count;
        }
      }
      return o;
    }
    if (!live) return 0;
    int64_t o = co.indptr[tile];
    if (w != tile) {
      o += co.indptr[w];  // (read by this group of lanes only, all of one wave, and overwritten behind that)
      if (speaks) co.indptr[w] = o;
    }
    return o;
  }
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
