// libcoop runtime pieces: error names, arena allocator, profiling table, graph handle, fill and scan kernels.
#include <mutex>
#include <new>
#include <vector>

#include "coop_internal.h"
#include "device_utils.h"

namespace coop {

// ---- profiling ------------------------------------------------------------------------------------------------
namespace {
struct Pending { int id; hipEvent_t a, b; };
struct Prof {
  std::mutex mu;
  bool on = false;
  int only = -1;  // when >= 0, the one kernel id that is timed
  double ms[K_COUNT_] = {};
  int64_t launches[K_COUNT_] = {};
  std::vector<Pending> pending;
  std::vector<hipEvent_t> pool;
  hipEvent_t open[K_COUNT_] = {};
} g_prof;

const char* const kKernelNames[K_COUNT_] = {
    "fill", "labor_scan", "labor_fill", "labor_fill_overflow", "labor_exact", "segments", "enum_list", "enum_walk", "ns_count", "ns_fill", "ns_select", "rw_walk", "rw_fill", "scan_local", "scan_offset",
    "unique_insert", "unique_flag", "unique_filter", "unique_collect", "unique_relabel", "unique_part_count", "unique_part_scatter", "unique_part_first", "copy_ids", "gather", "gather_mean", "owner_count", "owner_scatter", "validate_csr",
    "cache_lookup", "cache_select", "cache_evict", "cache_miss_rows", "cache_hit_rows"};

hipEvent_t take_event() {
  if (!g_prof.pool.empty()) { hipEvent_t e = g_prof.pool.back(); g_prof.pool.pop_back(); return e; }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// folds finished event pairs into the table; caller holds the lock
void collect_locked() {
  for (auto& p : g_prof.pending) {
    float ms = 0.f;
    if (hipEventSynchronize(p.b) == hipSuccess && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      g_prof.ms[p.id] += ms;
      g_prof.launches[p.id] += 1;
    }
    g_prof.pool.push_back(p.a);
    g_prof.pool.push_back(p.b);
  }
  g_prof.pending.clear();
}
}  // namespace

void prof_begin(int id, hipStream_t s) {
  if (!g_prof.on || (g_prof.only >= 0 && g_prof.only != id)) return;
  std::lock_guard<std::mutex> lk(g_prof.mu);
  hipEvent_t a = take_event();
  if (!a) return;
  (void)hipEventRecord(a, s);
  g_prof.open[id] = a;
}

void prof_end(int id, hipStream_t s) {
  if (!g_prof.on || (g_prof.only >= 0 && g_prof.only != id)) return;
  std::lock_guard<std::mutex> lk(g_prof.mu);
  hipEvent_t a = g_prof.open[id];
  if (!a) return;
  g_prof.open[id] = nullptr;
  hipEvent_t b = take_event();
  if (!b) { g_prof.pool.push_back(a); return; }
  (void)hipEventRecord(b, s);
  g_prof.pending.push_back({id, a, b});
  if (g_prof.pending.size() >= 4096) collect_locked();
}

// ---- fill -----------------------------------------------------------------------------------------------------
typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(kBlock) void k_fill_u64(uint64_t* __restrict__ p, int64_t n, uint64_t v) {
  // 16-byte stores over the even part when the base allows it, single words for the rest
  const bool wide = ((uintptr_t)p & 15) == 0;
  const int64_t n2 = wide ? n / 2 : 0;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  const u64x2 vv = {v, v};
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n2; i += stride) reinterpret_cast<u64x2*>(p)[i] = vv;
  for (int64_t i = 2 * n2 + (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) p[i] = v;
}

void fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s) {
  if (n <= 0) return;
  int64_t blocks = (n / 2 + kBlock - 1) / kBlock;
  if (blocks > 256 * 64) blocks = 256 * 64;
  if (blocks < 1) blocks = 1;
  COOP_LAUNCH(K_FILL, k_fill_u64, dim3((unsigned)blocks), dim3(kBlock), 0, s, p, n, v);
}

// ---- device-wide exclusive scan -------------------------------------------------------------------------------
// Two kernels, no inter-block waiting: (1) every block scans its own tile of kTile consecutive elements and records
// the tile's sum; (2) every block adds up the sums of the tiles in front of it (a few thousand words at most, read
// from L2) and shifts its tile by that offset; the last block also publishes the grand total.
constexpr int kItems = 8;
constexpr int kTile = kBlock * kItems;  // 2048
static_assert(kTile == (1 << kScanTileLog2), "TiledScan::at() finds an element's tile by a shift");

__device__ __forceinline__ int64_t block_incl_scan(int64_t v, int64_t* total, int64_t* lds /* [kWavesPerBlock] */) {
  return block_incl_scan_i64<kWavesPerBlock>(v, total, lds);
}

// (A thread's kItems elements lie side by side: where all of them are there they are loaded and stored 16 bytes at a time (the arrays
// have the alignment of their elements, which is what global memory instructions ask for).  Element by element, with a test for each,
// the scans of the dedup's counters took 6.4 and 8.5 us for 290 and 590 thousand of them, 4.8 and 5.8 so.)
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned long long u64x2_any __attribute__((ext_vector_type(2), aligned(8)));
struct LoadU32 {
  const uint32_t* in;
  __device__ __forceinline__ int64_t operator()(int64_t i) const { return in[i]; }
  __device__ __forceinline__ void all(int64_t i, int64_t (&x)[kItems]) const {
#pragma unroll
    for (int j = 0; j < kItems; j += 4) {
      const u32x4_any v = *reinterpret_cast<const u32x4_any*>(in + i + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[j + e] = v[e];
    }
  }
};
struct LoadPopc {  // element i = number of set bits of word i
  const uint64_t* bits;
  __device__ __forceinline__ int64_t operator()(int64_t i) const { return __popcll(bits[i]); }
  __device__ __forceinline__ void all(int64_t i, int64_t (&x)[kItems]) const {
#pragma unroll
    for (int j = 0; j < kItems; j += 2) {
      const u64x2_any v = *reinterpret_cast<const u64x2_any*>(bits + i + j);
      x[j] = __popcll(v[0]);
      x[j + 1] = __popcll(v[1]);
    }
  }
};
// elements base .. base + kItems - 1, those beyond n as 0; returns their sum
template <typename Load>
__device__ __forceinline__ int64_t load_items(const Load& load, int64_t base, int64_t n, int64_t (&x)[kItems]) {
  if (base + kItems <= n) {
    load.all(base, x);
  } else {
#pragma unroll
    for (int j = 0; j < kItems; ++j) x[j] = base + j < n ? load(base + j) : 0;
  }
  int64_t sum = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) sum += x[j];
  return sum;
}
// out[base + j] = run + the elements in front of j
__device__ __forceinline__ void store_items(uint32_t* __restrict__ out, int64_t base, int64_t n, const int64_t (&x)[kItems], int64_t run) {
  uint32_t y[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    y[j] = (uint32_t)run;
    run += x[j];
  }
  if (base + kItems <= n) {
#pragma unroll
    for (int j = 0; j < kItems; j += 4) *reinterpret_cast<u32x4_any*>(out + base + j) = u32x4_any{y[j], y[j + 1], y[j + 2], y[j + 3]};
  } else {
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (base + j < n) out[base + j] = y[j];
  }
}

template <typename Load, typename Out>
__global__ __launch_bounds__(kBlock) void k_scan_local(Load load, int64_t n, Out* __restrict__ out, int64_t* __restrict__ tile_sum) {
  __shared__ int64_t lds[kWavesPerBlock];
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;  // a thread owns 8 in a row
  int64_t x[kItems];
  const int64_t sum = load_items(load, base, n, x);
  int64_t tot;
  const int64_t incl = block_incl_scan(sum, &tot, lds);
  store_items(out, base, n, x, incl - sum);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

template <typename Out>
__global__ __launch_bounds__(kBlock) void k_scan_offset(int64_t n, Out* __restrict__ out, const int64_t* __restrict__ tile_sum,
                                                        Out* __restrict__ end_out, int64_t* total_out) {
  __shared__ int64_t lds[kWavesPerBlock];
  int64_t part = 0;
  for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kBlock) part += tile_sum[t];
  part = wave_sum_i64(part);
  if (lane_id() == 0) lds[wave_in_block()] = part;
  __syncthreads();
  int64_t off = 0;
#pragma unroll
  for (int i = 0; i < kWavesPerBlock; ++i) off += lds[i];
  const int64_t base = (int64_t)blockIdx.x * kTile;
  if (off != 0) {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = base + (int64_t)j * kBlock + threadIdx.x;
      if (i < n) out[i] = (Out)((int64_t)out[i] + off);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    const int64_t total = off + tile_sum[blockIdx.x];
    if (end_out) *end_out = (Out)total;  // the entry one past the end holds the grand total
    if (total_out) *total_out = total;
  }
}

// The same per-tile scan, and the scan of the tile sums by whichever block finishes last: one launch.  The consumer adds
// tile_prefix[tile] to an element when it reads it (TiledScan::at).  A tile's sum is exchanged into its place and the block counts
// itself behind that (tally_last), without a fence: 590 thousand counters 5.8 us.
__global__ __launch_bounds__(kBlock) void k_scan_tiled(LoadU32 load, int64_t n, uint32_t* __restrict__ out, int64_t* __restrict__ tile_sum,
                                                       uint32_t* __restrict__ tile_prefix, Ctl* ctl) {
  __shared__ int64_t lds[kWavesPerBlock];
  __shared__ uint32_t s_last;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;  // a thread owns 8 in a row
  int64_t x[kItems];
  const int64_t sum = load_items(load, base, n, x);
  int64_t tot;
  const int64_t incl = block_incl_scan(sum, &tot, lds);
  store_items(out, base, n, x, incl - sum);
  if (threadIdx.x == 0) {
    s_last = tile_sum_done(tot, tile_sum + blockIdx.x, ctl) ? 1u : 0u;
  }
  __syncthreads();
  if (s_last == 0) return;
  const int64_t tiles = gridDim.x;
  int64_t carry = 0;
  for (int64_t first = 0; first < tiles; first += kBlock) {
    const int64_t t = first + threadIdx.x;
    const int64_t v = t < tiles ? __hip_atomic_load(&tile_sum[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    int64_t all;
    const int64_t upto = block_incl_scan(v, &all, lds);
    if (t < tiles) tile_prefix[t] = (uint32_t)(carry + upto - v);
    carry += all;
  }
  if (threadIdx.x == 0) out[n] = (uint32_t)carry;  // the entry one past the end holds the grand total
}

// Short inputs: one block walks over the tiles with a running carry (one launch instead of two).
constexpr int64_t kScanSmall = 2 * kTile;  // 4096 elements (beyond that two parallel launches are quicker)
template <typename Load, typename Out>
__global__ __launch_bounds__(kBlock) void k_scan_small(Load load, int64_t n, Out* __restrict__ out, Out* __restrict__ end_out,
                                                       int64_t* total_out) {
  __shared__ int64_t lds[kWavesPerBlock];
  int64_t carry = 0;
  for (int64_t tile = 0; tile < n; tile += kTile) {
    const int64_t base = tile + (int64_t)threadIdx.x * kItems;
    int64_t x[kItems];
    const int64_t sum = load_items(load, base, n, x);
    int64_t tot;
    const int64_t incl = block_incl_scan(sum, &tot, lds);
    store_items(out, base, n, x, carry + incl - sum);
    carry += tot;
  }
  if (threadIdx.x == 0) {
    if (end_out) *end_out = (Out)carry;
    if (total_out) *total_out = carry;
  }
}

size_t scan_tmp_bytes(int64_t n) {  // tile sums, and the one-kernel scans' tile prefixes
  const int64_t tiles = (n + kTile - 1) / kTile;
  return (size_t)(tiles + 2) * sizeof(int64_t) * 2;
}

constexpr int64_t kScanTiledMax = 1024;  // tiles (2,097,152 elements) up to which the one-kernel scan is used (four rounds of the last block)
template <typename Load, typename Out>
static void scan_impl(Load load, int64_t n, Out* out, Out* end_out, int64_t* total_out, void* tmp, hipStream_t s) {
  if (n <= kScanSmall) {
    COOP_LAUNCH(K_SCAN_LOCAL, (k_scan_small<Load, Out>), dim3(1), dim3(kBlock), 0, s, load, n, out, end_out, total_out);
    return;
  }
  int64_t* tile_sum = (int64_t*)tmp;
  const int64_t tiles = (n + kTile - 1) / kTile;
  COOP_LAUNCH(K_SCAN_LOCAL, (k_scan_local<Load, Out>), dim3((unsigned)tiles), dim3(kBlock), 0, s, load, n, out, tile_sum);
  COOP_LAUNCH(K_SCAN_OFFSET, k_scan_offset<Out>, dim3((unsigned)tiles), dim3(kBlock), 0, s, n, out, tile_sum, end_out, total_out);
}

// counts to offsets, one launch (see CountOffsets); where one tile holds them, by a block that has nobody to wait for (30 counts: 6.6 us
// as a tile of several, 3.9 so)
constexpr int kTilesBlock = 1024, kTilesItems = 4;
static_assert(kTilesBlock * kTilesItems == 1 << kOffsetTileLog2, "a block takes a tile");
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_scan_tiles(ChunkedI32 in, int64_t n, int64_t* __restrict__ out, int64_t* total_out, Ctl* ctl, Publish pub,
                                                      int64_t* __restrict__ sums /* or null: scan_in_tiles */) {
  __shared__ int64_t lds[BLOCK / kWave];
  __shared__ uint32_t s_last;
  const int64_t tile = (int64_t)blockIdx.x << kOffsetTileLog2, base = tile + (int64_t)threadIdx.x * kTilesItems;  // a thread owns 4 in a row
  static_assert(kTilesItems == 4, "one load");
  typedef int i32x4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef long long i64x2 __attribute__((ext_vector_type(2)));
  int64_t x[kTilesItems], sum = 0;
  const int32_t* from = chunk_at(in, base);
  const bool whole = base + kTilesItems <= n;
  if (whole && chunk_at(in, base + kTilesItems - 1) == from + kTilesItems - 1) {  // (nearly every thread)
    const i32x4 v = *reinterpret_cast<const i32x4*>(from);
#pragma unroll
    for (int j = 0; j < kTilesItems; ++j) sum += x[j] = v[j];
  } else {
#pragma unroll
    for (int j = 0; j < kTilesItems; ++j) sum += x[j] = base + j < n ? *chunk_at(in, base + j) : 0;
  }
  int64_t tot;
  int64_t run = block_incl_scan_i64<BLOCK / kWave>(sum, &tot, lds) - sum;
  if (whole && (base != tile || gridDim.x == 1)) {
    i64x2* to = reinterpret_cast<i64x2*>(out + base);
    to[0] = i64x2{run, run + x[0]};
    to[1] = i64x2{run + x[0] + x[1], run + x[0] + x[1] + x[2]};
  } else {
#pragma unroll
    for (int j = 0; j < kTilesItems; ++j) {
      const int64_t i = base + j;
      if (i < n && (i != tile || gridDim.x == 1)) out[i] = run;
      run += x[j];
    }
  }
  if (sums != nullptr) {
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
    return;
  }
  if (gridDim.x == 1) {
    if (threadIdx.x == 0) {
      out[n] = tot;
      *total_out = tot;
      publish_ctl(pub);
    }
    return;
  }
  if (threadIdx.x == 0) s_last = tile_sum_done(tot, out + tile, ctl) ? 1u : 0u;
  __syncthreads();
  if (s_last == 0) return;
  const int64_t total = scan_tile_sums<BLOCK / kWave>(n, kOffsetTileLog2, out, lds);
  if (threadIdx.x == 0) {
    out[n] = total;
    *total_out = total;
    publish_ctl(pub);
  }
}

__global__ void k_store_total(int64_t* p, int64_t* total_out, Publish pub) {
  *p = 0;
  *total_out = 0;
  publish_ctl(pub);
}

void scan_tiles(const ChunkedI32& in, int64_t n, int64_t* out, int64_t* total_out, Ctl* ctl, hipStream_t s, const Publish* pub) {
  const Publish p = pub ? *pub : Publish{};
  if (n <= 0)  // out[0] = 0
    COOP_LAUNCH(K_FILL, k_store_total, dim3(1), dim3(1), 0, s, out, total_out, p);
  else if (n <= kBlock * kTilesItems)
    COOP_LAUNCH(K_SCAN_LOCAL, k_scan_tiles<kBlock>, dim3(1), dim3(kBlock), 0, s, in, n, out, total_out, ctl, p, (int64_t*)nullptr);
  else
    COOP_LAUNCH(K_SCAN_LOCAL, k_scan_tiles<kTilesBlock>, dim3((unsigned)((n + (1 << kOffsetTileLog2) - 1) >> kOffsetTileLog2)), dim3(kTilesBlock), 0, s, in, n, out,
                total_out, ctl, p, (int64_t*)nullptr);
}

void scan_in_tiles(const ChunkedI32& in, int64_t n, int64_t* out, int64_t* sums, hipStream_t s) {
  COOP_LAUNCH(K_SCAN_LOCAL, k_scan_tiles<kTilesBlock>, dim3((unsigned)((n + (1 << kOffsetTileLog2) - 1) >> kOffsetTileLog2)), dim3(kTilesBlock), 0, s, in, n, out,
              (int64_t*)nullptr, (Ctl*)nullptr, Publish{}, sums);
}

void scan_u32_to_u32(const uint32_t* in, int64_t n, uint32_t* out, void* tmp, hipStream_t s) {
  scan_impl<LoadU32, uint32_t>(LoadU32{in}, n, out, out + n, nullptr, tmp, s);
}

TiledScan<uint32_t> scan_u32_tiled(const uint32_t* in, int64_t n, uint32_t* out, void* tmp, Ctl* ctl, hipStream_t s) {
  const int64_t tiles = (n + kTile - 1) / kTile;
  if (n <= kScanSmall || tiles > kScanTiledMax) {  // one block, or two kernels
    scan_u32_to_u32(in, n, out, tmp, s);
    return TiledScan<uint32_t>{out, nullptr, n};
  }
  int64_t* tile_sum = (int64_t*)tmp;
  uint32_t* tile_prefix = (uint32_t*)(tile_sum + tiles + 2);
  COOP_LAUNCH(K_SCAN_LOCAL, k_scan_tiled, dim3((unsigned)tiles), dim3(kBlock), 0, s, LoadU32{in}, n, out, tile_sum, tile_prefix, ctl);
  return TiledScan<uint32_t>{out, tile_prefix, n};
}

void scan_popc_to_u32(const uint64_t* bits, int64_t n_words, uint32_t* out, int64_t* total_out, void* tmp, hipStream_t s) {
  scan_impl<LoadPopc, uint32_t>(LoadPopc{bits}, n_words, out, (uint32_t*)nullptr, total_out, tmp, s);
}

// ---- CSR validation -------------------------------------------------------------------------------------------
// Also a census of the degrees: census[k] = number of vertices whose list has 2^k entries or more but fewer than 2^(k+1)
// (k = 0..31; lists of 2^31 entries and more in the last counter).  The samplers size the part of a grid that is set
// aside for long lists from it.
__global__ __launch_bounds__(kBlock) void k_validate_csr(const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                         int64_t nv, int64_t ne, int32_t* __restrict__ bad,
                                                         unsigned long long* __restrict__ census) {
  __shared__ uint32_t tally[32];
  if (threadIdx.x < 32) tally[threadIdx.x] = 0;
  __syncthreads();
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  bool b = false;
  for (int64_t v = i; v < nv; v += stride) {
    const int64_t d = indptr[v + 1] - indptr[v];
    b |= d < 0;
    if (d > 0) {
      const int k = 63 - __builtin_clzll((unsigned long long)d);
      atomicAdd(&tally[k < 31 ? k : 31], 1u);
    }
  }
  for (int64_t e = i; e < ne; e += stride) b |= (uint32_t)indices[e] >= (uint64_t)nv;
  if (i == 0) b |= indptr[0] != 0 || indptr[nv] != ne;
  if (b) atomicOr(bad, 1);
  __syncthreads();
  if (threadIdx.x < 32 && tally[threadIdx.x] != 0) atomicAdd(&census[threadIdx.x], (unsigned long long)tally[threadIdx.x]);
}

// COOP_SYMMETRIC: checks that the lists are strictly ascending and that every edge t in N(s) has its reverse s in N(t),
// and records where: rev[e] = position of s in t's list, for the edge at position e of the indices array (bisection).
// Also adds up the entries of the lists longer than kLongListDegree: LABOR-0 works from the neighbours' side only on
// graphs where such lists hold a good part of the edges.
__global__ __launch_bounds__(kBlock) void k_build_reverse(const int64_t* __restrict__ indptr, const int32_t* __restrict__ indices,
                                                          int64_t nv, uint32_t* __restrict__ rev, int32_t* bad,
                                                          unsigned long long* long_mass) {
  // one wave per vertex at a time, lanes over its list
  if (*bad != 0) return;  // (a malformed CSR was reported by the kernel before this one: its offsets cannot be trusted)
  const int64_t n_waves = ((int64_t)gridDim.x * kBlock) >> 6;
  bool b = false;
  for (int64_t s = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6; s < nv; s += n_waves) {
    const int64_t beg = indptr[s], end = indptr[s + 1];
    if (lane_id() == 0 && end - beg > kLongListDegree) atomicAdd(long_mass, (unsigned long long)(end - beg));
    for (int64_t e = beg + lane_id(); e < end; e += kWave) {
      const int32_t t = indices[e];
      if (e > beg && indices[e - 1] >= t) b = true;
      const int64_t tb = indptr[t];
      const int64_t td = indptr[t + 1] - tb;
      int64_t lo = 0, hi = td;
      while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (indices[tb + mid] < (int32_t)s) lo = mid + 1; else hi = mid;
      }
      if (lo >= td || indices[tb + lo] != (int32_t)s) { b = true; lo = 0; }
      rev[e] = (uint32_t)lo;
    }
  }
  if (b) atomicOr(bad, 1);
}

}  // namespace coop

using namespace coop;

extern "C" {

const char* coop_strerror(int code) {
  switch (code) {
    case COOP_OK: return "ok";
    case COOP_E_NULL: return "null pointer argument";
    case COOP_E_RANGE: return "vertex id out of range";
    case COOP_E_DUPSEED: return "duplicate seed vertex";
    case COOP_E_ARG: return "invalid argument";
    case COOP_E_NOMEM: return "allocator returned no memory";
    case COOP_E_CAPACITY: return "workspace capacity exceeded";
    case COOP_E_HIP: return "HIP runtime error";
    case COOP_E_GRAPH: return "malformed CSR graph";
    default: return "unknown error";
  }
}

int coop_version(void) { return 2; }

void* coop_arena_alloc(void* arena, size_t bytes, int tag) {
  (void)tag;
  coop_arena* a = (coop_arena*)arena;
  if (!a || !a->base) return nullptr;
  const size_t need = (bytes + 255) & ~(size_t)255;
  if (a->used + need > a->bytes) return nullptr;
  void* p = (char*)a->base + a->used;
  a->used += need;
  return p;
}

void* coop_chunk_alloc(void* chunks, size_t bytes, int tag) {
  coop_chunks* c = (coop_chunks*)chunks;
  if (!c || !c->from) return nullptr;
  const size_t need = (bytes + 255) & ~(size_t)255;
  if (tag != COOP_TAG_SCRATCH || need < bytes || need > c->chunk_bytes / 4) return c->from(c->ctx, bytes, tag);
  if (need > c->left) {
    void* p = c->from(c->ctx, c->chunk_bytes, tag);
    if (!p) return c->from(c->ctx, bytes, tag);
    c->at = p;
    c->left = c->chunk_bytes;
  }
  void* p = c->at;
  c->at = (char*)p + need;
  c->left -= need;
  return p;
}

int coop_graph_load_with(const int64_t* indptr, const int32_t* indices, int64_t n_vertices, int64_t n_edges, int flags,
                         coop_alloc_fn alloc, void* alloc_ctx, void* stream, coop_graph** out) {
  if (!out) return COOP_E_NULL;
  *out = nullptr;
  if (!indptr || (!indices && n_edges > 0)) return COOP_E_NULL;
  if (n_vertices < 0 || n_vertices >= ((int64_t)1 << 31) || n_edges < 0 || (flags & ~(COOP_VALIDATE | COOP_SYMMETRIC))) return COOP_E_ARG;
  uint32_t* rev = nullptr;
  bool own_rev = false;  // the reverse index came from hipMalloc (no allocator given): coop_graph_free releases it
  int64_t long_mass = 0;
  bool have_census = false;
  int64_t census[32] = {};
  if (flags & (COOP_VALIDATE | COOP_SYMMETRIC)) {  // (the reverse index is built from offsets and ids that have been checked)
    hipStream_t s = (hipStream_t)stream;
    struct Check { int32_t bad, pad; unsigned long long long_mass; unsigned long long census[32]; };
    Check* d_chk = nullptr;
    if (alloc) {
      d_chk = (Check*)alloc(alloc_ctx, (sizeof(Check) + 255) & ~(size_t)255, COOP_TAG_SCRATCH);
      if (!d_chk) return COOP_E_NOMEM;
      if ((flags & COOP_SYMMETRIC) && n_edges > 0) {
        rev = (uint32_t*)alloc(alloc_ctx, (((size_t)n_edges * sizeof(uint32_t)) + 255) & ~(size_t)255, COOP_TAG_GRAPH);
        if (!rev) return COOP_E_NOMEM;
      }
    } else {
      COOP_HIP_TRY(hipMalloc((void**)&d_chk, sizeof(Check)));
      if ((flags & COOP_SYMMETRIC) && n_edges > 0) {
        if (hipMalloc((void**)&rev, (size_t)n_edges * sizeof(uint32_t)) != hipSuccess) {
          (void)hipFree(d_chk);
          return COOP_E_NOMEM;
        }
        own_rev = true;
      }
    }
    Check h_chk{};
    hipError_t e = hipMemcpyAsync(d_chk, &h_chk, sizeof(Check), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
      COOP_LAUNCH(K_VALIDATE, k_validate_csr, dim3(256 * 16), dim3(kBlock), 0, s, indptr, indices, n_vertices, n_edges, &d_chk->bad,
                  d_chk->census);
      if ((flags & COOP_SYMMETRIC) && n_vertices > 0 && n_edges > 0) {
        // (a grid holds fewer than 2^32 threads: the waves stride over the vertices)
        const int64_t want = (n_vertices * kWave + kBlock - 1) / kBlock;
        COOP_LAUNCH(K_VALIDATE, k_build_reverse, dim3((unsigned)(want < (1 << 22) ? want : (1 << 22))), dim3(kBlock), 0, s, indptr, indices,
                    n_vertices, rev, &d_chk->bad, &d_chk->long_mass);
      }
      e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(&h_chk, d_chk, sizeof(Check), hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (!alloc) (void)hipFree(d_chk);
    if (e != hipSuccess || h_chk.bad) {
      if (own_rev) (void)hipFree(rev);
      return e != hipSuccess ? COOP_E_HIP : COOP_E_GRAPH;
    }
    long_mass = (int64_t)h_chk.long_mass;
    have_census = true;
    for (int k = 0; k < 32; ++k) census[k] = (int64_t)h_chk.census[k];
  }
  coop_graph* g = new (std::nothrow) coop_graph{indptr, indices, n_vertices, n_edges, (flags & COOP_SYMMETRIC) != 0 && n_edges > 0, rev, long_mass, own_rev};
  if (!g) {
    if (own_rev) (void)hipFree(rev);
    return COOP_E_NOMEM;
  }
  g->have_census = have_census;
  for (int k = 0; k < 32; ++k) g->census[k] = census[k];
  *out = g;
  return COOP_OK;
}

int coop_graph_load(const int64_t* indptr, const int32_t* indices, int64_t n_vertices, int64_t n_edges, int flags,
                    void* stream, coop_graph** out) {
  return coop_graph_load_with(indptr, indices, n_vertices, n_edges, flags, nullptr, nullptr, stream, out);
}

int coop_graph_free(coop_graph* g) {
  if (g && g->rev_pos && g->own_rev) (void)hipFree(g->rev_pos);
  delete g;
  return COOP_OK;
}

int coop_profile_enable(int on) {
  std::lock_guard<std::mutex> lk(g_prof.mu);
  if (!on) collect_locked();
  g_prof.on = on != 0;
  return COOP_OK;
}

int coop_profile_filter(int id) {
  if (id >= K_COUNT_) return COOP_E_ARG;
  std::lock_guard<std::mutex> lk(g_prof.mu);
  g_prof.only = id < 0 ? -1 : id;
  return COOP_OK;
}

int coop_profile_reset(void) {
  std::lock_guard<std::mutex> lk(g_prof.mu);
  collect_locked();
  for (int i = 0; i < K_COUNT_; ++i) { g_prof.ms[i] = 0; g_prof.launches[i] = 0; }
  return COOP_OK;
}

int coop_profile_kernels(void) { return K_COUNT_; }

const char* coop_profile_name(int id) { return (id >= 0 && id < K_COUNT_) ? kKernelNames[id] : nullptr; }

int coop_profile_read(int id, double* total_ms, int64_t* launches) {
  if (id < 0 || id >= K_COUNT_) return COOP_E_ARG;
  std::lock_guard<std::mutex> lk(g_prof.mu);
  collect_locked();
  if (total_ms) *total_ms = g_prof.ms[id];
  if (launches) *launches = g_prof.launches[id];
  return COOP_OK;
}

}  // extern "C"
