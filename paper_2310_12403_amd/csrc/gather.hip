// Feature loading step of Algorithm 1: out[i, :] = feat[ids[i], :], an exact copy of bits.
//
// HBM-bound row gather.  The rows' items (device_utils.h: up to 16 bytes each, at whatever alignment the row has) are
// dealt to the threads of the grid in order, kGatherUnroll per thread in flight to cover the latency of the random row
// reads.  Loads and stores are non-temporal: a row is used once.  Against a power of two of lanes per row and the widest
// vectors that divide row and bases: rows of 75 fp16 columns (2-byte vectors before) 64 -> 24 us for 284 thousand rows, rows
// of 602 fp32 columns (8-byte vectors) 243 -> 229 us for 233 thousand (4.9 TB/s; a plain copy of 2 GiB reaches 4.9), rows
// of 100 fp32 columns (25 items on 32 lanes) 178 -> 170 us, rows of 128 fp16 columns unchanged.
#include <hip/hip_fp16.h>

#include <mutex>

#include "coop_internal.h"
#include "device_utils.h"

namespace coop {

constexpr int kGatherUnroll = 4;

template <int VB>
__global__ __launch_bounds__(kBlock) void k_gather(const char* __restrict__ feat, int64_t n_rows, RowShape sh, const int32_t* __restrict__ ids,
                                                   int64_t n_ids, char* __restrict__ out, int32_t* __restrict__ bad) {
  const BlockItems items((int64_t)blockIdx.x * (kBlock * kGatherUnroll), sh.vecs);
  int64_t row[kGatherUnroll];
  int32_t id[kGatherUnroll];
  uint32_t item[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    row[u] = items.row_of((uint32_t)(u * kBlock) + threadIdx.x, sh, &item[u]);
    id[u] = ids[row[u] < n_ids ? row[u] : n_ids - 1];  // (all of them requested before the first one is looked at)
  }
  typename RowVec<VB>::T x[kGatherUnroll];
  char* to[kGatherUnroll];
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    const int64_t at = BlockItems::byte_of<VB>(item[u], sh);
    to[u] = out + (row[u] < n_ids ? row[u] : n_ids - 1) * sh.row_bytes + at;
    // every load is issued, without a branch: that of an id out of range reads the place it would be written to
    x[u] = row_load_nt<VB>((uint64_t)(int64_t)id[u] < (uint64_t)n_rows ? feat + id[u] * sh.row_bytes + at : to[u]);
  }
#pragma unroll
  for (int u = 0; u < kGatherUnroll; ++u) {
    if (row[u] >= n_ids) continue;
    const bool ok = (uint64_t)(int64_t)id[u] < (uint64_t)n_rows;
    row_store_nt<VB>(to[u], ok ? x[u] : typename RowVec<VB>::T{});
    if (!ok && item[u] == 0) atomicOr(bad, 1);
  }
}

// ---- neighbour mean fused with the feature load ------------------------------------------------------------------
// out[i, :] = mean over the sampled in-edges e of destination i of feat[col[e], :]  (Eq. 1 with a mean aggregator,
// the first thing a GCN / GraphSAGE layer does with the loaded rows), 0 for a destination without edges.  The rows
// are read straight from the feature table and never written out individually: the kernel moves m rows in and
// n_dst rows out.  Accumulation is fp32, one lane per column group, edges in adjacency order (deterministic).
constexpr int kMeanUnroll = 4;

template <typename V, bool F16>
struct MeanAcc {
  static constexpr int kN = F16 ? (int)(sizeof(V) / 2) : (int)(sizeof(V) / 4);
  float a[kN];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < kN; ++i) a[i] = 0.f;
  }
  __device__ __forceinline__ void add(const V& x) {
    if constexpr (F16) {
      const __half* h = reinterpret_cast<const __half*>(&x);
#pragma unroll
      for (int i = 0; i < kN; ++i) a[i] += __half2float(h[i]);
    } else {
      const float* f = reinterpret_cast<const float*>(&x);
#pragma unroll
      for (int i = 0; i < kN; ++i) a[i] += f[i];
    }
  }
  __device__ __forceinline__ V mean(float count) const {
    V r;
    if constexpr (F16) {
      __half* h = reinterpret_cast<__half*>(&r);
#pragma unroll
      for (int i = 0; i < kN; ++i) h[i] = __float2half_rn(a[i] / count);
    } else {
      float* f = reinterpret_cast<float*>(&r);
#pragma unroll
      for (int i = 0; i < kN; ++i) f[i] = a[i] / count;
    }
    return r;
  }
};

template <int VB, bool F16>
__global__ __launch_bounds__(kBlock) void k_gather_mean(int64_t block0, const char* __restrict__ feat, int64_t n_rows, RowShape sh,
                                                        const int64_t* __restrict__ indptr, const int32_t* __restrict__ col,
                                                        int64_t n_dst, char* __restrict__ out, int32_t* __restrict__ bad) {
  typedef typename RowVec<VB>::T V;
  const BlockItems items((block0 + (int64_t)blockIdx.x) * kBlock, sh.vecs);
  uint32_t item;
  const int64_t i = items.row_of(threadIdx.x, sh, &item);
  if (i >= n_dst) return;
  const int64_t at = BlockItems::byte_of<VB>(item, sh);
  const int64_t beg = indptr[i], end = indptr[i + 1];
  MeanAcc<V, F16> acc;
  acc.clear();
  for (int64_t e = beg; e < end; e += kMeanUnroll) {
    V x[kMeanUnroll];
    bool ok[kMeanUnroll];
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u) {
      ok[u] = false;
      if (e + u < end) {
        const int64_t id = col[e + u];
        ok[u] = (uint64_t)id < (uint64_t)n_rows;
        if (ok[u]) x[u] = *reinterpret_cast<const typename RowVec<VB>::U*>(feat + id * sh.row_bytes + at);
        else if (item == 0) atomicOr(bad, 1);
      }
    }
#pragma unroll
    for (int u = 0; u < kMeanUnroll; ++u)
      if (ok[u]) acc.add(x[u]);
  }
  const int64_t cnt = end - beg;
  row_store_nt<VB>(out + i * sh.row_bytes + at, cnt > 0 ? acc.mean((float)cnt) : V{});
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_bad_mu;
// Sticky "an id was out of range" word.  A device variable of this library's code object (zero when the code object is
// loaded): every GPU has its own copy at its own address, which hipGetSymbolAddress gives for the current device.
// Nothing is allocated for it, so the entry points that promise not to allocate can report through it as well.
static __device__ int32_t g_bad_word;
int32_t* g_bad_flag[kMaxDevices] = {};  // per device: the address of that device's copy

}  // namespace

// the current device's flag word (its address is looked up on first use and kept for the life of the process)
int32_t* bad_flag() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_bad_mu);
  if (!g_bad_flag[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_bad_word)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_bad_flag[dev] = (int32_t*)p;
  }
  return g_bad_flag[dev];
}

namespace {

template <int VB>
void launch_gather(const void* feat, int64_t n_rows, const RowShape& sh, const int32_t* ids, int64_t n_ids, void* out, int32_t* bad,
                   hipStream_t s) {
  constexpr int64_t per_block = kBlock * kGatherUnroll;
  const unsigned grid = (unsigned)((n_ids * (int64_t)sh.vecs + per_block - 1) / per_block);
  COOP_LAUNCH(K_GATHER, k_gather<VB>, dim3(grid), dim3(kBlock), 0, s, (const char*)feat, n_rows, sh, ids, n_ids, (char*)out, bad);
}
}  // namespace

}  // namespace coop

using namespace coop;

extern "C" int coop_gather(const void* feat, int64_t n_rows, int32_t dim, int dtype, const int32_t* ids, int64_t n_ids, void* out,
                           void* stream) {
  if (dtype != COOP_F32 && dtype != COOP_F16) return COOP_E_ARG;
  if (dim < 1 || n_rows < 0 || n_ids < 0) return COOP_E_ARG;
  if (n_ids == 0) return COOP_OK;
  if (!feat || !ids || !out) return COOP_E_NULL;
  const RowShape sh = row_shape((int64_t)dim * (dtype == COOP_F32 ? 4 : 2));
  if ((n_ids + 255) / 256 > 0x7FFFFFFF || n_ids > ((int64_t)0x7FFFFFFF * kBlock) / (int64_t)sh.vecs) return COOP_E_ARG;
  int32_t* bad = bad_flag();
  if (!bad) return COOP_E_HIP;
  hipStream_t s = (hipStream_t)stream;
  if ((((uintptr_t)feat | (uintptr_t)out) & 1) != 0) return COOP_E_ARG;  // fp16 / fp32 tables are at least 2-byte aligned
  switch (sh.vec_bytes) {
    case 16: launch_gather<16>(feat, n_rows, sh, ids, n_ids, out, bad, s); break;
    case 8: launch_gather<8>(feat, n_rows, sh, ids, n_ids, out, bad, s); break;
    case 4: launch_gather<4>(feat, n_rows, sh, ids, n_ids, out, bad, s); break;
    default: launch_gather<2>(feat, n_rows, sh, ids, n_ids, out, bad, s); break;
  }
  if (hipGetLastError() != hipSuccess) return COOP_E_HIP;
  return COOP_OK;
}

namespace {
template <int VB, bool F16>
void launch_mean(const void* feat, int64_t n_rows, const RowShape& sh, const int64_t* indptr, const int32_t* col, int64_t n_dst,
                 void* out, int32_t* bad, hipStream_t s) {
  const int64_t blocks = (n_dst * (int64_t)sh.vecs + kBlock - 1) / kBlock;
  for (int64_t b = 0; b < blocks; b += kSliceBlocks)
    COOP_LAUNCH(K_GATHER_MEAN, (k_gather_mean<VB, F16>), dim3((unsigned)(blocks - b < kSliceBlocks ? blocks - b : kSliceBlocks)), dim3(kBlock),
                0, s, b, (const char*)feat, n_rows, sh, indptr, col, n_dst, (char*)out, bad);
}
}  // namespace

extern "C" int coop_gather_mean(const void* feat, int64_t n_rows, int32_t dim, int dtype, const int64_t* indptr,
                                const int32_t* col_global, int64_t n_dst, void* out, void* stream) {
  if (dtype != COOP_F32 && dtype != COOP_F16) return COOP_E_ARG;
  if (dim < 1 || n_rows < 0 || n_dst < 0) return COOP_E_ARG;
  if (n_dst == 0) return COOP_OK;
  if (!feat || !indptr || !out) return COOP_E_NULL;  // col_global may be NULL only if there are no edges; not checkable here
  const RowShape sh = row_shape((int64_t)dim * (dtype == COOP_F32 ? 4 : 2));
  if ((n_dst + 255) / 256 > 0x7FFFFFFF || n_dst > ((int64_t)0x7FFFFFFF * kBlock) / (int64_t)sh.vecs) return COOP_E_ARG;
  int32_t* bad = bad_flag();
  if (!bad) return COOP_E_HIP;
  hipStream_t s = (hipStream_t)stream;
  if ((((uintptr_t)feat | (uintptr_t)out) & (dtype == COOP_F16 ? 1 : 3)) != 0) return COOP_E_ARG;
  if (dtype == COOP_F16) {
    switch (sh.vec_bytes) {
      case 16: launch_mean<16, true>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
      case 8: launch_mean<8, true>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
      case 4: launch_mean<4, true>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
      default: launch_mean<2, true>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
    }
  } else {
    switch (sh.vec_bytes) {
      case 16: launch_mean<16, false>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
      case 8: launch_mean<8, false>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
      default: launch_mean<4, false>(feat, n_rows, sh, indptr, col_global, n_dst, out, bad, s); break;
    }
  }
  if (hipGetLastError() != hipSuccess) return COOP_E_HIP;
  return COOP_OK;
}

extern "C" int coop_gather_status(void* stream) {
  int32_t* bad = bad_flag();
  if (!bad) return COOP_E_HIP;
  hipStream_t s = (hipStream_t)stream;
  int32_t h = 0;
  COOP_HIP_TRY(hipMemcpyAsync(&h, bad, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  COOP_HIP_TRY(hipStreamSynchronize(s));
  if (h) {
    COOP_HIP_TRY(hipMemsetAsync(bad, 0, sizeof(int32_t), s));
    COOP_HIP_TRY(hipStreamSynchronize(s));
    return COOP_E_RANGE;
  }
  return COOP_OK;
}
