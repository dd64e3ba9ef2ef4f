// A neighbour list on its way to a wave: what the traversals read (k_ns_fill, k_labor_scan_plain, and blend_scan.h with c > 0).
#pragma once
#include "device_utils.h"
#include "dealing.h"
#include "variates.h"

namespace coop {

// A list read through a buffer descriptor: an addition per load in the place of a lane's 64-bit address, and entries behind the
// end come back as zeros without a test (the whole offset is in the vector register: the check leaves a scalar offset out).
// 16 bytes per lane or 4, at the alignment of the entries.
struct ListLoads {
  static constexpr int kAux = 2;  // non-temporal
  __amdgpu_buffer_rsrc_t rsrc;
  int lane4, lane16;
  __device__ __forceinline__ ListLoads(const int32_t* list, uint32_t n /* <= 2^28 */)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(list), 0, (int)(n * 4u), 0x00020000)), lane4(lane_id() * 4), lane16(lane_id() * 16) {}
  __device__ __forceinline__ u32x4 group(uint32_t g) const {  // entries 256 g + 4 lane ..
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane16 + (int)(g * 1024u), 0, kAux);
  }
  __device__ __forceinline__ uint32_t entry(uint32_t at) const { return __builtin_amdgcn_raw_buffer_load_b32(rsrc, lane4 + (int)(at * 4u), 0, kAux); }
};

// The entries of a list (or of a stretch of it): whole groups of 256, and the rest 64 at a time.  Everything that fits is requested
// at once; a loop over the groups asks for group g + GROUPS when it is through with group g.
constexpr uint32_t kGroup = kWave * 4;  // entries of a 16-byte load by every lane
constexpr uint32_t kReaderGroups = 4;   // ... of which so many are in flight
constexpr uint32_t kStretchMost = 1u << 28;  // entries that a descriptor's offsets reach: longer lists are read in stretches (g_stretch)
template <uint32_t GROUPS = kReaderGroups>
struct ListReader {
  ListLoads in;
  uint32_t n, n_groups;
  u32x4 ring[GROUPS];
  uint32_t rest[4];
  __device__ __forceinline__ ListReader(const int32_t* list, uint32_t entries) : in(list, entries), n(entries), n_groups(entries / kGroup) {
    // (no load for what is not there: 16 bytes per lane cost a CU 16 clocks, also where every lane is behind the end)
    const uint32_t tail = n & ~(kGroup - 1);
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      rest[q] = any_value();
      if (tail + q * kWave < n) rest[q] = in.entry(tail + q * kWave);
    }
#pragma unroll
    for (uint32_t q = 0; q < GROUPS; ++q) {
      ring[q] = u32x4{any_value(), any_value(), any_value(), any_value()};
      if (q < n_groups) ring[q] = in.group(q);
    }
  }
};

}  // namespace coop
