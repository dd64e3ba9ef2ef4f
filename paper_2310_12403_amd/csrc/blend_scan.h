// The traversal with blended variates (c > 0), of LABOR-0 and of NS: lists to stage-1 passers, a queue of them in LDS, the blend in
// fp32 for a full wave of them at a time.
//
// Stage 2 is some 230 instructions for up to 64 candidates, stage 1 27 for 64 entries and layer, of which 1 to 10 in a hundred pass.  What
// lies between is kept short: a group's candidates take their places together, without a branch per entry; the queue is emptied
// from its end, so that nothing moves to the front; and stage 2 stands once per group of a step and layer (seventeen copies per layer, one
// behind every place where the queue can fill up, did not fit the instruction cache).
#pragma once
#include "blend_filters.h"
#include "list_reader.h"
#include "sample_internal.h"

namespace coop {

// The exact blend.  (Not inlined, for kernels that are not about it: see k_ns_redo.)
static __device__ __attribute__((noinline)) uint32_t blend_exact(uint32_t u1, uint32_t u2, double cw, double sw) {
  return kit_phi_to_u32(__builtin_fma(cw, kit_phi_inv_u32(u1), sw * kit_phi_inv_u32(u2)));
}

// Stage-1 passers of one covered layer wait here (per wave, in LDS): the neighbour, its list position, and the lane that has its
// list's thresholds.  The last kWave places: one per lane that nobody reads.
constexpr uint32_t kBlendQueue = 3 * kWave;
template <bool NS>
struct BlendQueue {
  StageEntry at[kBlendQueue + kWave];
  uint8_t slot[kBlendQueue + kWave];
  uint32_t own[kWave];              // what the sink has taken so far from the list of each lane
  float lim2[kWave];                // threshold of stage 2 of the list of each lane
  float keep2[NS ? 1 : kWave];      // (LABOR-0) ... from below
  uint32_t mid_a[NS ? kWave : 1], mid_b[NS ? kWave : 1];  // (NS) its words of the two uniforms
};

// What a wave of a blended scan has at hand: NF layers, of LABOR-0 or of NS (then NF = 1), and what takes the estimates of stage 2.
template <int NF, bool NS, typename Sink>
struct BlendScan {
  BlendQueue<NS>* queue;   // [NF]
  uint32_t waiting[NF];    // entries in the queues (the same in every lane; below 64 between calls)
  uint32_t head_a[NF], tail_a[NF], head_b[NF], tail_b[NF];  // key words, in vector registers
  uint32_t mid_a, mid_b;  // (NS: of the list that the entries at hand belong to)
  float cwf, swf;
  Sink sink;

  __device__ __forceinline__ void set_keys(int l, const LayerKeys& K) {
    head_a[l] = vector_copy(K.Ka[4]);
    tail_a[l] = vector_copy(K.Ka[NS ? 3 : 1]);
    head_b[l] = vector_copy(K.Kb[4]);
    tail_b[l] = vector_copy(K.Kb[NS ? 3 : 1]);
    waiting[l] = 0;
  }

  // Stage 2 on n <= 64 entries of layer l's queue from `from` on: the two uniforms again, the blend in fp32.
  __device__ __forceinline__ void second(int l, uint32_t from, uint32_t n) {
    const uint32_t lane = (uint32_t)lane_id();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    StageEntry e{0, 0};
    uint32_t slot = 0;
    if (lane < n) {
      e = queue[l].at[from + lane];
      slot = queue[l].slot[from + lane];
    }
    const uint32_t ma = NS ? queue[l].mid_a[slot] : 0u, mb = NS ? queue[l].mid_b[slot] : 0u;
    const uint32_t u1 = words_uniform<NS>(head_a[l], ma, tail_a[l], (uint32_t)e.t), u2 = words_uniform<NS>(head_b[l], mb, tail_b[l], (uint32_t)e.t);
    sink.take(queue, l, lane < n, e, slot, u1, u2, __builtin_fmaf(cwf, approx_phi_inv_f32(u1), swf * approx_phi_inv_f32(u2)));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  // Four entries per lane, those of the masks m[0..3] being stage-1 passers of layer l, at list positions j + e step: they join the
  // layer's queue, together where they fit (nearly always) or 64 at most at a time, and whole waves of them go through stage 2.
  // (The last ones first: nothing has to move to the front.)
  __device__ __forceinline__ void join(int l, const uint32_t (&t)[4], const uint64_t (&m)[4], uint32_t j, uint32_t step, uint32_t slot) {
    if ((m[0] | m[1] | m[2] | m[3]) == 0) return;
    const uint32_t idle = kBlendQueue + (uint32_t)lane_id();
    const uint32_t all = waiting[l] + (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
    const uint64_t m0 = m[0], m1 = m[1], m2 = m[2], m3 = m[3];
    const uint32_t t0 = t[0], t1 = t[1], t2 = t[2], t3 = t[3];
    uint32_t done = 0;
    if (all <= kBlendQueue) {
      uint32_t to = waiting[l];
#pragma unroll
      for (int e = 0; e < 4; ++e) to = lanes_below_plus(m[e], to);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t at = lane_in(m[e]) ? to : idle;
        queue[l].at[at] = StageEntry{(int32_t)t[e], j + e * step};
        queue[l].slot[at] = (uint8_t)slot;
        to += lane_in(m[e]) ? 1u : 0u;
      }
      waiting[l] = all;
      done = 4;
    }
#pragma nounroll
    for (;;) {
      if (waiting[l] >= (uint32_t)kWave) {
        waiting[l] -= kWave;
        second(l, waiting[l], kWave);
        continue;
      }
      if (done == 4) break;
      const uint64_t mm = done < 2 ? (done == 0 ? m0 : m1) : (done == 2 ? m2 : m3);
      const uint32_t tt = done < 2 ? (done == 0 ? t0 : t1) : (done == 2 ? t2 : t3);
      const uint32_t to = lanes_below_plus(mm, waiting[l]);  // (below 128)
      if (lane_in(mm)) {
        queue[l].at[to] = StageEntry{(int32_t)tt, j + done * step};
        queue[l].slot[to] = (uint8_t)slot;
      }
      waiting[l] += (uint32_t)__popcll(mm);
      ++done;
    }
  }
  __device__ __forceinline__ void flush() {
#pragma unroll
    for (int l = 0; l < NF; ++l)
      if (waiting[l] != 0) {
        second(l, 0u, waiting[l]);
        waiting[l] = 0;
      }
  }

  // Stage 1 for one entry.  It looks at the uniforms without their last fold: the bounds come rounded up to whole upper halves, so that
  // nothing is lost.  The test is (lo <= a1) | (lo <= a2 & hi <= b2), a1 <= a2.
  __device__ __forceinline__ uint64_t passes(int l, uint32_t t, uint32_t a1, uint32_t a2, uint32_t b2) const {
    const uint32_t u1 = words_rough<NS>(head_a[l], mid_a, tail_a[l], t), u2 = words_rough<NS>(head_b[l], mid_b, tail_b[l], t);
    const uint32_t lo = u1 < u2 ? u1 : u2, hi = u1 < u2 ? u2 : u1;
    const uint32_t edge = hi <= b2 ? a2 : a1;
    return compare_mask(lo <= edge);
  }

  // Stage 1 on a list (or a stretch of it that starts at list position j0) whose thresholds lane `slot` has.
  __device__ __forceinline__ void collect(ListReader<>& L, uint32_t j0, uint32_t slot, const uint32_t (&a1)[NF], const uint32_t (&a2)[NF],
                                          const uint32_t (&b2)[NF]) {
    const uint32_t lane = (uint32_t)lane_id();
    for (uint32_t g0 = 0; g0 < L.n_groups; g0 += kReaderGroups) {
#pragma unroll
      for (uint32_t q = 0; q < kReaderGroups; ++q) {
        const uint32_t g = g0 + q;
        if (g >= L.n_groups) break;
        const uint32_t t[4] = {L.ring[q][0], L.ring[q][1], L.ring[q][2], L.ring[q][3]};
#pragma unroll
        for (int l = 0; l < NF; ++l) {  // (layer by layer: the masks of all of them would not fit the scalar registers)
          uint64_t m[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) m[e] = passes(l, t[e], a1[l], a2[l], b2[l]);
          join(l, t, m, j0 + g * kGroup + lane * 4, 1u, slot);
        }
        if (g + kReaderGroups < L.n_groups) L.ring[q] = L.in.group(g + kReaderGroups);
      }
    }
    const uint32_t tail = L.n & ~(kGroup - 1);
    if (tail == L.n) return;
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      uint64_t m[4] = {0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (tail + q * kWave < L.n) m[q] = passes(l, L.rest[q], a1[l], a2[l], b2[l]) & low_lanes(L.n - tail - q * kWave);
      join(l, L.rest, m, j0 + tail + lane, (uint32_t)kWave, slot);
    }
  }
};

}  // namespace coop
