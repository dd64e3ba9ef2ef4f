// NS layers (App. A.1.1): a destination of degree d <= k keeps all of N(s); otherwise it keeps the k neighbours with
// the smallest (R_ts, list position), a uniform k-subset.  Kept edges leave in (destination order, adjacency order).
// The count is known without looking at the list (min(k, d)), so every list is read once, by the fill pass.
#include "blend_scan.h"

namespace coop {

// Filters between a blended NS variate and its exact evaluation, for the candidate test R <= bound (c > 0 only).
struct NsBlendThr {
  uint32_t a2, a1, b2;  // integer bounds on min(U1, U2) and max(U1, U2), as for LABOR-0
  float lim2;           // the blend in fp32 above this cannot be a candidate
};
__device__ __forceinline__ NsBlendThr ns_blend_thresholds(uint32_t bound, double cw, double sw) {
  const double tau = blend_tau(bound);
  const PreThr p = blend_first_thresholds(bound, tau, cw, sw);
  return NsBlendThr{p.a2, p.a1, p.b2, blend_second_threshold(bound, tau, cw + sw)};
}

// One destination's neighbour list as the fill pass sees it (written by the count pass, so that the fill pass
// reaches the list with one dependent load instead of three).
struct NsRecord {
  int64_t beg;
  uint32_t d;
  int32_t s;
  uint32_t bound;  // first candidate bound: about `target` of the d variates are expected below it
  uint32_t mid;    // the destination's word of the variates of group g (ns_mid)
};

// (long_min > 0: the destinations whose list is longer than long_min entries, and than k, are also queued in long_list,
// in no particular order, *n_long counting them: the traversal kernels give those to their first waves, see there.  A
// block reserves its places with one returning atomic, and those on one address are taken one after the other, some 20 ns
// each: 675 thousand destinations took 40 us in blocks of 256 and take 28 in blocks of 1,024 threads with two each.  Below
// kNsCountWideFrom destinations, and with c > 0, where every destination has its thresholds evaluated in fp64, the small
// blocks are the quicker ones: 10 us against 12 for 110 thousand, 5 against 8 for 16 thousand, and half the time with c > 0;
// with c > 0 below 16,384 blocks of one wave, which spread over more CUs.)
constexpr int64_t kNsCountWideFrom = 262144;
constexpr int ns_tile_log2(int n) { return n <= 1 ? 0 : 1 + ns_tile_log2(n / 2); }
template <int kNsCountBlock, int kNsCountEach>
__global__ __launch_bounds__(kNsCountBlock) void k_ns_count(const int64_t* __restrict__ g_indptr, int64_t n_vertices,
                                                            const int32_t* dst, int64_t n_dst, uint32_t k, uint32_t target,
                                                            int64_t* __restrict__ indptr, NsRecord* __restrict__ rec,
                                                            NsBlendThr* __restrict__ bthr /* null when c = 0 */, LayerKeys keys, double cw, double sw, Ctl* ctl,
                                                            uint32_t long_min, uint32_t* __restrict__ long_list, uint32_t* __restrict__ n_long,
                                                            Clear clear, Begin begin, Publish pub) {
  dst = begin_in_block(begin, dst);
  clear_words(clear);
  constexpr int kWaves = kNsCountBlock / kWave;
  __shared__ uint32_t wave_long[kWaves];
  __shared__ uint32_t block_base, s_last;
  __shared__ int64_t lds[kWaves];
  const uint32_t* K = keys.Ka;
  const int64_t i0 = (int64_t)blockIdx.x * (kNsCountBlock * kNsCountEach) + threadIdx.x;
  bool is_long[kNsCountEach];
  int64_t cnt[kNsCountEach];
  int32_t s[kNsCountEach];
  int64_t beg[kNsCountEach], end[kNsCountEach];
#pragma unroll
  for (int u = 0; u < kNsCountEach; ++u) {
    const int64_t i = i0 + u * kNsCountBlock;
    s[u] = i < n_dst ? dst[i] : -1;
  }
#pragma unroll
  for (int u = 0; u < kNsCountEach; ++u) {
    beg[u] = end[u] = 0;
    if ((uint64_t)(uint32_t)s[u] < (uint64_t)n_vertices) {
      beg[u] = g_indptr[s[u]];
      end[u] = g_indptr[s[u] + 1];
    }
  }
#pragma unroll
  for (int u = 0; u < kNsCountEach; ++u) {
    const int64_t i = i0 + u * kNsCountBlock;
    is_long[u] = false;
    cnt[u] = 0;
    if (i >= n_dst) continue;
    if ((uint64_t)(uint32_t)s[u] >= (uint64_t)n_vertices) {
      atomicOr(&ctl->err_range, 1);
      __threadfence();  // (before the block counts itself, below)
      rec[i] = NsRecord{0, 0u, 0, 0u, 0u};
      if (bthr) bthr[i] = NsBlendThr{0u, 0u, 0u, 0.0f};
      continue;
    }
    const int64_t d = end[u] - beg[u];
    cnt[u] = d < (int64_t)k ? d : (int64_t)k;
    // bound such that E[#candidates] = target: R <= bound with probability (bound + 1) / 2^32 (one 64-bit division per
    // list, here where every lane has a list of its own)
    uint64_t bound = d > 0 ? ((uint64_t)target << 32) / (uint64_t)d : 0xFFFFFFFFull;
    if (bound > 0xFFFFFFFFull) bound = 0xFFFFFFFFull;  // d <= target: every neighbour is a candidate
    rec[i] = NsRecord{beg[u], (uint32_t)d, s[u], (uint32_t)bound, ns_mid(K, ns_sigma(K, (uint32_t)s[u]))};
    if (bthr) bthr[i] = d > (int64_t)k ? ns_blend_thresholds((uint32_t)bound, cw, sw) : NsBlendThr{0u, 0u, 0u, 0.0f};
    is_long[u] = long_min != 0 && d > (int64_t)long_min && d > (int64_t)k;
  }
  if (long_min != 0) {  // (the same for every thread)
    uint64_t mask[kNsCountEach];
    uint32_t mine = 0;
#pragma unroll
    for (int u = 0; u < kNsCountEach; ++u) {
      mask[u] = ballot64(is_long[u]);
      mine += (uint32_t)__popcll(mask[u]);
    }
    const int wib = wave_in_block();
    if (lane_id() == 0) wave_long[wib] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {  // one reservation per block
      uint32_t total = 0;
      for (int w = 0; w < kWaves; ++w) total += wave_long[w];
      block_base = total ? atomicAdd(n_long, total) : 0u;
    }
    __syncthreads();
    uint32_t at = block_base;
    for (int w = 0; w < wib; ++w) at += wave_long[w];
#pragma unroll
    for (int u = 0; u < kNsCountEach; ++u) {
      const uint32_t to = at + lanes_below(mask[u]);
      if (is_long[u] && (int64_t)to < n_dst) long_list[to] = (uint32_t)(i0 + u * kNsCountBlock);  // (always: a destination is queued at most once)
      at += (uint32_t)__popcll(mask[u]);
    }
  }
  // The offsets, as scan_tiles leaves them, the block's destinations being a tile.  (Two launches of 5 us less than a scan of stored
  // counts.)
  int64_t in_front = 0;
#pragma unroll
  for (int u = 0; u < kNsCountEach; ++u) {
    const int64_t i = i0 + u * kNsCountBlock;
    int64_t sum;
    const int64_t upto = in_front + block_incl_scan_i64<kWaves>(cnt[u], &sum, lds);
    if (i < n_dst && (u != 0 || threadIdx.x != 0)) indptr[i] = upto - cnt[u];
    in_front += sum;
  }
  int64_t total = in_front;
  if (gridDim.x == 1) {  // (nobody to wait for: 3.0 us in the place of 4.6)
    if (threadIdx.x == 0) indptr[0] = 0;
  } else {
    if (threadIdx.x == 0) s_last = tile_sum_done(in_front, indptr + i0, ctl) ? 1u : 0u;
    __syncthreads();
    if (s_last == 0) return;
    constexpr int kLog2 = ns_tile_log2(kNsCountBlock * kNsCountEach);
    total = scan_tile_sums<kWaves>(n_dst, kLog2, indptr, lds);
  }
  if (threadIdx.x == 0) {
    indptr[n_dst] = total;
    ctl->total_edges = total;
    if (pub.h != nullptr) {
      Ctl c = *ctl;  // (the fields of earlier kernels; those of this one follow)
      c.total_edges = total;
      c.err_range = __hip_atomic_load(&ctl->err_range, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      send_ctl(pub.h, pub.ticket, c);
    }
  }
}

// The offset of destination w, its final value put in the place of what k_ns_count left there: by one wave per destination, in
// the first kernel that uses the offsets.
__device__ __forceinline__ int64_t ns_offset(const int64_t* indptr, int64_t w, int tile_log2) {
  const int64_t tile = w >> tile_log2 << tile_log2;
  return indptr[tile] + (w != tile ? indptr[w] : 0);
}
__device__ __forceinline__ void ns_settle_offset(int64_t* indptr, int64_t w, int tile_log2, int64_t o) {
  if ((w & (((int64_t)1 << tile_log2) - 1)) != 0) indptr[w] = o;
}

constexpr uint32_t kNsMaxSelect = 1024;  // largest fanout for which a longer list is subsampled through the candidate arrays
constexpr int64_t kNsQueueFrom = 32768;  // destinations from which the long lists are queued for the first waves
constexpr int kNsLongDefault = 2048;
int g_ns_long_min = kNsLongDefault;      // COOP_TUNE_NS_LONG_LIST: lists longer than this are queued (0 = none)
constexpr uint32_t kNsRedo = 0xFFFFFFFFu;  // candidate count of a destination that the two-kernel path leaves to k_ns_redo
// Such destinations, about one in 10^4, are found by their marks in n_cand.  A wave looks at as many marks as leave at least
// kNsRedoWaves waves, up to one per lane: a wave for each mark costs 0.2 ns a mark (675 thousand destinations: 451 us for the
// traversal and this, against 314).  Where one neighbour occurs many times over, every list can be among them, so there is no
// queue (an atomic per list on its counter, one after the other) and no bound on the waves: 100 thousand such lists 1.86 ms,
// as with a wave each, against 9.3 with a queue and 1,024 waves.
constexpr int64_t kNsRedoWaves = 16384;
constexpr int64_t kNsFillWaves = 16384;  // k_ns_fill's waves take up to eight destinations, where that leaves at least this many waves

typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int kNsGroups = 4;  // 16-byte groups per lane and step of the fast traversal
// Groups of a list in flight in k_ns_fill: as many as 64 registers hold.  A list of 2 million entries is one wave's, waiting for
// memory, and a group is requested when the one in its place has been looked at: 1.81 ms with four in flight, 1.72 with five, 1.64
// with six, 1.58 with seven; short lists the same with any of them.
constexpr uint32_t kFillGroups = 7;

// Stage-1 passers of the blended path wait here (per wave, in LDS) until 64 of them can be evaluated together.
constexpr int kNsQueueCap = 2 * kWave;
struct NsQueue {
  int32_t t[kNsQueueCap];
  uint32_t j[kNsQueueCap];
  uint32_t u1[kNsQueueCap];  // (ns_rough)
  uint32_t u2[kNsQueueCap];
};

// A candidate in LDS; slot_key orders by (variate, list position), the order of the selection.
struct alignas(16) NsSlot {
  uint32_t j, r;  // list position, variate
  int32_t t;      // the vertex
  uint32_t keep;  // among the k smallest
};
__device__ __forceinline__ uint64_t slot_key(const NsSlot* c) { return ((uint64_t)c->r << 32) | c->j; }

// One pass over a list of d entries, c = 0: position and vertex of every neighbour whose variate is <= bound go to
// the slots, in list order (those beyond `cap` are counted but not stored); returns how many qualified.
//
// Bound by the issue of instructions: the chip issues 560 G vector ones of this kind a second (two per ns and CU) and as many
// scalar ones, and of the 225 M and 190 M that 717 thousand lists took, 13 of each 64 entries were the two mixers and the
// test, the others what a list and a candidate cost besides.  So: whole groups of 256
// entries (16 bytes per lane, at whatever alignment the list has: memory instructions take any) need no lane mask, and what
// is left, fewer than 256, is read 64 at a time, so that neither ragged ends nor half a group of idle lanes are paid for;
// the test leaves only masks in scalar registers; a group's masks give every lane the place of its first candidate, a
// lane's next one is a slot further, and lanes without one write to a slot of their own that nobody reads, so that there is no
// branch per entry.  The variate is not kept but evaluated again for the few dozen candidates.  kFillGroups
// groups are in flight, each requested as soon as its registers are free.
__device__ __forceinline__ uint32_t ns_collect_plain(ListReader<kFillGroups>& L, uint32_t j0, uint32_t bound, const NsKeys& K, NsSlot* __restrict__ slot, uint32_t cap,
                                                     uint32_t n_c) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t idle = cap + lane;  // (the slots behind the candidates')
  for (uint32_t g0 = 0; g0 < L.n_groups; g0 += kFillGroups) {
#pragma unroll
    for (uint32_t q = 0; q < kFillGroups; ++q) {
      const uint32_t g = g0 + q;
      if (g >= L.n_groups) break;
      uint64_t m[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = compare_mask(ns_uniform(K, L.ring[q][e]) <= bound);
      if ((m[0] | m[1] | m[2] | m[3]) != 0) {
        uint32_t to = n_c;
#pragma unroll
        for (int e = 0; e < 4; ++e) to = lanes_below_plus(m[e], to);
        const uint32_t j = j0 + g * kGroup + lane * 4;
        // (Whatever the group holds then fits the cap + kWave slots.  Those from cap on are the idle lanes' as well, who may write over
        // a candidate there: nobody looks at it, since with more than cap candidates the list is collected again.)
        if (n_c + kGroup <= cap + (uint32_t)kWave) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            NsSlot* s = slot + (lane_in(m[e]) ? to : idle);
            s->j = j + e;
            s->t = (int32_t)L.ring[q][e];
            to += lane_in(m[e]) ? 1u : 0u;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (lane_in(m[e])) {
              if (to < cap) {
                slot[to].j = j + e;
                slot[to].t = (int32_t)L.ring[q][e];
              }
              ++to;
            }
          }
        }
        n_c = (uint32_t)__builtin_amdgcn_readlane((int)to, kWave - 1);
      }
      if (g + kFillGroups < L.n_groups) L.ring[q] = L.in.group(g + kFillGroups);
    }
  }
  const uint32_t tail = L.n & ~(kGroup - 1);
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t at = tail + q * kWave;
    if (at >= L.n) return n_c;
    const uint64_t m = compare_mask(ns_uniform(K, L.rest[q]) <= bound) & low_lanes(L.n - at);
    const uint32_t to = lanes_below_plus(m, n_c);
    n_c += (uint32_t)__popcll(m);
    if (lane_in(n_c <= cap ? m : 0ull)) {
      slot[to].j = j0 + at + lane;
      slot[to].t = (int32_t)L.rest[q];
    }
  }
  return n_c;
}

// The same with c > 0.  The variate of an entry is evaluated exactly only if the integer bounds and then the fp32 blend cannot
// rule it out; the survivors of the integer bounds are evaluated 64 at a time.  The candidates are in no particular order.
template <bool VEC4>
__device__ __forceinline__ uint32_t ns_collect(const int32_t* __restrict__ g_indices, int64_t beg, uint32_t d, uint32_t bound,
                                               const NsBlendThr& bt, const VariateParams& vp, uint32_t sigma_a, uint32_t sigma_b,
                                               NsSlot* __restrict__ slot, uint32_t cap, NsQueue* __restrict__ q) {
  const uint32_t lane = (uint32_t)lane_id();
  uint32_t n_c = 0;
  auto append = [&](bool in, uint32_t r, uint32_t j, int32_t t) {
    const uint64_t mask = ballot64(in);
    if (mask == 0) return;
    const uint32_t p = n_c + lanes_below(mask);
    if (in && p < cap) {
      slot[p].j = j;
      slot[p].r = r;
      slot[p].t = t;
    }
    n_c += (uint32_t)__popcll(mask);
  };
  // ---- the queue, and evaluation of its first n entries
  uint32_t qn = 0;
  const float cwf = (float)vp.cw, swf = (float)vp.sw;
  auto evaluate = [&](uint32_t n) {
    int32_t t = 0;
    uint32_t j = 0, R = 0;
    bool in = false;
    if (lane < n) {
      t = q->t[lane];
      j = q->j[lane];
      const uint32_t u1 = ns_exact(vp.K.Ka, q->u1[lane]), u2 = ns_exact(vp.K.Kb, q->u2[lane]);
      if (__builtin_fmaf(cwf, approx_phi_inv_f32(u1), swf * approx_phi_inv_f32(u2)) <= bt.lim2) {
        R = blend_exact(u1, u2, vp.cw, vp.sw);
        in = R <= bound;
      }
    }
    append(in, R, j, t);
  };
  auto enqueue = [&](bool pre, int32_t t, uint32_t j, uint32_t u1, uint32_t u2) {
    const uint64_t mask = ballot64(pre);
    if (mask == 0) return;
    if (pre) {
      const uint32_t at = qn + lanes_below(mask);  // below 128
      q->t[at] = t; q->j[at] = j; q->u1[at] = u1; q->u2[at] = u2;
    }
    qn += (uint32_t)__popcll(mask);
    __builtin_amdgcn_wave_barrier();
    if (qn >= (uint32_t)kWave) {
      evaluate(kWave);
      const uint32_t rest = qn - kWave;  // fewer than 64: to the front
      int32_t mt = 0;
      uint32_t mj = 0, m1 = 0, m2 = 0;
      if (lane < rest) { mt = q->t[kWave + lane]; mj = q->j[kWave + lane]; m1 = q->u1[kWave + lane]; m2 = q->u2[kWave + lane]; }
      __builtin_amdgcn_wave_barrier();
      if (lane < rest) { q->t[lane] = mt; q->j[lane] = mj; q->u1[lane] = m1; q->u2[lane] = m2; }
      qn = rest;
      __builtin_amdgcn_wave_barrier();
    }
  };
  // first look at one entry: the integer bounds on its two uniforms (without their last fold, and the bounds rounded up to
  // whole upper halves, so that nothing is lost: ns_exact finishes the passers')
  auto first_look = [&](bool valid, int32_t t, uint32_t& r, uint32_t& u2) -> bool {
    const uint32_t folded = fold16((uint32_t)t);
    r = ns_rough(vp.K.Ka, folded, sigma_a);
    u2 = ns_rough(vp.K.Kb, folded, sigma_b);
    const uint32_t lo = r < u2 ? r : u2, hi = r < u2 ? u2 : r;
    return valid & ((lo <= (bt.a1 | 0xFFFFu)) | ((lo <= (bt.a2 | 0xFFFFu)) & (hi <= (bt.b2 | 0xFFFFu))));
  };

  if (!VEC4 || d <= (uint32_t)kWave) {
    for (uint32_t base = 0; base < d; base += kWave) {
      const uint32_t j = base + lane;
      int32_t t = 0;
      if (j < d) t = g_indices[beg + j];
      uint32_t r = 0, u2 = 0;
      const bool flag = first_look(j < d, t, r, u2);
      enqueue(flag, t, j, r, u2);
    }
  } else {
    constexpr uint32_t kStep = kWave * 4 * kNsGroups;
    const int64_t abeg = beg & ~(int64_t)3;        // first aligned group
    const uint32_t head = (uint32_t)(beg - abeg);  // entries of that group that precede the list
    const uint32_t total = head + d;               // list end, relative to abeg
    const uint32_t vec_end = total & ~3u;          // whole groups end here
    const uint32_t vec_beg = head ? 4u : 0u;       // whole groups start here
    const int32_t* __restrict__ p = g_indices + abeg;
    // (no loads of the next step before this step's entries are hashed: the registers are needed more)
    // the ragged ends (lanes 0..2: the entries in front of the first whole group; lanes 3..5: those behind the last one) are
    // requested now, not when the whole groups are done, so that a short list waits for memory once
    const uint32_t end_pos = lane < 3 ? head + lane : vec_end + (lane - 3);
    const bool end_valid = lane < 3 ? (head != 0 && end_pos < 4) : (lane < 6 && end_pos < total);
    int32_t end_t = 0;
    if (end_valid) end_t = p[end_pos];
    for (uint32_t base = vec_beg; base < vec_end; base += kStep) {
      i32x4 buf[kNsGroups];
      bool ok[kNsGroups];
#pragma unroll
      for (int gq = 0; gq < kNsGroups; ++gq) {
        const uint32_t r = base + (uint32_t)(gq * kWave * 4) + lane * 4;
        ok[gq] = r < vec_end;
        buf[gq] = i32x4{0, 0, 0, 0};
        if (ok[gq]) buf[gq] = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(p + r));
      }
      auto group = [&](int gq, bool valid) {
        const uint32_t r = base + (uint32_t)(gq * kWave * 4) + lane * 4;
        uint32_t R[4], U2[4];
        bool flag[4];
        bool any = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          flag[e] = first_look(valid, buf[gq][e], R[e], U2[e]);
          any |= flag[e];
        }
        if (ballot64(any) != 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) enqueue(flag[e], buf[gq][e], r + e - head, R[e], U2[e]);
        }
      };
#pragma unroll
      for (int gq = 0; gq < kNsGroups; ++gq) {
        if (base + (uint32_t)(gq * kWave * 4) >= vec_end) break;  // wave-uniform: the rest of this step lies behind the list
        group(gq, ok[gq]);
      }
    }
    {  // the ragged ends
      uint32_t r = 0, u2 = 0;
      const bool flag = first_look(end_valid, end_t, r, u2);
      enqueue(flag, end_t, end_pos - head, r, u2);
    }
  }
  if (qn != 0) evaluate(qn);
  __builtin_amdgcn_wave_barrier();
  return n_c;
}

// The k smallest by (variate, list position) among the n_c candidates in LDS (k <= n_c <= cap), written to the edge arrays
// from o on in adjacency order: every candidate's rank among the candidates is counted, ranks below k are kept, and a
// kept candidate's place is the number of kept candidates in front of it in the list.
//
// One candidate per lane, its key at hand; slots up to the next multiple of four behind the n candidates are there.  Every lane
// reads the keys one after the other from LDS (the same address for all lanes: a broadcast), two vector instructions per
// candidate where reading variate and position out of the other lanes' registers cost seven.
__device__ __forceinline__ uint32_t ns_rank(uint32_t n, const NsSlot* slot, uint64_t my_key) {
  uint32_t rank = 0;
  const uint32_t n_u = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
  for (uint32_t q = 0; q < n_u; q += 4)
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) rank += slot_key(slot + q + e) < my_key;
  return rank;
}
// fills the slots behind the n candidates up to a multiple of four with keys above all others (n <= 64)
__device__ __forceinline__ void ns_pad(uint32_t n, NsSlot* slot) {
  const uint32_t lane = (uint32_t)lane_id();
  if (lane < 4) slot[n + lane].j = slot[n + lane].r = 0xFFFFFFFFu;
}
__device__ __forceinline__ uint32_t ns_rank_of(uint32_t n_c, const NsSlot* slot, uint64_t my_key) {
  uint32_t rank = 0;
  for (uint32_t q = 0; q < n_c; ++q) rank += slot_key(slot + q) < my_key;
  return rank;
}
// More candidates than lanes (all with a variate <= bound).  The border of the k smallest is bisected, between 0 and `bound` and
// until exactly k lie on its side: some log2(n_c) + 1 counts, an LDS read and a comparison per 64 candidates, in the place of a rank
// for every candidate.  Of equal variates at the border the first in the list are kept.  ORDERED: the candidates stand in list order
// (c = 0), so a kept one's place is the number of kept ones in front of it; otherwise the k kept ones move to the front and are
// ranked by position.
// (Steps over 90 thousand lists of 30 to 1,500 entries, fanouts 60 and 200: 447 and 3,512 us with ranks, 217 and 515; c > 0 684 and
// 4,431, 412 and 1,196.  30 such lists with fanout 1,000: 2,461 and 73, c > 0 2,792 and 410.)
template <bool ORDERED>
__device__ __forceinline__ void ns_rank_write_many(uint32_t n_c, uint32_t k, uint32_t bound, NsSlot* slot, int64_t o, int64_t beg,
                                                   EdgeOut edges) {
  const uint32_t lane = (uint32_t)lane_id();
  auto settle = [] {
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
  };
  auto upto = [&](uint32_t border) {  // (slots up to the next multiple of 64 are there)
    uint32_t n = 0;
#pragma unroll 4
    for (uint32_t base = 0; base < n_c; base += kWave) n += (uint32_t)__popcll(compare_mask(slot[base + lane].r <= border) & low_lanes(n_c - base));
    return n;
  };
  constexpr uint32_t kAll = 0xFFFFFFFFu;
  uint32_t lo = 0, hi = bound, border = bound, need = kAll;  // of the candidates at the border `need` are kept
  while (n_c != k) {  // #{r <= hi} >= k
    border = lo + (hi - lo) / 2;
    const uint32_t n = upto(border);
    if (n == k) break;
    if (lo == hi) {
      need = k - (border == 0 ? 0u : upto(border - 1));
      break;
    }
    if (n < k) lo = border + 1;
    else hi = border;
  }
  if (!ORDERED && need != kAll) {
    for (uint32_t i = lane; i < n_c; i += kWave) {
      uint32_t rank = 0;
      if (slot[i].r == border)
        for (uint32_t q = 0; q < n_c; ++q) rank += slot[q].r == border && slot[q].j < slot[i].j;
      slot[i].keep = rank < need;
    }
    settle();
  }
  uint32_t placed = 0, ties = 0;
  for (uint32_t base = 0; base < n_c; base += kWave) {
    const uint32_t i = base + lane;
    const NsSlot c = slot[i];
    bool keep = i < n_c && c.r <= border;
    if (need != kAll && ORDERED) {
      const uint64_t m = ballot64(keep && c.r == border);
      if (c.r == border) keep = keep && ties + lanes_below(m) < need;
      ties += (uint32_t)__popcll(m);
    } else if (need != kAll && c.r == border) {
      keep = keep && c.keep != 0;
    }
    const uint64_t m = ballot64(keep);
    const uint32_t place = placed + lanes_below(m);
    placed += (uint32_t)__popcll(m);
    if (ORDERED) {
      if (keep) {
        put_edge(edges, o, place, c.t, beg + c.j);
      }
    } else {
      settle();
      if (keep) {  // (place <= i: that slot was read in this round or before)
        slot[place].j = c.j;
        slot[place].t = c.t;
      }
      settle();
    }
  }
  if (ORDERED) return;
  for (uint32_t base = 0; base < k; base += kWave) {
    const uint32_t i = base + lane;
    const uint32_t my_j = slot[i].j;
    uint32_t place = 0;
#pragma unroll 4
    for (uint32_t q = 0; q < k; ++q) place += slot[q].j < my_j;
    if (i < k) {
      put_edge(edges, o, place, slot[i].t, beg + my_j);
    }
  }
}
// The lanes of the k smallest r among those of `has` (popcount > k >= 1), or 0 where equal variates stand across the border.  The
// variates of a shrinking set of lanes are tried as the border, two vector instructions each, four tries for 18 lanes: ranking
// all of them takes two per lane.
__device__ __forceinline__ uint64_t ns_smallest(uint32_t r, uint64_t has, uint32_t k) {
  uint64_t open = has, upto;  // the k-th smallest is one of `open`
  for (;;) {
    const uint32_t border = (uint32_t)__builtin_amdgcn_readlane((int)r, __builtin_ctzll(open));
    const uint64_t below = compare_mask(r < border) & has;
    upto = compare_mask(r <= border) & has;
    if ((uint32_t)__popcll(below) >= k) open &= below;
    else if ((uint32_t)__popcll(upto) < k) open &= ~upto;
    else return (uint32_t)__popcll(upto) == k ? upto : 0ull;
  }
}
// (after ns_collect_plain: the candidates stand in list order, and their variates are evaluated here)
__device__ __forceinline__ void ns_rank_write_plain(uint32_t n_c, uint32_t k, uint32_t bound, const NsKeys& K, NsSlot* slot, int64_t o, int64_t beg, EdgeOut edges) {
  const uint32_t lane = (uint32_t)lane_id();
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  if (n_c <= (uint32_t)kWave) {
    const uint32_t j = slot[lane].j;  // (cap >= 256: the slots behind the candidates are there)
    const int32_t t = slot[lane].t;
    uint64_t kept = low_lanes(n_c);
    if (n_c != k) {
      const uint32_t r = ns_uniform(K, (uint32_t)t);
      kept = ns_smallest(r, kept, k);
      if (kept == 0) {  // by variate and position
        slot[lane].r = r;
        __builtin_amdgcn_wave_barrier();
        __threadfence_block();
        kept = ballot64(lane < n_c && ns_rank_of(n_c, slot, ((uint64_t)r << 32) | j) < k);
      }
    }
    if (lane_in(kept)) {
      const uint32_t place = lanes_below(kept);
      put_edge(edges, o, place, t, beg + j);
    }
    return;
  }
  for (uint32_t i = lane; i < n_c; i += kWave) slot[i].r = ns_uniform(K, (uint32_t)slot[i].t);
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  ns_rank_write_many<true>(n_c, k, bound, slot, o, beg, edges);
}
__device__ __forceinline__ void ns_rank_write(uint32_t n_c, uint32_t k, uint32_t bound, NsSlot* slot, int64_t o, int64_t beg, EdgeOut edges) {
  const uint32_t lane = (uint32_t)lane_id();
  if (n_c <= (uint32_t)kWave) ns_pad(n_c, slot);
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  if (n_c > (uint32_t)kWave) {
    ns_rank_write_many<false>(n_c, k, bound, slot, o, beg, edges);
    return;
  }
  const bool has = lane < n_c;
  const uint64_t my_key = has ? slot_key(slot + lane) : ~0ull;
  const uint32_t my_j = (uint32_t)my_key;
  const int32_t my_t = has ? slot[lane].t : 0;
  const bool keep = ns_rank(n_c, slot, my_key) < k && has;
  const uint64_t kept = ballot64(keep);
  uint32_t place = 0;  // kept candidates in front of this one in the list
  uint64_t rest = kept;
  while (rest != 0) {
    const int q = __builtin_ctzll(rest);
    rest &= rest - 1;
    place += (uint32_t)__builtin_amdgcn_readlane((int)my_j, q) < my_j;
  }
  if (keep) {
    put_edge(edges, o, place, my_t, beg + my_j);
  }
}

// Selection of the k smallest (R, j) among d > k neighbours, one wave per destination:
//   1. one pass over the list collects, in LDS, the candidates with R <= bound, where bound is chosen so that about
//      `target` of them are expected (target > k, target < cap);
//   2. if fewer than k or more than cap candidates turn up, the bound is bisected and the pass repeated (rare);
//   3. every candidate's rank by (R, j) among the candidates is counted: ranks below k are kept;
//   4. every kept candidate's place is the number of kept candidates in front of it in the list.
//
// The degree distribution is heavy-tailed and a wave takes a whole list, so the lists longer than long_min entries
// are not left where the destination order puts them (a hub that starts late would keep the kernel waiting for one
// wave): k_ns_count queues them, the waves of the first long_blocks blocks of the grid take one queued list each (the
// queue's length is read from device memory), and the other blocks take the destinations in order and skip the queued
// ones.

// The next bound to try for a list that turned up n_c candidates, fewer than k or more than cap (false: there is none)
__device__ __forceinline__ bool ns_next_bound(uint32_t n_c, uint32_t k, uint32_t* lo, uint32_t* hi, uint32_t* bound) {
  if (n_c < k) {
    if (*bound == 0xFFFFFFFFu) return false;
    *lo = *bound + 1;
  } else {  // cannot be bracketed (more than cap - k equal variates): report instead of guessing
    if (*bound == 0) return false;
    *hi = *bound - 1;
  }
  if (*lo > *hi) return false;
  // too few and no upper failure yet: double the bound (a midpoint of the whole range would flood the buffer)
  if (*hi == 0xFFFFFFFFu && n_c < k) *bound = *bound < 0x7FFFFFFFu ? 2 * *bound + 1 : 0xFFFFFFFFu;
  else *bound = *lo + (*hi - *lo) / 2;
  return true;
}

// (Pointers that say they do not overlap and no test for a tag: without either, every load waits for the store before it.  10 thousand
// lists of 900 entries, fanout 1,000: the fill 142 us, 94 so.)
__device__ __forceinline__ void ns_copy_list(const int32_t* __restrict__ from, uint32_t d, int64_t beg, int32_t* __restrict__ col, int64_t* __restrict__ eid) {
#pragma unroll 8
  for (uint32_t j = (uint32_t)lane_id(); j < d; j += kWave) {
    col[j] = from[j];
    eid[j] = beg + j;
  }
}

// The lists that are kept whole, of a wave's destinations, 64 >> each_log2 lanes and g of each: short ones together, those longer than
// 4 entries for each of the lanes one after the other by the whole wave.  (Steps over 90 thousand lists of 30 to
// 1,500 entries 1.99 ms with eight lanes for each, 1.51 so; a thousand lists of a papers100M shape 74 us with a load at a time, 61 with
// eight in flight.)
__device__ __forceinline__ void ns_copy_whole(const int32_t* __restrict__ g_indices, const NsRecord& g, int64_t o, bool whole, uint32_t k, int each_log2,
                                              EdgeOut edges) {
  const uint32_t lane = (uint32_t)lane_id(), lanes = 64u >> each_log2, sub = lane & (lanes - 1);
  if (whole && g.d <= 4 * lanes) {
    for (uint32_t j = sub; j < g.d; j += lanes) {
      put_edge(edges, o, j, (g_indices + g.beg)[j], g.beg + j);
    }
  }
  if (k <= 4 * lanes) return;
  auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
  auto of64 = [&](int64_t x, int q) { return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)x >> 32), q) << 32) | of((uint32_t)x, q)); };
  for (uint64_t todo = ballot64(whole && sub == 0 && g.d > 4 * lanes); todo != 0; todo &= todo - 1) {
    const int at = __builtin_ctzll(todo);
    const uint32_t d = of(g.d, at);
    const int64_t beg = of64(g.beg, at), to = of64(o, at);
    if (edges.tag == nullptr) ns_copy_list(g_indices + beg, d, beg, edges.col + to, edges.eid + to);
    else for (uint32_t j = lane; j < d; j += kWave) put_edge(edges, to, j, (g_indices + beg)[j], beg + j);
  }
}

// c = 0.  A wave takes `each` neighbouring destinations (at most 64; the dispatcher starts one-wave blocks at some 5 per ns, 150 us
// for 745 thousand that do nothing).  Their records come in one load, a destination per lane; lists no longer than the fanout
// are copied together, 64 / each lanes for each; the others go one after the other through the whole wave, the next one's entries
// requested before this one's candidates are selected.  Last layer of a quarter of the papers100M shape, 717 thousand
// destinations, 380 M entries: 494 us with a wave for each, 225 M vector and 191 M scalar instructions; 400 now, with 144 M
// and 159 M (the entries alone, at the rate of a copy: 310).
__global__ __launch_bounds__(kWave, 8) void k_ns_fill(const int32_t* __restrict__ g_indices, const NsRecord* __restrict__ rec, uint32_t n_dst, uint32_t k,
                                                    uint32_t cap, LayerKeys keys, int64_t* indptr, int64_t first, int tile_log2,
                                                    EdgeOut edges, int64_t edge_limit, Ctl* ctl,
                                                    uint32_t long_min, const uint32_t* __restrict__ long_list,
                                                    const uint32_t* __restrict__ n_long, int long_blocks, Dealing deal, uint32_t stretch) {
  extern __shared__ __align__(16) uint32_t lds_words[];  // cap slots, and one per lane
  NsSlot* slot = reinterpret_cast<NsSlot*>(lds_words);
  const uint32_t lane = (uint32_t)lane_id();
  uint32_t w0, n_mine = 1, skip_above = 0xFFFFFFFFu;
  int each_log2 = 0;
  if ((int)blockIdx.x < long_blocks) {  // the first blocks: a queued long list each (the queue's length is read from device memory)
    uint32_t n_queued = *n_long;
    if (n_queued > n_dst) n_queued = n_dst;  // (holds by construction; keeps every access inside the queue regardless)
    if (blockIdx.x >= n_queued) return;
    w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)long_list[blockIdx.x]);
  } else {
    w0 = (uint32_t)deal.first_list(blockIdx.x - (uint32_t)long_blocks, &each_log2);
    n_mine = 1u << each_log2;
    if (long_min != 0) skip_above = long_min;
  }
  if (w0 >= n_dst) return;
  if (n_mine > n_dst - w0) n_mine = n_dst - w0;
  // a lane's destination: its number among the wave's in the copying below, and so, shifted, where the loop finds it
  const uint32_t w = w0 + ((lane >> (6 - each_log2)) < n_mine ? lane >> (6 - each_log2) : n_mine - 1);
  const NsRecord g = rec[w];
  const int64_t o = ns_offset(indptr, first + w, tile_log2), o_end = o + (g.d < k ? g.d : k);
  const bool mine = (lane >> (6 - each_log2)) < n_mine, speaks = mine && (lane & ((64u >> each_log2) - 1)) == 0;
  // (longer than skip_above: queued, one of the first waves takes it)
  if (speaks && (g.d <= k || g.d <= skip_above)) ns_settle_offset(indptr, first + w, tile_log2, o);
  const bool live = mine && g.d != 0 && o_end <= edge_limit;  // (no room: the caller redoes the layer)
  ns_copy_whole(g_indices, g, o, live && g.d <= k, k, each_log2, edges);
  if (k > kNsMaxSelect) return;  // degrees above a fanout that the candidate buffer cannot serve: left to k_ns_fill_wide
  uint64_t todo = ballot64(live && speaks && g.d > k && g.d <= skip_above);
  if (todo == 0) return;
  auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
  auto of64 = [&](int64_t x, int q) { return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)x >> 32), q) << 32) | of((uint32_t)x, q)); };
  int at = __builtin_ctzll(todo);
  uint32_t d = of(g.d, at), bound = of(g.bound, at), mid = of(g.mid, at);
  int64_t beg = of64(g.beg, at), o_this = of64(o, at);
  uint32_t lo = 0, hi = 0xFFFFFFFFu, attempt = 0;  // bisection bracket on the bound, used only after a failed pass
  uint32_t j0 = 0, n_c = 0;                        // entries looked at in earlier stretches of the list, candidates so far
  const uint32_t head = vector_copy(keys.Ka[4]), tail = vector_copy(keys.Ka[3]);
  for (ListReader<kFillGroups> L(g_indices + beg, d < stretch ? d : stretch);;) {
    const NsKeys K{head, vector_copy(mid), tail};
    n_c = ns_collect_plain(L, j0, bound, K, slot, cap, n_c);
    const uint32_t found = n_c;
    const int64_t o_done = o_this, beg_done = beg;
    const uint32_t bound_done = bound;
    bool select = false;
    if (d - j0 > stretch) {  // the list's next stretch
      j0 += stretch;
    } else if ((n_c < k || n_c > cap) && ++attempt < 40 && ns_next_bound(n_c, k, &lo, &hi, &bound)) {  // the list once more
      j0 = n_c = 0;
    } else {  // the next list
      select = n_c >= k && n_c <= cap;
      if (!select && lane == 0) atomicOr(&ctl->err_capacity, 1);
      todo &= todo - 1;
      at = todo != 0 ? __builtin_ctzll(todo) : 0;
      d = todo != 0 ? of(g.d, at) : 0u;
      bound = of(g.bound, at);
      mid = of(g.mid, at);
      beg = of64(g.beg, at);
      o_this = of64(o, at);
      lo = j0 = n_c = attempt = 0;
      hi = 0xFFFFFFFFu;
    }
    L = ListReader<kFillGroups>(g_indices + beg + j0, d - j0 < stretch ? d - j0 : stretch);
    if (select) ns_rank_write_plain(found, k, bound_done, K, slot, o_done, beg_done, edges);
    if (todo == 0) break;
    __builtin_amdgcn_wave_barrier();
  }
}

// c > 0: one destination with exact variates
template <bool VEC4>
__device__ __forceinline__ void ns_redo_one(int64_t w, int wib, uint32_t* lds_words, NsQueue* queue, const int32_t* __restrict__ g_indices,
                                            const NsRecord* __restrict__ rec, const NsBlendThr* __restrict__ bthr, uint32_t k, uint32_t cap,
                                            const VariateParams& vp, const int64_t* __restrict__ eptr, EdgeOut edges, int64_t edge_limit, Ctl* ctl) {
  const int64_t o = eptr[w];
  const NsRecord g = rec[w];
  if (g.d <= k || k > kNsMaxSelect) return;  // (never marked)
  if (o + k > edge_limit) return;  // (by its own record: eptr[w + 1] may be the next slice's, whose offsets are not settled yet)
  NsSlot* slot = reinterpret_cast<NsSlot*>(lds_words) + (size_t)wib * cap;  // [cap]
  const uint32_t sigma_a = ns_sigma(vp.K.Ka, (uint32_t)g.s), sigma_b = ns_sigma(vp.K.Kb, (uint32_t)g.s);
  uint32_t lo = 0, hi = 0xFFFFFFFFu, bound = g.bound;
  NsBlendThr bt = bthr[w];
  uint32_t n_c = 0;
  for (int attempt = 0; attempt < 40; ++attempt) {
    n_c = ns_collect<VEC4>(g_indices, g.beg, g.d, bound, bt, vp, sigma_a, sigma_b, slot, cap, queue);
    if (n_c >= k && n_c <= cap) break;
    if (!ns_next_bound(n_c, k, &lo, &hi, &bound)) { n_c = 0; break; }
    bt = ns_blend_thresholds(bound, vp.cw, vp.sw);  // (every lane computes the same)
    __builtin_amdgcn_wave_barrier();
  }
  if (n_c < k || n_c > cap) {
    if (lane_id() == 0) atomicOr(&ctl->err_capacity, 1);
    return;
  }
  ns_rank_write(n_c, k, bound, slot, o, g.beg, edges);
}

// c > 0: the destinations that the two kernels below leave over.  A wave looks at 2^lists_log2 marks at once.  (Six waves per
// SIMD, 80 registers and some scratch memory, and the exact blend as a function in the place of 31 copies: with three
// waves the lists took 3.0 ms in the place of 1.86.)
template <bool VEC4>
__global__ __launch_bounds__(kWave, 6) void k_ns_redo(const int32_t* __restrict__ g_indices,
                                                    const NsRecord* __restrict__ rec, const NsBlendThr* __restrict__ bthr,
                                                    int64_t n_dst, uint32_t k,
                                                    uint32_t cap, int waves_per_block, VariateParams vp,
                                                    const int64_t* __restrict__ eptr, EdgeOut edges, int64_t edge_limit, Ctl* ctl,
                                                    const uint32_t* __restrict__ n_cand, int lists_log2) {
  extern __shared__ __align__(16) uint32_t lds_words[];  // per wave as above, and a queue behind all of them
  NsQueue* queues = reinterpret_cast<NsQueue*>(lds_words + (size_t)waves_per_block * cap * 4);
  const int wib = uniform_wave_in_block();
  if (wib >= waves_per_block) return;
  const int64_t w0 = ((int64_t)blockIdx.x * waves_per_block + wib) << lists_log2;
  const int lane = lane_id();
  uint64_t left = ballot64(lane < (1 << lists_log2) && w0 + lane < n_dst && n_cand[w0 + lane] == kNsRedo);
  while (left != 0) {
    const int64_t w = w0 + __builtin_ctzll(left);
    left &= left - 1;
    ns_redo_one<VEC4>(w, wib, lds_words, &queues[wib], g_indices, rec, bthr, k, cap, vp, eptr, edges, edge_limit, ctl);
    __builtin_amdgcn_wave_barrier();
  }
}

// ---- c > 0 in two kernels ----------------------------------------------------------------------------------------
// The exact blend (two inverse normal distribution functions and one forward, in fp64) needs four times the registers of
// the traversal and is wanted for a few dozen candidates per list only.  So the traversal kernel stops at the fp32
// filter and leaves what passes, (list position, vertex) pairs, in a row of row_cap entries per destination; a second
// kernel evaluates those exactly, drops the ones above the bound and selects.  A destination whose row overflows, or
// that ends up with fewer than k candidates (about one in 10^4), is marked and done again by k_ns_redo, which adjusts
// the bound.
//
// The traversal's waves take destinations as k_ns_fill's do, which says what its parts are for; its candidates go through the
// queue of a blended scan, which lives across the wave's lists (with a list to itself a wave of the fp32 stage had a quarter of its
// lanes at work where 15 candidates are expected).
struct NsSink {
  StageEntry* rows;  // of the wave's first destination
  uint32_t row_cap, shift;
  __device__ __forceinline__ void take(BlendQueue<true>* queue, int, bool there, const StageEntry& e, uint32_t slot, uint32_t, uint32_t, float est) {
    if (there && est <= queue->lim2[slot]) {
      const uint32_t at = atomicAdd(&queue->own[slot], 1u);
      if (at < row_cap) rows[(size_t)(slot >> shift) * row_cap + at] = e;
    }
  }
};

__global__ __launch_bounds__(kWave, 7) void k_ns_collect(const int32_t* __restrict__ g_indices, const NsRecord* __restrict__ rec,
                                                         const NsBlendThr* __restrict__ bthr, uint32_t n_dst, uint32_t k, LayerKeys keys, float cw,
                                                         float sw, int64_t* indptr, int64_t first, int tile_log2, EdgeOut edges, int64_t edge_limit, StageEntry* __restrict__ rows, uint32_t row_cap,
                                                         uint32_t* __restrict__ n_cand, uint32_t long_min, const uint32_t* __restrict__ long_list,
                                                         const uint32_t* __restrict__ n_long, int long_blocks, Dealing deal, uint32_t stretch) {
  __shared__ BlendQueue<true> queue;
  const uint32_t lane = (uint32_t)lane_id();
  uint32_t w0, n_mine = 1, skip_above = 0xFFFFFFFFu;
  int each_log2 = 0;
  if ((int)blockIdx.x < long_blocks) {
    uint32_t n_queued = *n_long;
    if (n_queued > n_dst) n_queued = n_dst;  // (holds by construction; keeps every access inside the queue regardless)
    if (blockIdx.x >= n_queued) return;
    w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)long_list[blockIdx.x]);
  } else {
    w0 = (uint32_t)deal.first_list(blockIdx.x - (uint32_t)long_blocks, &each_log2);
    n_mine = 1u << each_log2;
    if (long_min != 0) skip_above = long_min;
  }
  if (w0 >= n_dst) return;
  if (n_mine > n_dst - w0) n_mine = n_dst - w0;
  const uint32_t lanes = 64u >> each_log2, sub = lane & (lanes - 1), number = lane >> (6 - each_log2);
  const uint32_t w = w0 + (number < n_mine ? number : n_mine - 1);
  const NsRecord g = rec[w];
  const NsBlendThr bt = bthr[w];
  const int64_t o = ns_offset(indptr, first + w, tile_log2), o_end = o + (g.d < k ? g.d : k);
  const bool mine = number < n_mine && (g.d <= k || g.d <= skip_above), speaks = mine && sub == 0;  // (the others: queued)
  if (speaks) ns_settle_offset(indptr, first + w, tile_log2, o);
  const bool live = mine && g.d != 0 && o_end <= edge_limit;  // (no room: the caller redoes the layer)
  ns_copy_whole(g_indices, g, o, live && g.d <= k, k, each_log2, edges);
  const bool sampled = live && g.d > k && k <= kNsMaxSelect;  // (a larger fanout: k_ns_fill_wide)
  BlendScan<1, true, NsSink> S;
  S.queue = &queue;
  S.set_keys(0, keys);
  S.cwf = cw;
  S.swf = sw;
  S.sink = NsSink{rows + (size_t)w0 * row_cap, row_cap, (uint32_t)(6 - each_log2)};
  const uint32_t mid_a = g.mid, mid_b = ns_mid(keys.Kb, ns_sigma(keys.Kb, (uint32_t)g.s));
  const uint32_t my_a1 = bt.a1 | 0xFFFFu, my_a2 = bt.a2 | 0xFFFFu, my_b2 = bt.b2 | 0xFFFFu;
  queue.mid_a[lane] = mid_a;
  queue.mid_b[lane] = mid_b;
  queue.lim2[lane] = bt.lim2;
  queue.own[lane] = 0;
  const uint32_t together = each_log2 != 0 ? 2 * lanes : 0;
  if (ballot64(sampled && g.d <= together) != 0) {
    uint32_t t[4] = {0, 0, 0, 0};
    uint64_t m[4] = {0, 0, 0, 0};
    S.mid_a = mid_a;
    S.mid_b = mid_b;
    bool in[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      in[r] = sampled && g.d <= together && sub + r * lanes < g.d;
      if (in[r]) t[r] = (uint32_t)(g_indices + g.beg)[sub + r * lanes];
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) m[r] = S.passes(0, t[r], my_a1, my_a2, my_b2) & ballot64(in[r]);
    S.join(0, t, m, sub, lanes, lane & ~(lanes - 1));
  }
  uint64_t todo = ballot64(sampled && sub == 0 && g.d > together);
  if (todo != 0) {
    auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
    auto of64 = [&](int64_t x, int q) { return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)x >> 32), q) << 32) | of((uint32_t)x, q)); };
    int at = __builtin_ctzll(todo);
    uint32_t d = of(g.d, at), j0 = 0, a1[1], a2[1], b2[1];
    int64_t beg = of64(g.beg, at);
    auto take = [&]() {
      a1[0] = of(my_a1, at);
      a2[0] = of(my_a2, at);
      b2[0] = of(my_b2, at);
      S.mid_a = vector_copy(of(mid_a, at));
      S.mid_b = vector_copy(of(mid_b, at));
    };
    take();
    for (ListReader<> L(g_indices + beg, d < stretch ? d : stretch);;) {
      S.collect(L, j0, (uint32_t)at, a1, a2, b2);
      if (d - j0 > stretch) {  // the list's next stretch
        j0 += stretch;
      } else {
        todo &= todo - 1;
        if (todo == 0) break;
        at = __builtin_ctzll(todo);
        d = of(g.d, at);
        beg = of64(g.beg, at);
        j0 = 0;
        take();
      }
      L = ListReader<>(g_indices + beg + j0, d - j0 < stretch ? d - j0 : stretch);
    }
  }
  S.flush();
  if (speaks) {  // (0: nothing left to do; too few even before the exact test, or no room in the row: k_ns_redo)
    const uint32_t n = queue.own[lane];
    n_cand[w] = !sampled ? 0u : n < k || n > row_cap ? kNsRedo : n;
  }
}

// One destination's candidates, by the whole wave (n = n_cand[w], not 0).
__device__ __forceinline__ void ns_select_one(int64_t w, uint32_t n, NsSlot* slot, const NsRecord* __restrict__ rec, uint32_t k, const VariateParams& vp,
                                              const int64_t* __restrict__ eptr, EdgeOut edges,
                                              const StageEntry* __restrict__ rows, uint32_t row_cap, uint32_t* __restrict__ n_cand,
                                              const NsBlendThr* __restrict__ bthr) {
  const uint32_t lane = (uint32_t)lane_id();
  const NsRecord g = rec[w];
  const uint32_t sigma_a = ns_sigma(vp.K.Ka, (uint32_t)g.s), sigma_b = ns_sigma(vp.K.Kb, (uint32_t)g.s);
  const StageEntry* row = rows + (size_t)w * row_cap;
  if (n <= (uint32_t)kWave) {
    // The usual case, one candidate per lane.  Only the set of the k smallest matters, so the fp32 blend (within
    // `allow` / 10 of the exact one in normal space) decides wherever it can: with e_k the k-th smallest estimate and
    // m = 2 allow, a candidate below e_k - m is among the k smallest, one above e_k + m is not, and the exact variates
    // are needed only to choose among those in between, and only if there are more of them than places left.
    const bool has = lane < n;
    StageEntry c{0, 0xFFFFFFFFu};
    if (has) c = row[lane];
    const uint32_t u1 = keyed_uniform<true>(vp.K.Ka, (uint32_t)c.t, sigma_a), u2 = keyed_uniform<true>(vp.K.Kb, (uint32_t)c.t, sigma_b);
    const float est = has ? __builtin_fmaf((float)vp.cw, approx_phi_inv_f32(u1), (float)vp.sw * approx_phi_inv_f32(u2)) : __builtin_inff();
    // rank by (estimate, lane): the estimates (finite for every candidate) go to LDS as 64-bit keys, their bits mapped so
    // that unsigned order is numeric order, and every lane reads them back as broadcasts (as in ns_rank_write)
    const uint32_t eb = __float_as_uint(est);
    const uint64_t est_key = ((uint64_t)(eb ^ ((uint32_t)((int32_t)eb >> 31) | 0x80000000u)) << 32) | lane;
    if (has) { slot[lane].j = lane; slot[lane].r = (uint32_t)(est_key >> 32); }
    ns_pad(n, slot);
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
    const uint32_t rank_est = ns_rank(n, slot, est_key);
    const uint64_t kth = ballot64(has && rank_est == k - 1);  // exactly one lane (n >= k)
    const float e_k = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(est), __builtin_ctzll(kth)));
    const float allow = (float)((vp.cw + vp.sw) * kPhiInvF32Allow + 2.0 * kBlendAbsWiden);
    const float m = 2.0f * allow;
    // outside |e_k| <= 5 two different blends can share a 32-bit variate, and the estimate says nothing about ties; and
    // e_k must lie safely below what the traversal's filter let through, or a neighbour that it dropped could belong
    // to the k smallest
    if (!(e_k >= -5.0f && e_k <= 5.0f) || !(e_k + m <= bthr[w].lim2 - m)) {
      if (lane == 0) n_cand[w] = kNsRedo;
      return;
    }
    const bool in = has && est < e_k - m;
    const bool und = has && !in && est <= e_k + m;
    const uint64_t und_mask = ballot64(und);
    const uint32_t need = k - (uint32_t)__popcll(ballot64(in));  // >= 1: the k-th itself is undecided
    bool keep = in || und;
    if ((uint32_t)__popcll(und_mask) > need) {  // wave-uniform
      uint32_t R = 0;
      if (und) R = blend_exact(u1, u2, vp.cw, vp.sw);
      const uint64_t my_key = ((uint64_t)R << 32) | c.j;
      uint32_t rank_u = 0;
      uint64_t rest = und_mask;
      while (rest != 0) {
        const int q = __builtin_ctzll(rest);
        rest &= rest - 1;
        const uint64_t key = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)R, q) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)c.j, q);
        rank_u += key < my_key;
      }
      keep = in || (und && rank_u < need);
    }
    const uint64_t kept = ballot64(keep);
    uint32_t place = 0;  // kept candidates in front of this one in the list
    uint64_t rest = kept;
    while (rest != 0) {
      const int q = __builtin_ctzll(rest);
      rest &= rest - 1;
      place += (uint32_t)__builtin_amdgcn_readlane((int)c.j, q) < c.j;
    }
    if (keep) {
      const int64_t o = eptr[w];
      put_edge(edges, o, place, c.t, g.beg + c.j);
    }
    return;
  }
  uint32_t n_c = 0;  // candidates with R <= bound, compacted into LDS
  for (uint32_t base = 0; base < n; base += kWave) {
    const uint32_t i = base + lane;
    StageEntry c{0, 0u};
    uint32_t R = 0;
    bool in = false;
    if (i < n) {
      c = row[i];
      const uint32_t u1 = keyed_uniform<true>(vp.K.Ka, (uint32_t)c.t, sigma_a), u2 = keyed_uniform<true>(vp.K.Kb, (uint32_t)c.t, sigma_b);
      R = blend_exact(u1, u2, vp.cw, vp.sw);
      in = R <= g.bound;
    }
    const uint64_t mask = ballot64(in);
    const uint32_t at = n_c + lanes_below(mask);
    if (in) { slot[at].j = c.j; slot[at].r = R; slot[at].t = c.t; }  // (n <= cap)
    n_c += (uint32_t)__popcll(mask);
  }
  if (n_c < k) {
    if (lane == 0) n_cand[w] = kNsRedo;
    return;
  }
  ns_rank_write(n_c, k, g.bound, slot, eptr[w], g.beg, edges);
}


// A wave takes 2^each_log2 destinations, 2^(6 - group_log2) of them at a time with 2^group_log2 lanes each; those with more candidates
// than that follow one by one.  (As ns_select_one, whose comments say why; a destination per wave had 15 to 35 of its lanes at
// work, and starting a wave for each took a third of the time.)
__global__ __launch_bounds__(kWave, 6) void k_ns_select(const NsRecord* __restrict__ rec, int64_t n_dst, uint32_t k, VariateParams vp,
                                                     const int64_t* __restrict__ eptr, EdgeOut edges,
                                                     const StageEntry* __restrict__ rows, uint32_t row_cap, uint32_t* __restrict__ n_cand,
                                                     const NsBlendThr* __restrict__ bthr, int each_log2, int group_log2) {
  extern __shared__ __align__(16) uint32_t lds_words[];  // slots for ns_select_one, at least kWave
  NsSlot* slot = reinterpret_cast<NsSlot*>(lds_words);
  uint64_t* key_of = reinterpret_cast<uint64_t*>(lds_words);  // [kWave] the groups' keys, then positions
  uint32_t* j_of = lds_words;
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t G = 1u << group_log2, at0 = lane & ~(G - 1), sub = lane & (G - 1);
  const uint64_t group = low_lanes(G) << at0;
  const int64_t w_first = (int64_t)blockIdx.x << each_log2;
  const uint32_t n_mine = n_dst - w_first < ((int64_t)1 << each_log2) ? (uint32_t)(n_dst - w_first) : 1u << each_log2;
  const float cwf = (float)vp.cw, swf = (float)vp.sw;
  const float allow = (float)((vp.cw + vp.sw) * kPhiInvF32Allow + 2.0 * kBlendAbsWiden);
  const float m = 2.0f * allow;
  auto settle = [] {
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
  };
  // What is known of the wave's destinations, one per lane, all of it requested together: with the requests of every step waiting
  // for one another 250 thousand destinations with 15 candidates each took 49 us, now 44 (and before that, with a wave each, 112).
  const int64_t w_lane = w_first + (lane < n_mine ? lane : n_mine - 1);
  uint32_t all_n = n_cand[w_lane];
  if (all_n == kNsRedo || lane >= n_mine) all_n = 0;  // (0: done by the collecting kernel)
  const NsRecord all_rec = rec[w_lane];
  const float all_lim2 = bthr[w_lane].lim2;
  const int64_t all_o = eptr[w_lane];
  const uint32_t all_sa = ns_sigma(vp.K.Ka, (uint32_t)all_rec.s), all_sb = ns_sigma(vp.K.Kb, (uint32_t)all_rec.s);
  auto share = [](uint32_t x, uint32_t from) { return (uint32_t)__shfl((int)x, (int)from, kWave); };
  auto share64 = [&](int64_t x, uint32_t from) { return (int64_t)(((uint64_t)share((uint32_t)((uint64_t)x >> 32), from) << 32) | share((uint32_t)x, from)); };
  const uint32_t step = 64u >> group_log2;
  auto fetch = [&](uint32_t i0) {  // the candidates of the step that begins with the wave's destination i0
    const uint32_t i = i0 + (lane >> group_log2);
    const uint32_t n = share(all_n, i < n_mine ? i : i0);  // (every lane takes part)
    StageEntry c{0, 0xFFFFFFFFu};
    if (i < n_mine && n <= G && sub < n) c = rows[(size_t)(w_first + i) * row_cap + sub];
    return c;
  };
  StageEntry next = fetch(0);
  for (uint32_t i0 = 0; i0 < n_mine; i0 += step) {
    const uint32_t i = i0 + (lane >> group_log2), from = i < n_mine ? i : i0;
    const int64_t w0 = w_first + i0, w = w_first + i;
    uint32_t n = share(all_n, from);
    if (i >= n_mine) n = 0;
    uint64_t many = ballot64(n > G && sub == 0);
    if (n > G) n = 0;
    const StageEntry c = next;
    if (i0 + step < n_mine) next = fetch(i0 + step);
    if (ballot64(n != 0) != 0) {
      const bool has = sub < n;
      const uint32_t sigma_a = share(all_sa, from), sigma_b = share(all_sb, from);
      const uint32_t u1 = keyed_uniform<true>(vp.K.Ka, (uint32_t)c.t, sigma_a), u2 = keyed_uniform<true>(vp.K.Kb, (uint32_t)c.t, sigma_b);
      const float est = __builtin_fmaf(cwf, approx_phi_inv_f32(u1), swf * approx_phi_inv_f32(u2));
      const uint32_t eb = __float_as_uint(est);
      const uint64_t est_key = has ? ((uint64_t)(eb ^ ((uint32_t)((int32_t)eb >> 31) | 0x80000000u)) << 32) | lane : ~0ull;
      uint32_t most = 0;  // candidates of the largest group
      for (uint32_t q = 0; q < (uint32_t)kWave; q += G) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)n, (int)q);
        most = x > most ? x : most;
      }
      // a group's keys, one after the other: every lane counts those below its own (what stands behind the group's candidates is above all)
      auto rank_of = [&](uint64_t key) {
        settle();
        key_of[lane] = key;
        settle();
        uint32_t rank = 0;
        for (uint32_t q = 0; q < most; q += 4)
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) rank += key_of[at0 + q + e] < key;
        return rank;
      };
      const uint32_t rank_est = rank_of(est_key);
      // the k-th smallest estimate
      settle();
      if (has && rank_est == k - 1) reinterpret_cast<float*>(lds_words)[at0] = est;
      settle();
      const float e_k = n != 0 ? reinterpret_cast<float*>(lds_words)[at0] : 0.0f;
      const float lim2 = __shfl(all_lim2, (int)from, kWave);
      const bool sure = n != 0 && e_k >= -5.0f && e_k <= 5.0f && e_k + m <= lim2 - m;
      if (n != 0 && !sure && sub == 0) n_cand[w] = kNsRedo;
      const bool in = has && sure && est < e_k - m;
      const bool und = has && sure && !in && est <= e_k + m;
      const uint32_t n_in = (uint32_t)__popcll(ballot64(in) & group), n_und = (uint32_t)__popcll(ballot64(und) & group);
      const bool choose = und && n_und > k - n_in;
      bool keep = in || und;
      if (ballot64(choose) != 0) {
        uint32_t R = 0;
        if (choose) R = blend_exact(u1, u2, vp.cw, vp.sw);
        const uint32_t rank_u = rank_of(choose ? ((uint64_t)R << 32) | c.j : ~0ull);
        if (choose) keep = rank_u < k - n_in;
      }
      // a kept candidate's place is the number of kept ones in front of it in the list
      const uint32_t number = lanes_below(ballot64(keep) & group);
      settle();
      if (keep) j_of[at0 + number] = c.j;  // (k of them, where there are any)
      settle();
      const int64_t o = share64(all_o, from), beg = share64(all_rec.beg, from);
      if (keep) {
        uint32_t place = 0;
        for (uint32_t q = 0; q < k; ++q) place += j_of[at0 + q] < c.j;
        put_edge(edges, o, place, c.t, beg + c.j);
      }
    }
    while (many != 0) {
      const int q = __builtin_ctzll(many);
      many &= many - 1;
      const int64_t w_q = w0 + (q >> group_log2);
      settle();
      ns_select_one(w_q, (uint32_t)__builtin_amdgcn_readlane((int)all_n, (int)(w_q - w_first)), slot, rec, k, vp, eptr, edges, rows, row_cap, n_cand, bthr);
    }
    settle();
  }
}

// ---- fanouts above kNsMaxSelect ----------------------------------------------------------------------------------
// The k smallest (R, j) of a list longer than k, for a k that the candidate arrays in LDS cannot hold: no candidates are
// stored at all.  A bisection over the 32-bit variates finds the smallest B with #{R <= B} >= k (one pass over the list
// per step, 32 steps); everything below B is kept, and of the entries with R = B (normally one) the first
// k - #{R < B} in list order.  The last pass writes the kept entries in adjacency order, 64 at a time, each at the
// running count plus its rank in the ballot.  One wave per destination; 34 passes over a list, variates recomputed in
// each: a path for the rare call with a fanout in the thousands, not for speed.
template <bool BLEND>
__global__ __launch_bounds__(kBlock) void k_ns_fill_wide(const int32_t* __restrict__ g_indices, const NsRecord* __restrict__ rec,
                                                         int64_t n_dst, uint32_t k, VariateParams vp, const int64_t* __restrict__ eptr,
                                                         int32_t* __restrict__ col_global, int64_t* __restrict__ eid, int64_t edge_limit) {
  const int64_t w = (int64_t)blockIdx.x * kWavesPerBlock + uniform_wave_in_block();
  if (w >= n_dst) return;
  const NsRecord g = rec[w];
  if (g.d <= k) return;  // (copied whole by the fill kernel)
  if (eptr[w] + k > edge_limit) return;
  const uint32_t lane = (uint32_t)lane_id();
  const int32_t* __restrict__ list = g_indices + g.beg;
  const uint32_t d = g.d;
  const uint32_t sigma_a = ns_sigma(vp.K.Ka, (uint32_t)g.s);
  const uint32_t sigma_b = BLEND ? ns_sigma(vp.K.Kb, (uint32_t)g.s) : 0u;
  auto count_le = [&](uint32_t B) -> uint32_t {
    uint32_t n = 0;
    for (uint32_t base = 0; base < d; base += kWave) {
      const uint32_t j = base + lane;
      bool in = false;
      if (j < d) in = variate<true, BLEND>(vp, (uint32_t)list[j], sigma_a, sigma_b) <= B;
      n += (uint32_t)__popcll(ballot64(in));
    }
    return n;
  };
  uint64_t lo = 0, hi = 0xFFFFFFFFull;  // #{R <= hi} >= k throughout (d > k)
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo) / 2;
    if (count_le((uint32_t)mid) >= k) hi = mid;
    else lo = mid + 1;
  }
  const uint32_t B = (uint32_t)lo;
  const uint32_t below = B == 0 ? 0u : count_le(B - 1);
  const uint32_t need = k - below;  // of the entries with R = B, the first `need` in list order (>= 1)
  const int64_t o = eptr[w];
  uint32_t placed = 0, ties = 0;
  for (uint32_t base = 0; base < d; base += kWave) {
    const uint32_t j = base + lane;
    int32_t t = 0;
    uint32_t R = 0xFFFFFFFFu;
    if (j < d) {
      t = list[j];
      R = variate<true, BLEND>(vp, (uint32_t)t, sigma_a, sigma_b);
    }
    const bool eq = j < d && R == B;
    const uint64_t eq_mask = ballot64(eq);
    const bool keep = j < d && (R < B || (eq && ties + lanes_below(eq_mask) < need));
    const uint64_t keep_mask = ballot64(keep);
    if (keep) {
      const uint32_t at = placed + lanes_below(keep_mask);  // below k: exactly k entries are kept
      col_global[o + at] = t;  // (no tag: the dedup of layers with such fanouts reads keys)
      eid[o + at] = g.beg + j;
    }
    placed += (uint32_t)__popcll(keep_mask);
    ties += (uint32_t)__popcll(eq_mask);
  }
}

int ns_layer(const SampleCtx& cx, int l, const int32_t* dst, int64_t n_dst, coop_block* blk, int64_t edge_cap) {
  const bool defer = edge_cap > 0;
  hipStream_t s = cx.s;
  Alloc& alloc = *cx.alloc;
  const uint32_t k = (uint32_t)cx.fanouts[l];
  VariateParams vp{};
  layer_keys(cx.seed, COOP_NS, l, cx.group, vp.K.Ka);
  layer_keys(cx.seed, COOP_NS, l, cx.group + 1, vp.K.Kb);
  vp.cw = cx.cw;
  vp.sw = cx.sw;
  blk->indptr = alloc.get<int64_t>(n_dst + 1, COOP_TAG_OUTPUT);
  NsRecord* rec = alloc.get<NsRecord>(n_dst, COOP_TAG_SCRATCH);
  NsBlendThr* bthr = cx.blend ? alloc.get<NsBlendThr>(n_dst, COOP_TAG_SCRATCH) : nullptr;
  if (alloc.failed) return COOP_E_NOMEM;
  // candidate buffer: cap >= 4k (power of two, at least 256).  With a fanout above kNsMaxSelect the lists longer than
  // the fanout are left to k_ns_fill_wide, which keeps no candidates.
  const uint32_t k_sel = k < kNsMaxSelect ? k : kNsMaxSelect;
  uint32_t cap = 256;
  while (cap < 4 * k_sel) cap <<= 1;
  // expected candidates (at most 2k + 16): k + 2 sqrt(k) + 2 with independent variates, where a list that turns up fewer
  // than k candidates (two in a hundred at k = 10) is simply collected again with twice the bound, and every candidate
  // costs an append and ranking work (measured: 5 % off the fill pass against k + 4 sqrt(k) + 4); k + 4 sqrt(k) + 4 with
  // dependent variates, where a list that falls short (one in 10^4) goes through the one-kernel path again.
  uint32_t root = 1;
  while (root * root < k_sel) ++root;
  uint32_t target = cx.blend ? k_sel + 4 * root + 4 : k_sel + 2 * root + 2;
  if (target > 2 * k_sel + 16) target = 2 * k_sel + 16;
  // long lists first (see k_ns_fill): worth its queue from a few tens of thousands of destinations on
  // (default: passes over many destinations of a graph with hubs; where the registration has added the entries of the
  // lists above kLongListDegree up, a graph on which they hold less than an eighth of the edges is left alone: the queue
  // costs the count pass a reservation per block and buys nothing there)
  const bool hubs = !cx.g->symmetric || cx.g->long_mass >= cx.g->n_edges / 8;
  const bool queue_long = g_ns_long_min != 0 && n_dst <= kSliceLists / 2 /* (the queue's waves are launched in front of the others) */ &&
                          (g_ns_long_min != kNsLongDefault || (n_dst >= kNsQueueFrom && hubs));
  const uint32_t long_min = queue_long ? (uint32_t)g_ns_long_min : 0u;
  uint32_t* long_list = queue_long ? alloc.get<uint32_t>(n_dst, COOP_TAG_SCRATCH) : nullptr;
  uint32_t* n_long = cx.d_piece_count + l;  // (zero at the start of the call and whenever the layer is redone)
  if (alloc.failed) return COOP_E_NOMEM;
  const Publish pub = defer ? Publish{} : begin_publish(cx.d_ctl, cx.h_ctl);  // (not deferred: the kernel also sends the sizes to the host)
  const Clear clear = n_dst > 0 ? take_clear(cx) : Clear{nullptr, 0};
  int tile_log2 = 0;
#define COOP_NS_COUNT(BLOCK, EACH)                                                                                                             \
  do {                                                                                                                                         \
    tile_log2 = ns_tile_log2(BLOCK * EACH);                                                                                                    \
    const Begin begin = take_begin(cx, blocks_for(n_dst, BLOCK * EACH));                                                                       \
    COOP_LAUNCH(K_NS_COUNT, (k_ns_count<BLOCK, EACH>), dim3(blocks_for(n_dst, BLOCK * EACH)), dim3(BLOCK), 0, s, cx.g->indptr,                 \
                cx.g->n_vertices, dst, n_dst, k, target, blk->indptr, rec, bthr, vp.K, cx.cw, cx.sw, cx.d_ctl, long_min, long_list, n_long,    \
                clear, begin, pub);                                                                                                            \
  } while (0)
  if (n_dst >= kNsCountWideFrom && !cx.blend) COOP_NS_COUNT(1024, 2);
  else if (n_dst >= 16384 || (n_dst > 0 && !cx.blend)) COOP_NS_COUNT(kBlock, 1);
  else if (n_dst > 0) COOP_NS_COUNT(kWave, 1);
  else scan_tiles(ChunkedI32{}, 0, blk->indptr, &cx.d_ctl->total_edges, cx.d_ctl, s, &pub);
#undef COOP_NS_COUNT
  if (!defer) {
    const int rc = wait_ctl(pub, cx.h_ctl, s);
    if (rc != COOP_OK) return rc;
  }
  const int64_t m = defer ? edge_cap : cx.h_ctl->total_edges;  // entries of the edge arrays
  blk->n_edges = defer ? -1 : m;
  blk->col_global = alloc.get<int32_t>(m, COOP_TAG_OUTPUT);
  blk->eid = alloc.get<int64_t>(m, COOP_TAG_OUTPUT);
  blk->col_local = alloc.get<int32_t>(m, COOP_TAG_OUTPUT);
  if (alloc.failed) return COOP_E_NOMEM;
  const EdgeOut edges{blk->col_global, blk->eid, cx.tags};
  if (m > 0 && n_dst > 0) {
    // one wave per block: a block leaves the CU when its slowest wave is done, and a wave takes one list, short or long;
    // with four waves a block's slots stood empty for much of its life (fill 1.61 -> 1.52 ms on the papers100M-shaped
    // layer; with dependent variates the traversal 3.0 -> 2.57 ms and the selection 0.99 -> 0.91)
    const int wpb = 1;
    const size_t shmem = (size_t)wpb * cap * 16 + (cx.blend ? (size_t)wpb * sizeof(NsQueue) : 0);
    StageEntry* rows = nullptr;
    uint32_t* n_cand = nullptr;
    uint32_t row_cap = 64;
    if (cx.blend) {
      // rows of the two-kernel path: room for twice the expected candidates (at least 64, at most the LDS capacity)
      while (row_cap < 2 * target && row_cap < cap) row_cap <<= 1;
      rows = alloc.get<StageEntry>(n_dst * (int64_t)row_cap, COOP_TAG_SCRATCH);
      n_cand = alloc.get<uint32_t>(n_dst, COOP_TAG_SCRATCH);
      if (alloc.failed) return COOP_E_NOMEM;
    }
    // the queue's waves, one per queued list: as many as there can be lists that long, by the degree census of the
    // registration and by the number of edges (the unused ones end at once)
    int64_t most_long = cx.g->n_edges / (int64_t)(long_min ? long_min : 1) + 1;
    if (most_long > n_dst) most_long = n_dst;
    if (long_min != 0 && most_long > cx.g->lists_longer_than(long_min)) most_long = cx.g->lists_longer_than(long_min);
    const int long_blocks = queue_long ? (int)blocks_for(most_long, wpb) : 0;
    for (int64_t b = 0; b < n_dst; b += kSliceLists) {  // (one slice, unless there are 67 million destinations)
      const int64_t n = n_dst - b < kSliceLists ? n_dst - b : kSliceLists;
      const dim3 grid_w(blocks_for(n, kWavesPerBlock));
      int each_log2 = 0;
      while (each_log2 < 3 && (n >> (each_log2 + 1)) >= kNsFillWaves) ++each_log2;
      const Dealing deal = deal_lists(n, each_log2, finer_last(cx.g->degrees(), each_log2, l > 0));
      const NsRecord* rec_b = rec + b;
      const NsBlendThr* bthr_b = cx.blend ? bthr + b : nullptr;
      const int64_t* eptr_b = blk->indptr + b;
#define COOP_NS_ARGS cx.g->indices, rec_b, bthr_b, n, k, cap, wpb, vp, eptr_b, edges, m
      if (cx.blend) {
        StageEntry* rows_b = rows + b * (int64_t)row_cap;
        // Lanes per destination in the selection: as many as hold the candidates of most (a tenth more pass the filters than are
        // expected; 250 thousand destinations with 15 expected: 112 us with 64 lanes and a wave for each, 49 with 32 and eight a wave).
        const int group_log2 = target <= 10 ? 4 : target <= 24 ? 5 : 6;
        // (Also where more candidates than lanes are expected: a wave for each of 400 thousand destinations whose lists are shorter than
        // a fanout of 60 cost 91 us, eight a wave 32; over longer lists, 65,536 to 262,144 of them, fanout 200, no difference but noise.)
        const int select_log2 = each_log2 > 6 - group_log2 ? each_log2 : 6 - group_log2;
        uint32_t* n_cand_b = n_cand + b;
        int lists_log2 = 0;
        while (lists_log2 < 6 && (n >> (lists_log2 + 1)) >= kNsRedoWaves) ++lists_log2;
        const dim3 grid_redo(blocks_for(n, (int64_t)wpb << lists_log2));
        COOP_LAUNCH(K_NS_FILL, k_ns_collect, dim3(deal.blocks + (unsigned)long_blocks), dim3(kWave), 0, s, cx.g->indices,
                    rec_b, bthr_b, (uint32_t)n, k, vp.K, (float)vp.cw, (float)vp.sw, blk->indptr, b, tile_log2, edges, m, rows_b,
                    row_cap, n_cand_b, long_min, (const uint32_t*)long_list, (const uint32_t*)n_long, long_blocks, deal, (uint32_t)g_stretch);
        COOP_LAUNCH(K_NS_SELECT, k_ns_select, dim3(blocks_for(n, (int64_t)1 << select_log2)), dim3(kWave), (size_t)cap * sizeof(NsSlot), s, rec_b, n, k, vp,
                    eptr_b, edges, (const StageEntry*)rows_b, row_cap, n_cand_b, bthr_b, select_log2, group_log2);
#define COOP_NS_BLEND(VEC4) \
  COOP_LAUNCH(K_NS_FILL, k_ns_redo<VEC4>, grid_redo, dim3(wpb * kWave), shmem, s, COOP_NS_ARGS, cx.d_ctl, (const uint32_t*)n_cand_b, lists_log2)
        if (cx.vec4) { COOP_NS_BLEND(true); } else { COOP_NS_BLEND(false); }
#undef COOP_NS_BLEND
      } else {
        COOP_LAUNCH(K_NS_FILL, k_ns_fill, dim3(deal.blocks + (unsigned)long_blocks), dim3(kWave),
                    (cap + kWave) * sizeof(NsSlot), s, cx.g->indices, rec_b, (uint32_t)n, k, cap, vp.K, blk->indptr, b, tile_log2,
                    edges, m, cx.d_ctl, long_min, (const uint32_t*)long_list, (const uint32_t*)n_long, long_blocks, deal,
                    (uint32_t)g_stretch);
      }
#undef COOP_NS_ARGS
      if (k > kNsMaxSelect) {  // the lists longer than such a fanout (the kernels above skip them)
        if (cx.blend) COOP_LAUNCH(K_NS_FILL, k_ns_fill_wide<true>, grid_w, dim3(kBlock), 0, s, cx.g->indices, rec_b, n, k, vp, eptr_b,
                                  blk->col_global, blk->eid, m);
        else COOP_LAUNCH(K_NS_FILL, k_ns_fill_wide<false>, grid_w, dim3(kBlock), 0, s, cx.g->indices, rec_b, n, k, vp, eptr_b,
                         blk->col_global, blk->eid, m);
      }
    }
  }
  return COOP_OK;
}

}  // namespace coop
