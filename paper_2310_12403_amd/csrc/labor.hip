// LABOR-0 layers (App. A.1.2): edge (t -> s) is kept iff r_t <= k / d_s, i.e. R_t * d_s <= k * 2^32 in integers,
// which for d_s > k is R_t <= floor(k * 2^32 / d_s).  Kept edges leave in (destination order, adjacency order).
//
// Every neighbour list is read ONCE per minibatch.  S^l is a prefix of S^{l+1} (Eq. 2), so a vertex that becomes a
// destination at layer l is a destination at every later layer too, with the same list and a different key: the scan
// pass of layer l therefore covers only the vertices new at layer l and evaluates, for each neighbour, the keep tests
// of layers l .. L-1 at once (one mixer evaluation per layer, one read of the entry).  The kept (vertex, position)
// pairs are parked in small per-destination staging rows, one row set per covered layer; building layer l' later is
// a scan over the kept-edge counts and a copy of the rows.  A row that overflows is rare; those lists are scanned a
// second time, in order, straight into the edge arrays.
#include "device_utils.h"
#include "blend_scan.h"
#include "list_reader.h"
#include "sample_internal.h"

namespace coop {

constexpr uint32_t kAllThr = 0xFFFFFFFFu;  // threshold of a list no longer than the fanout: everything is kept

struct ScanOut {
  StageEntry* stage[kMaxFuse];
  int32_t* cnt[kMaxFuse];
};

struct FusedKeys {
  LayerKeys K[kMaxFuse];
  double cw, sw;
};

// The pieces of one layer's destinations, by the pass that scanned them.
struct LayerChunks {
  const Segment* seg[kMaxFuse];
  const uint32_t* thr[kMaxFuse];
  const StageEntry* stage[kMaxFuse];
  int64_t start[kMaxFuse];
  int n_chunks;
  __device__ __forceinline__ int find(int64_t w) const {
    int p = 0;
#pragma unroll
    for (int q = 1; q < kMaxFuse; ++q)
      if (q < n_chunks && w >= start[q]) p = q;
    return p;
  }
};

// ---- LABOR-0 from the other side (c = 0, symmetric graph) ----------------------------------------------------------
// R_t = mix(t ^ K0) ^ K1 is a bijection of the 32-bit integers, so the vertices with R_t <= u_max can be listed without
// looking at the graph: t = unmix(u ^ K1) ^ K0 for u = 0 .. u_max, kept if t < |V|.  A destination s with a list longer
// than D keeps exactly the neighbours with R_t <= floor(k 2^32 / d_s) < k 2^32 / D: all of them are among the
// |V| k / D vertices listed for u_max = floor(k 2^32 / (D + 1)).  On a symmetric graph "t is a neighbour of s" can be
// decided from t's side: the kernel walks the (mostly short) lists of the listed vertices, looks every entry s up in the
// table of long destinations, and where R_t is within that destination's threshold it has found a kept edge, whose
// position in the destination's own list comes from the graph handle's index of reverse positions.  The long lists,
// most of the entries that a scan would have to read, are never read.
__device__ __forceinline__ uint32_t long_slot(uint32_t s) { return (uint32_t)(((uint64_t)s * 0x9E3779B97F4A7C15ull) >> 32); }
// a slot of the table of long destinations: key = vertex + 1 (0: empty), its list index, its thresholds; one 32-byte
// sector.  Open addressing, and no key lies further than kLongProbes slots from its home: a table too full for that
// makes the pass fall back to the ordinary scan.
struct alignas(32) LongSlot { uint32_t key, list, thr[kMaxFuse], pad[2]; };
constexpr uint32_t kLongProbes = 64;
// In front of the table, a bit per hash value says whether any long destination has it: the walk keeps these bits in
// LDS, and goes to the table (in L2) only for the entries that pass, the long destinations' own and a few per cent more.
constexpr uint32_t kLongBits = 1u << 18;  // 32 KB
constexpr int kWalkBlock = 512;           // three blocks per CU, each with the bits in LDS
__device__ __forceinline__ uint32_t long_bit(uint32_t s) { return long_slot(s) >> 14; }

struct EnumItem { int64_t beg; uint32_t len, t, u, pad; };  // up to kEnumItem entries of listed vertex t's list; u = R_t
constexpr uint32_t kEnumItem = 64;         // entries per item: 16 lanes walk it, 4 entries each, loaded together
constexpr int kListBlock = 512;            // threads per block of k_enum_list
constexpr uint32_t kEnumListSpan = 16384;  // variates per block of k_enum_list (few blocks: each reserves its items with a
                                           // same-address atomic, and those are taken one after the other, some 20 ns each)
constexpr uint32_t kEnumListStep = 1024;   // variates per step of a block (2 per thread), between two barriers
constexpr uint32_t kEnumListBuf = 2048;    // vertices a block collects before it writes their items out (53 KB: three blocks per CU)

struct EnumOut {
  EnumItem* item[kMaxFuse];    // [item_cap[f]] per covered layer
  uint32_t* n_item[kMaxFuse];  // one counter each
  uint32_t item_cap[kMaxFuse];
};

// blockIdx.y = covered layer f: lists the vertices with R_t <= u_max[f].  A block takes kEnumListSpan consecutive
// variates, collects the vertices they belong to in LDS, fetches their list bounds, and writes their lists, cut into
// items, to the layer's item list: one reservation (a same-address atomic) per flush (one in 40 of the variates of a
// papers100M-sized graph gives a vertex).
__global__ __launch_bounds__(kListBlock) void k_enum_list(FusedKeys keys, uint32_t um0, uint32_t um1, uint32_t um2, uint32_t um3,
                                                      int64_t n_vertices, const int64_t* __restrict__ g_indptr, EnumOut eo, Ctl* ctl,
                                                      uint32_t todo /* bit f: layer f is to be listed (the others have their lists) */) {
  __shared__ uint2 buf[kEnumListBuf];     // (t, u)
  __shared__ uint32_t s_d[kEnumListBuf], s_at[kEnumListBuf];
  __shared__ int64_t s_beg[kEnumListBuf];
  __shared__ uint16_t s_long[kEnumListBuf];  // the collected vertices that give more than one item
  __shared__ uint32_t n_buf, n_local, n_long, base;
  const int f = blockIdx.y;
  const uint32_t u_max = f == 0 ? um0 : f == 1 ? um1 : f == 2 ? um2 : um3;
  const uint32_t K0 = keys.K[f].Ka[0], K1 = keys.K[f].Ka[1];
  const uint64_t first = (uint64_t)blockIdx.x * kEnumListSpan;
  if (first > u_max || ((todo >> f) & 1u) == 0) return;  // block-uniform
  EnumItem* __restrict__ item_f = f == 0 ? eo.item[0] : f == 1 ? eo.item[1] : f == 2 ? eo.item[2] : eo.item[3];
  uint32_t* n_item_f = f == 0 ? eo.n_item[0] : f == 1 ? eo.n_item[1] : f == 2 ? eo.n_item[2] : eo.n_item[3];
  const uint32_t item_cap_f = f == 0 ? eo.item_cap[0] : f == 1 ? eo.item_cap[1] : f == 2 ? eo.item_cap[2] : eo.item_cap[3];
  if (threadIdx.x == 0) { n_buf = 0; n_local = 0; n_long = 0; }
  __syncthreads();
  auto flush = [&]() {  // block-uniform call, after a barrier
    const uint32_t nb = n_buf;  // <= kEnumListBuf: a step adds at most kEnumListStep and is taken only when that many fit
    for (uint32_t i = threadIdx.x; i < nb; i += kListBlock) {
      const uint32_t t = buf[i].x;
      const int64_t beg = g_indptr[t];
      const uint32_t d = (uint32_t)(g_indptr[t + 1] - beg);  // (0: a vertex without neighbours is nobody's neighbour)
      s_d[i] = d;
      s_beg[i] = beg;
      if (d != 0) s_at[i] = atomicAdd(&n_local, (d + kEnumItem - 1) / kEnumItem);
      if (d > kEnumItem) s_long[atomicAdd(&n_long, 1u)] = (uint16_t)i;
    }
    __syncthreads();
    if (threadIdx.x == 0) base = n_local ? atomicAdd(n_item_f, n_local) : 0u;
    __syncthreads();
    if (base + n_local > item_cap_f) {
      if (threadIdx.x == 0) atomicOr(&ctl->cand_overflow, 1);  // (the pass is redone without this shortcut)
    } else {
      for (uint32_t i = threadIdx.x; i < nb; i += kListBlock) {  // a thread per vertex with one item
        const uint32_t d = s_d[i];
        if (d != 0 && d <= kEnumItem) item_f[base + s_at[i]] = EnumItem{s_beg[i], d, buf[i].x, buf[i].y, 0u};
      }
      // a wave for each of the others (their bounds are at hand: read again, one list after the other, they were most of the
      // kernel's 40 us)
      for (uint32_t v = threadIdx.x / kWave; v < n_long; v += kListBlock / kWave) {
        const uint32_t i = s_long[v];
        const uint32_t d = s_d[i];
        const uint2 tu = buf[i];
        const int64_t beg = s_beg[i];
        EnumItem* to = item_f + base + s_at[i];
        for (uint32_t q = (uint32_t)lane_id(); (uint64_t)q * kEnumItem < d; q += kWave) {
          const uint32_t off = q * kEnumItem;
          to[q] = EnumItem{beg + off, d - off < kEnumItem ? d - off : kEnumItem, tu.x, tu.y, 0u};
        }
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) { n_buf = 0; n_local = 0; n_long = 0; }
    __syncthreads();
  };
  for (uint32_t step = 0; step < kEnumListSpan; step += kEnumListStep) {
#pragma unroll
    for (uint32_t q = 0; q < kEnumListStep; q += kListBlock) {
      const uint64_t u = first + step + q + threadIdx.x;
      const uint32_t t = unmix32((uint32_t)u ^ K1) ^ K0;
      if (u <= u_max && (uint64_t)t < (uint64_t)n_vertices) buf[atomicAdd(&n_buf, 1u)] = make_uint2(t, (uint32_t)u);
    }
    __syncthreads();
    const bool nearly_full = n_buf > kEnumListBuf - kEnumListStep;  // read by everyone before anyone adds again
    __syncthreads();
    if (nearly_full) flush();
  }
  flush();
}

// blockIdx.y = covered layer f: 16 lanes per item; a lane's four entries are requested together, and so are the table
// slots of those that pass the bit test.
// A kept edge costs a chain of three dependent memory operations (its reverse position, a returning atomic on its
// destination's counter, the store into the staging row), and a step of 256 entries finds only a handful: committed on
// the spot they would make the wave wait out that chain in every step with a few lanes at work.  So the kept edges of a
// wave wait in a queue in LDS and are committed 64 at a time, every lane with a chain of its own, and once more when the
// wave is through its items.
struct WalkQueue {
  uint32_t n;  // entries waiting (below 128; the same for every lane of the wave)
  uint32_t list[2 * kWave];
  int32_t t[2 * kWave];
  uint32_t pos_lo[2 * kWave], pos_hi[2 * kWave];  // position of the entry in the graph's indices
};
__global__ __launch_bounds__(kWalkBlock, 6) void k_enum_walk(const int32_t* __restrict__ g_indices, const uint32_t* __restrict__ rev_pos,
                                                          const uint32_t* __restrict__ long_bits, const LongSlot* __restrict__ long_tab,
                                                          uint32_t long_mask, uint32_t stage_cap, ScanOut out, EnumOut eo, Ctl* ctl) {
  __shared__ uint32_t bits[kLongBits / 32];
  __shared__ WalkQueue queues[kWalkBlock / kWave];
  const int f = blockIdx.y;
  if (ctl->cand_overflow != 0) return;  // (some items were not written, or some destinations not entered: the pass is redone)
  WalkQueue& wq = queues[threadIdx.x / kWave];
  if ((threadIdx.x & (kWave - 1)) == 0) wq.n = 0;
  for (uint32_t i = threadIdx.x; i < kLongBits / 128; i += kWalkBlock)
    reinterpret_cast<uint4*>(bits)[i] = reinterpret_cast<const uint4*>(long_bits)[i];
  __syncthreads();
  uint32_t total = *(f == 0 ? eo.n_item[0] : f == 1 ? eo.n_item[1] : f == 2 ? eo.n_item[2] : eo.n_item[3]);
  const uint32_t item_cap_f = f == 0 ? eo.item_cap[0] : f == 1 ? eo.item_cap[1] : f == 2 ? eo.item_cap[2] : eo.item_cap[3];
  if (total > item_cap_f) total = item_cap_f;
  const EnumItem* __restrict__ item_f = f == 0 ? eo.item[0] : f == 1 ? eo.item[1] : f == 2 ? eo.item[2] : eo.item[3];
  int32_t* __restrict__ cnt_f = f == 0 ? out.cnt[0] : f == 1 ? out.cnt[1] : f == 2 ? out.cnt[2] : out.cnt[3];
  StageEntry* __restrict__ stage_f = f == 0 ? out.stage[0] : f == 1 ? out.stage[1] : f == 2 ? out.stage[2] : out.stage[3];
  const uint32_t sub = threadIdx.x & 15u;
  const uint32_t groups = (gridDim.x * kWalkBlock) >> 4;
  // The first `n` queued edges (n <= 64), shared out among the lanes that are still here (the 16-lane groups of a wave
  // run out of items at different times): reverse position, place in the row, store.
  auto commit = [&](uint32_t n) {
    const uint64_t here = ballot64(true);
    const uint32_t n_here = (uint32_t)__popcll(here);
    for (uint32_t i = lanes_below(here); i < n; i += n_here) {
      const uint32_t list = wq.list[i];
      const uint32_t j = rev_pos[((uint64_t)wq.pos_hi[i] << 32) | wq.pos_lo[i]];
      const uint32_t at = (uint32_t)atomicAdd(&cnt_f[list], 1);
      if (at < stage_cap) stage_f[(size_t)list * stage_cap + at] = StageEntry{wq.t[i], j};
      else if (at == stage_cap) atomicAdd(&ctl->n_overflow, 1);  // exactly one entry sees the row fill up
    }
  };
  // (two items ahead: while the table slots of the current item are in flight, so are the entries of the next one and the
  // record of the one after it)
  uint32_t c = (blockIdx.x * kWalkBlock + threadIdx.x) >> 4;
  if (c >= total) return;
  EnumItem it = item_f[c];
  EnumItem it_next = it;
  if (c + groups < total) it_next = item_f[c + groups];
  uint32_t s4[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t j = (uint32_t)e * 16u + sub;
    s4[e] = (uint32_t)g_indices[it.beg + (j < it.len ? j : it.len - 1)];  // (len >= 1; a lane past the end repeats the last entry)
  }
  for (;;) {
    const bool more = c + groups < total;
    uint32_t h4[4];
    bool maybe[4];
    uint4 head4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t b = long_bit(s4[e]);
      maybe[e] = (uint32_t)e * 16u + sub < it.len && ((bits[b >> 5] >> (b & 31u)) & 1u) != 0;
      h4[e] = long_slot(s4[e]) & long_mask;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (maybe[e]) head4[e] = *reinterpret_cast<const uint4*>(&long_tab[h4[e]]);
    // The requests for the next rounds go out behind the table slots, not in front of them: loads come back in the
    // order in which they were sent, and the slots (in L2) must not wait for these (in HBM).
    asm volatile("" ::: "memory");
    EnumItem it_next2 = it_next;
    if ((uint64_t)c + 2ull * groups < total) it_next2 = item_f[c + 2u * groups];
    uint32_t s4_next[4] = {0, 0, 0, 0};
    if (more) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t j = (uint32_t)e * 16u + sub;
        s4_next[e] = (uint32_t)g_indices[it_next.beg + (j < it_next.len ? j : it_next.len - 1)];
      }
    }
    asm volatile("" ::: "memory");
    // Which entries are long destinations of this pass (the key in a slot is the vertex + 1, 0 an empty slot), and is
    // R_t within their threshold?  An entry whose home slot holds another key moves on to the next slot; the entries
    // of a lane do so together, a round of requests at a time.
    uint32_t list4[4];
    bool open4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) open4[e] = maybe[e];
    for (uint32_t probe = 1;; ++probe) {
      bool again = false;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (open4[e]) {
          if (head4[e].x == s4[e] + 1) {
            open4[e] = false;
            list4[e] = head4[e].y;
            maybe[e] = it.u <= (f == 0 ? head4[e].z : f == 1 ? head4[e].w : long_tab[h4[e]].thr[f]);
          } else if (head4[e].x == 0 || probe >= kLongProbes) {
            open4[e] = false;
            maybe[e] = false;
          } else {
            h4[e] = (h4[e] + 1) & long_mask;
            again = true;
          }
        }
      if (!again) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (open4[e]) head4[e] = *reinterpret_cast<const uint4*>(&long_tab[h4[e]]);
    }
    // kept edges t -> s join the wave's queue; a full wave of them is committed at once
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint64_t mask = ballot64(maybe[e]);
      if (mask == 0) continue;
      uint32_t nq = wq.n;  // (below 64 here)
      if (maybe[e]) {
        const uint32_t at = nq + lanes_below(mask);
        const uint64_t pos = (uint64_t)it.beg + (uint32_t)e * 16u + sub;
        wq.list[at] = list4[e];
        wq.t[at] = (int32_t)it.t;
        wq.pos_lo[at] = (uint32_t)pos;
        wq.pos_hi[at] = (uint32_t)(pos >> 32);
      }
      nq += (uint32_t)__popcll(mask);
      __builtin_amdgcn_wave_barrier();
      if (nq >= (uint32_t)kWave) {
        commit(kWave);
        __builtin_amdgcn_wave_barrier();
        const uint32_t rest = nq - kWave;  // fewer than 64: to the front
        const uint64_t here = ballot64(true);
        const uint32_t n_here = (uint32_t)__popcll(here);
        // (in rounds of the lanes that are here, each round read before it is written: a round only writes below what it read)
        for (uint32_t first = 0; first < rest; first += n_here) {
          const uint32_t i = first + lanes_below(here);
          uint32_t ml = 0, mlo = 0, mhi = 0;
          int32_t mt = 0;
          if (i < rest) { ml = wq.list[kWave + i]; mt = wq.t[kWave + i]; mlo = wq.pos_lo[kWave + i]; mhi = wq.pos_hi[kWave + i]; }
          __builtin_amdgcn_wave_barrier();
          if (i < rest) { wq.list[i] = ml; wq.t[i] = mt; wq.pos_lo[i] = mlo; wq.pos_hi[i] = mhi; }
          __builtin_amdgcn_wave_barrier();
        }
        nq = rest;
      }
      if (lanes_below(ballot64(true)) == 0) wq.n = nq;
      __builtin_amdgcn_wave_barrier();
    }
    if (!more) break;
    c += groups;
    it = it_next;
    it_next = it_next2;
#pragma unroll
    for (int e = 0; e < 4; ++e) s4[e] = s4_next[e];
  }
  // what still waits, fewer than 64 (every lane that had an item arrives here, whenever its group ran out)
  __builtin_amdgcn_wave_barrier();
  commit(wq.n);
}

// list records of the destinations scanned in this pass, and their keep thresholds for the nf covered layers
// (pthr, lim2: the blended path's first and second filter thresholds, null when c = 0)
// Large blocks: one queue reservation (a same-address atomic) per 1,024 destinations.  Below kSegWideFrom destinations small
// ones, which spread over more CUs what the thresholds of a blend cost in fp64 (1,024 destinations, three layers: 13 us in
// one block, 10 in sixteen; 110 thousand with two layers 15 and 9).
constexpr int64_t kSegWideFrom = 65536;
constexpr int64_t kSegSharedBelow = 16384;
constexpr uint32_t kPiecesByLane = 8;  // pieces of a list that its lane writes by itself
// (c > 0) The buffer of candidates for the exact blend is split into kCandSub sub-buffers with a counter each (a block appends to sub-buffer blockIdx mod
// kCandSub): appending costs an atomic with a returned value, and a single counter would serialise them.
constexpr int kCandSub = 256;
// With SHARED (blocks of three waves and c > 0) the first wave has the block's 64 destinations, and the two others evaluate some of their
// thresholds, each of them a chain of several hundred fp64 instructions: four behind one another in the place of seven (1,024 to 16
// thousand destinations of the reddit-shaped step with a cache: 10.5 us a launch and 8.5).
template <int kSegBlock, bool SHARED = false>
__global__ __launch_bounds__(kSegBlock) void k_segments(const int64_t* __restrict__ g_indptr, int64_t n_vertices,
                                                     const int32_t* dst, int64_t n, int nf,
                                                     uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3, Segment* __restrict__ seg,
                                                     uint32_t* __restrict__ thr, PreThr* __restrict__ pthr, float* __restrict__ lim2,
                                                     double cw, double sw, Ctl* ctl,
                                                     PieceCut cut, Piece* __restrict__ pieces, uint32_t piece_cap,
                                                     uint32_t* __restrict__ piece_count, ScanOut out, uint32_t enum_degree,
                                                     uint32_t* __restrict__ long_bits, LongSlot* __restrict__ long_tab, uint32_t long_mask,
                                                     Clear clear, Begin begin, uint32_t* __restrict__ cand_count /* kCandSub, set to zero; null when c = 0 */) {
  dst = begin_in_block(begin, dst);
  clear_words(clear);
  if (cand_count != nullptr && blockIdx.x == 0)
    for (int q = threadIdx.x; q < kCandSub; q += kSegBlock) cand_count[q] = 0;
  __shared__ uint32_t s_wave_at[kSegBlock / kWave];
  __shared__ uint32_t s_base, s_total;
  constexpr int kDestinations = SHARED ? kWave : kSegBlock;
  const int64_t i = (int64_t)blockIdx.x * kDestinations + (SHARED ? (int)(threadIdx.x & (kWave - 1)) : (int)threadIdx.x);
  const int share = SHARED ? uniform_wave_in_block() : 0;
  if (SHARED && share != 0 && i < n) {
    const int32_t s = dst[i];
    uint32_t d = 0;
    if ((uint64_t)(uint32_t)s < (uint64_t)n_vertices) d = (uint32_t)(g_indptr[s + 1] - g_indptr[s]);
    const uint32_t ks[kMaxFuse] = {k0, k1, k2, k3};
#pragma unroll
    for (int f = 0; f < kMaxFuse; ++f)
      if (f < nf) {
        const uint32_t t = d > ks[f] ? (uint32_t)(((uint64_t)ks[f] << 32) / (uint64_t)d) : kAllThr;
        if (share == 1) {
          pthr[(int64_t)f * n + i].a2 = t < kThrAllPass ? blend_a2(blend_x2(blend_tau(t), cw, sw)) : 0xFFFFFFFFu;
        } else {
          pthr[(int64_t)f * n + i].keep2 = blend_keep_threshold(t, cw + sw);
          lim2[(int64_t)f * n + i] = blend_second_threshold(t, blend_tau(t), cw + sw);
        }
      }
  }
  const bool live = share == 0 && i < n;
  Segment g{0, 0, 0};
  bool sampled = live;  // every covered layer keeps a proper subset (d > k)
  uint32_t thr_mine[kMaxFuse] = {0, 0, 0, 0};
  if (live) {
    const int32_t s = dst[i];
    if ((uint64_t)(uint32_t)s >= (uint64_t)n_vertices) {
      atomicOr(&ctl->err_range, 1);
    } else {
      g.beg = g_indptr[s];
      g.d = (uint32_t)(g_indptr[s + 1] - g.beg);
    }
    const uint32_t ks[kMaxFuse] = {k0, k1, k2, k3};
#pragma unroll
    for (int f = 0; f < kMaxFuse; ++f)
      if (f < nf) {
        const uint32_t t = g.d > ks[f] ? (uint32_t)(((uint64_t)ks[f] << 32) / (uint64_t)g.d) : kAllThr;
        sampled &= t != kAllThr;
        thr[(int64_t)f * n + i] = t;
        thr_mine[f] = t;
        if constexpr (SHARED) {
          uint32_t a1 = 0xFFFFFFFFu, b2 = 0xFFFFFFFFu;
          if (t < kThrAllPass) {
            const double tau = blend_tau(t);
            blend_strip(tau, blend_x2(tau, cw, sw), cw, sw, &a1, &b2);
          }
          pthr[(int64_t)f * n + i].a1 = a1;
          pthr[(int64_t)f * n + i].b2 = b2;
        } else if (pthr) {
          const double tau = blend_tau(t);
          PreThr pt = blend_first_thresholds(t, tau, cw, sw);
          pt.keep2 = blend_keep_threshold(t, cw + sw);
          pthr[(int64_t)f * n + i] = pt;
          lim2[(int64_t)f * n + i] = blend_second_threshold(t, tau, cw + sw);
        }
      }
  }
  // A list longer than enum_degree (when that is not 0) is not scanned at all: its kept neighbours are found from the
  // other side (k_enum_*).  The destination is entered in the table that maps such vertices to their list.
  const bool from_other_side = enum_degree != 0 && sampled && g.d > enum_degree;
  if (from_other_side) {
    g.split = 1;  // (the scan leaves it alone, like a list cut into pieces)
#pragma unroll
    for (int f = 0; f < kMaxFuse; ++f)
      if (f < nf) out.cnt[f][i] = 0;  // kept edges are counted by atomics
    const unsigned long long mine = ((unsigned long long)(uint32_t)i << 32) | ((uint32_t)dst[i] + 1u);  // (key, list)
    uint32_t h = long_slot((uint32_t)dst[i]) & long_mask;
    bool entered = false;
    for (uint32_t probe = 0; probe < kLongProbes && !entered; ++probe) {
      if (atomicCAS(reinterpret_cast<unsigned long long*>(&long_tab[h]), 0ull, mine) == 0ull) {
        entered = true;
#pragma unroll
        for (int f = 0; f < kMaxFuse; ++f)
          if (f < nf) long_tab[h].thr[f] = thr_mine[f];
      }
      h = (h + 1) & long_mask;
    }
    if (!entered) atomicOr(&ctl->cand_overflow, 1);  // (the pass is redone without this shortcut)
    const uint32_t b = long_bit((uint32_t)dst[i]);
    atomicOr(&long_bits[b >> 5], 1u << (b & 31u));
    sampled = false;  // no pieces
  }
  if (cut.len == 0) {  // wave-uniform
    if (live) seg[i] = g;
    return;
  }
  // A long list is cut into pieces (PieceCut: equal lengths, multiples of 4), each scanned by a wave
  // of its own: the waves of the scan then all have about the same amount of work whatever the degree distribution.
  // The block reserves queue slots for all its long lists with one atomic; a lane then writes its list's pieces by itself, or, where
  // those are many, the wave does together.  (4,000 lists of 300 to 5,000 entries 13.8 us a launch with the wave on every list in turn,
  // 6.9 so, 6.3 with none cut.)
  const uint32_t np = sampled && g.d > cut.split_min ? cut.pieces(g.d) : 0u;
  const uint32_t incl = wave_incl_scan(np);
  const uint32_t lane = (uint32_t)lane_id();
  const int wv = uniform_wave_in_block();
  if (lane == kWave - 1) s_wave_at[wv] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t sum = 0;
    for (int q = 0; q < kSegBlock / kWave; ++q) { const uint32_t t = s_wave_at[q]; s_wave_at[q] = sum; sum += t; }
    s_total = sum;
    s_base = sum != 0 ? atomicAdd(piece_count, sum) : 0u;
  }
  __syncthreads();
  const uint32_t total = s_total;
  if (total != 0) {  // block-uniform
    const uint32_t block_base = s_base;
    // room suffices for distinct destinations (cut_pieces; short of that only on unaligned indices, whose queue lies in an array of the
    // layer); a seed list with duplicates may run out: its lists then stay whole and what was reserved becomes empty slots
    const bool fits = block_base <= piece_cap && total <= piece_cap - block_base;
    const uint32_t base = block_base + s_wave_at[wv];
    if (np <= kPiecesByLane) {
      const uint32_t at = base + incl - np, list = (uint32_t)i;
      for (uint32_t q = 0; q < np; ++q)
        if (at + q < piece_cap) pieces[at + q] = fits ? Piece{list, q} : Piece{kNoPiece, 0u};
    }
    uint64_t todo = ballot64(np > kPiecesByLane);
    while (todo != 0) {
      const int src = __builtin_ctzll(todo);
      todo &= todo - 1;
      const uint32_t np_s = (uint32_t)__builtin_amdgcn_readlane((int)np, src);
      const uint32_t at = base + (uint32_t)__builtin_amdgcn_readlane((int)incl, src) - np_s;
      const uint32_t list = (uint32_t)((int64_t)blockIdx.x * kDestinations + (threadIdx.x & ~(kWave - 1)) + src);
      for (uint32_t q = lane; q < np_s; q += kWave)
        if (at + q < piece_cap) pieces[at + q] = fits ? Piece{list, q} : Piece{kNoPiece, 0u};
    }
    if (fits && np != 0) {
      g.split = cut.each(g.d);
#pragma unroll
      for (int f = 0; f < kMaxFuse; ++f)
        if (f < nf) out.cnt[f][i] = 0;  // the pieces add their counts
    }
  }
  if (live) seg[i] = g;
}

// Ordered visit of the neighbour list [beg, beg + d) of one destination by the whole wave, one entry per lane and
// step: calls emit(rank, t, j) for every kept neighbour t at list position j, rank counting kept neighbours in
// adjacency order.  Returns the number kept (same value in every lane).  Used by the overflow pass.
template <bool BLEND, typename Emit>
__device__ __forceinline__ uint32_t labor_scan_ordered(const int32_t* __restrict__ g_indices, int64_t beg, uint32_t d, uint32_t thr,
                                                       const LayerKeys& K, double cw, double sw, Emit emit) {
  const int lane = lane_id();
  const bool all = thr == kAllThr;
  uint32_t count = 0;
  for (uint32_t base = 0; base < d; base += kWave) {
    const uint32_t j = base + lane;
    bool kp = j < d;
    int32_t t = 0;
    if (kp) {
      t = g_indices[beg + j];
      if (!all) kp = variate<false, BLEND>(K, cw, sw, (uint32_t)t, 0u, 0u) <= thr;
    }
    const uint64_t m = ballot64(kp);
    if (kp) emit(count + lanes_below(m), t, j);
    count += (uint32_t)__popcll(m);
  }
  return count;
}

// ---- independent variates (c = 0) ---------------------------------------------------------------------------------
// A wave's kept entries of one list, layer by layer: in list order in LDS until the list is done, then one 8-byte store per
// lane to the destination's staging row.
constexpr uint32_t kKeptSlots = 64;  // (no staging row is longer; what a list keeps beyond it is counted, not stored)
struct KeptSlots { StageEntry at[kKeptSlots + kWave]; };  // the last kWave: a slot per lane that nobody reads

template <int NF>
struct PlainKeys { uint32_t head[NF], tail[NF]; };  // in vector registers (vector_copy)
__device__ __forceinline__ uint32_t labor_uniform(uint32_t head, uint32_t tail, uint32_t t) { return words_uniform<false>(head, 0u, tail, t); }

// One pass over a list (or a stretch of it that starts at list position j0) for NF layers: neighbours with R_t <= thr[l] go to
// layer l's slots behind the n[l] that are there; those behind kKeptSlots are counted, not stored.
template <int NF>
__device__ __forceinline__ void labor_collect(ListReader<>& L, uint32_t j0, const uint32_t (&thr)[NF], const PlainKeys<NF>& K, KeptSlots* slots,
                                              uint32_t (&n)[NF]) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t idle = kKeptSlots + lane;
  for (uint32_t g0 = 0; g0 < L.n_groups; g0 += kReaderGroups) {
#pragma unroll
    for (uint32_t q = 0; q < kReaderGroups; ++q) {
      const uint32_t g = g0 + q;
      if (g >= L.n_groups) break;
      uint64_t m[NF][4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int l = 0; l < NF; ++l) m[l][e] = compare_mask(labor_uniform(K.head[l], K.tail[l], L.ring[q][e]) <= thr[l]);
#pragma unroll
      for (int l = 0; l < NF; ++l) {
        if ((m[l][0] | m[l][1] | m[l][2] | m[l][3]) == 0) continue;
        uint32_t to = n[l];
#pragma unroll
        for (int e = 0; e < 4; ++e) to = lanes_below_plus(m[l][e], to);
#pragma unroll
        for (int e = 0; e < 4; ++e) n[l] += (uint32_t)__popcll(m[l][e]);
        const uint32_t j = j0 + g * kGroup + lane * 4;
        if (n[l] <= kKeptSlots) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            slots[l].at[lane_in(m[l][e]) ? to : idle] = StageEntry{(int32_t)L.ring[q][e], j + e};
            to += lane_in(m[l][e]) ? 1u : 0u;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (lane_in(m[l][e])) {
              if (to < kKeptSlots) slots[l].at[to] = StageEntry{(int32_t)L.ring[q][e], j + e};
              ++to;
            }
          }
        }
      }
      if (g + kReaderGroups < L.n_groups) L.ring[q] = L.in.group(g + kReaderGroups);
    }
  }
  const uint32_t tail = L.n & ~(kGroup - 1);
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t at = tail + q * kWave;
    if (at >= L.n) return;
    const uint64_t there = low_lanes(L.n - at);
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      const uint64_t m = compare_mask(labor_uniform(K.head[l], K.tail[l], L.rest[q]) <= thr[l]) & there;
      if (m == 0) continue;
      const uint32_t to = lanes_below_plus(m, n[l]);
      n[l] += (uint32_t)__popcll(m);
      if (lane_in(m) && to < kKeptSlots) slots[l].at[to] = StageEntry{(int32_t)L.rest[q], j0 + at + lane};
    }
  }
}

// The scan pass with independent variates.  As k_ns_fill, which says what its parts are for: a wave takes `each` neighbouring
// destinations (a power of two, at most 64), lists of up to twice the 64 / each lanes that a destination has are looked at
// together, the others one after the other through the whole wave, the next one's entries requested before this one's kept
// entries leave.  The first `piece_blocks` blocks take the pieces of the long lists (block b takes pieces b,
// b + piece_blocks, ... of the queue, whose length is read from device memory); a piece adds its kept-edge counts to the list's
// counters and puts its entries wherever that leaves them in the staging row: the fill pass sorts the rows by list position.
//
// Bound by instruction issue next to HBM: last layer of the products shape, 480 thousand lists, 95 us with a list at a time, an
// ordered pass per layer over the short ones, lane masks in every group and a store to the row from every step with a kept entry,
// 68 now; the papers100M shape without the lists above 8,192 entries, 290 M entries in three passes, 345 us and 320, 310 with
// the last lists dealt two to a wave (the entries alone, at the rate of a copy: 237).  The next list's entries requested before this one's are looked at: 91 us and 330, for the
// registers.
template <int NF>
__global__ __launch_bounds__(kWave, NF == 1 ? 8 : NF == 2 ? 7 : 6) void k_labor_scan_plain(const int32_t* __restrict__ g_indices, const Segment* __restrict__ seg,
                                                               const uint32_t* __restrict__ thr_all, int64_t n, Dealing deal, FusedKeys keys,
                                                               uint32_t stage_cap, ScanOut out, Ctl* ctl, int piece_blocks,
                                                               const Piece* __restrict__ pieces, const uint32_t* __restrict__ piece_count,
                                                               uint32_t piece_cap, uint32_t stretch) {
  __shared__ KeptSlots slots[NF];
  const uint32_t lane = (uint32_t)lane_id();
  auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
  auto of64 = [&](int64_t x, int q) { return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)x >> 32), q) << 32) | of((uint32_t)x, q)); };
  PlainKeys<NF> K;
#pragma unroll
  for (int l = 0; l < NF; ++l) { K.head[l] = vector_copy(keys.K[l].Ka[4]); K.tail[l] = vector_copy(keys.K[l].Ka[1]); }
  auto settle = [] {
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
  };
  if ((int)blockIdx.x < piece_blocks) {
    uint32_t n_pieces = *piece_count;
    if (n_pieces > piece_cap) n_pieces = piece_cap;
    for (uint32_t p = blockIdx.x; p < n_pieces; p += (uint32_t)piece_blocks) {
      const Piece pc = pieces[p];
      const uint32_t list = of(pc.list, 0), q = of(pc.q, 0);
      if (list == kNoPiece) continue;
      const Segment g = seg[list];
      const int64_t beg = of64(g.beg, 0);
      uint32_t len;
      const int64_t j0 = piece_start(of(g.d, 0), of(g.split, 0), q, &len);
      if (j0 < 0) continue;
      uint32_t thr[NF], kept[NF];
#pragma unroll
      for (int l = 0; l < NF; ++l) { thr[l] = of(thr_all[(int64_t)l * n + list], 0); kept[l] = 0; }
      ListReader<> L(g_indices + beg + j0, len);
      labor_collect<NF>(L, (uint32_t)j0, thr, K, slots, kept);
      settle();
#pragma unroll
      for (int l = 0; l < NF; ++l) {
        const uint32_t c = kept[l];
        if (c == 0) continue;
        uint32_t at = 0;
        if (lane == 0) at = (uint32_t)atomicAdd(&out.cnt[l][list], (int32_t)c);
        at = of(at, 0);
        if (at + c <= stage_cap) {  // c <= stage_cap <= kKeptSlots: every entry has its slot
          if (lane < c) out.stage[l][(size_t)list * stage_cap + at + lane] = slots[l].at[lane];
        } else if (at <= stage_cap && lane == 0) {
          atomicAdd(&ctl->n_overflow, 1);  // the one piece that takes the row over its capacity reports the list
        }
      }
      settle();
    }
    return;
  }
  int each_log2;
  const int64_t w0 = deal.first_list(blockIdx.x - (uint32_t)piece_blocks, &each_log2);
  if (w0 >= n) return;
  const uint32_t n_mine = n - w0 < ((int64_t)1 << each_log2) ? (uint32_t)(n - w0) : 1u << each_log2;
  const uint32_t lanes = 64u >> each_log2, sub = lane & (lanes - 1), number = lane >> (6 - each_log2);
  const int64_t w = w0 + (number < n_mine ? number : n_mine - 1);
  const Segment g = seg[w];
  uint32_t my_thr[NF], my_kept[NF];
#pragma unroll
  for (int l = 0; l < NF; ++l) { my_thr[l] = thr_all[(int64_t)l * n + w]; my_kept[l] = 0; }
  const bool live = number < n_mine && g.split == 0, speaks = live && sub == 0;  // (split: scanned by other waves, or not at all)
  const uint32_t together = each_log2 != 0 ? 2 * lanes : 0;
  if (ballot64(live && g.d <= together && g.d != 0) != 0) {
    const uint64_t group = low_lanes(lanes) << (number * lanes);
    bool in[2];
    uint32_t t[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      in[r] = live && g.d <= together && sub + r * lanes < g.d;
      t[r] = 0;
      if (in[r]) t[r] = (uint32_t)(g_indices + g.beg)[sub + r * lanes];
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int l = 0; l < NF; ++l) {
        const bool keep = in[r] && labor_uniform(K.head[l], K.tail[l], t[r]) <= my_thr[l];
        const uint64_t m = ballot64(keep) & group;
        const uint32_t place = my_kept[l] + lanes_below(m);
        if (keep && place < stage_cap) out.stage[l][(size_t)w * stage_cap + place] = StageEntry{(int32_t)t[r], sub + r * lanes};
        my_kept[l] += (uint32_t)__popcll(m);
      }
  }
  uint64_t todo = ballot64(speaks && g.d > together);
  if (todo != 0) {
    int at = __builtin_ctzll(todo);
    uint32_t d = of(g.d, at), j0 = 0, thr[NF], kept[NF];
    int64_t beg = of64(g.beg, at);
#pragma unroll
    for (int l = 0; l < NF; ++l) { thr[l] = of(my_thr[l], at); kept[l] = 0; }
    for (ListReader<> L(g_indices + beg, d < stretch ? d : stretch);;) {
      labor_collect<NF>(L, j0, thr, K, slots, kept);
      if (d - j0 > stretch) {  // the list's next stretch
        j0 += stretch;
        L = ListReader<>(g_indices + beg + j0, d - j0 < stretch ? d - j0 : stretch);
        continue;
      }
      const int done = at;
      todo &= todo - 1;
      at = todo != 0 ? __builtin_ctzll(todo) : 0;
      d = todo != 0 ? of(g.d, at) : 0u;
      beg = of64(g.beg, at);
      j0 = 0;
      L = ListReader<>(g_indices + beg, d < stretch ? d : stretch);
      settle();
#pragma unroll
      for (int l = 0; l < NF; ++l) {
        const uint32_t c = kept[l] < stage_cap ? kept[l] : stage_cap;
        if (lane < c) out.stage[l][(size_t)(w0 + (done >> (6 - each_log2))) * stage_cap + lane] = slots[l].at[lane];
        if ((int)lane == done) my_kept[l] = kept[l];
        thr[l] = of(my_thr[l], at);
        kept[l] = 0;
      }
      settle();
      if (todo == 0) break;
    }
  }
  if (speaks) {
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      out.cnt[l][w] = (int32_t)my_kept[l];
      if (my_kept[l] > stage_cap) atomicAdd(&ctl->n_overflow, 1);
    }
  }
}

// ---- blended variates (c > 0) -------------------------------------------------------------------------------------
// The exact blend (two Phi^-1 and a Phi in binary64) costs about a hundred times the integer path and needs four
// times the registers of the traversal, so it is reached in three stages:
//   1. integer bounds on min(U1, U2) and max(U1, U2) (per list and layer; in the traversal loop);
//   2. the blend in fp32, for a full wave of stage-1 passers at a time, taken from a per-wave queue in LDS that lives
//      across the wave's lists: an estimate safely above the keep threshold is dropped, one safely below is a kept
//      edge, and only the narrow band in between (a few percent of the kept edges) is left undecided;
//   3. the exact blend for the undecided, in a kernel of its own (k_labor_exact) over a buffer in device memory that
//      the scan kernel appended them to: the scan kernel keeps the occupancy of a streaming kernel, the exact stage
//      runs with every lane busy.
// A kept edge takes the next free slot of its destination's staging row with an atomic on the row's counter; rows
// filled this way are unordered and the fill pass ranks them by list position.

// A candidate for the exact blend.
struct Cand {
  int32_t t;       // neighbour
  uint32_t j;      // its position in the destination's list
  uint32_t list;   // destination, index within the pass
  uint32_t layer;  // covered layer, 0 .. NF-1
};
struct CandOut {
  Cand* buf;          // [kCandSub][cap_each]
  uint32_t* count;    // [kCandSub] entries appended so far (may run past cap_each: the excess is dropped, the pass redone)
  uint32_t cap_each;
};

// What stage 2 leads to (blend_scan.h): an estimate safely below the threshold is a kept edge (it takes the next free slot of its
// destination's staging row: by a counter in LDS, where no other wave of the kernel has that destination); one safely above is
// dropped; the few in between are appended to the candidate buffer of the exact stage (one atomic per call), or, EXACT, evaluated
// here.
template <bool EXACT>
struct LaborSink {
  ScanOut out;
  CandOut cand;
  Ctl* ctl;
  uint32_t stage_cap;
  uint32_t first, shift;  // the list of lane s is first + (s >> shift)
  bool owns;              // no other wave of this kernel keeps edges of these lists
  const uint32_t* thr_all;  // (EXACT) [NF][n] keep thresholds
  int64_t n;
  double cw, sw;
  __device__ __forceinline__ void take(BlendQueue<false>* queue, int l, bool there, const StageEntry& e, uint32_t slot, uint32_t u1, uint32_t u2, float est) {
    const uint32_t lane = (uint32_t)lane_id();
    bool keep = there && est <= queue[l].keep2[slot];
    const bool maybe = there && !keep && est <= queue[l].lim2[slot];
    const uint32_t list = first + (slot >> shift);
    if constexpr (EXACT) {
      if (maybe) keep = blend_exact(u1, u2, cw, sw) <= thr_all[(int64_t)l * n + list];
    }
    if (keep) {
      const uint32_t at = owns ? atomicAdd(&queue[l].own[slot], 1u) : (uint32_t)atomicAdd(&out.cnt[l][list], 1);
      if (at < stage_cap) out.stage[l][(size_t)list * stage_cap + at] = e;
      else if (at == stage_cap && !owns) atomicAdd(&ctl->n_overflow, 1);  // exactly one entry sees the row fill up (owns: at the end)
    }
    if constexpr (EXACT) return;
    const uint64_t mask = ballot64(maybe);
    if (mask == 0) return;
    const uint32_t sub = blockIdx.x & (kCandSub - 1);
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&cand.count[sub], (uint32_t)__popcll(mask));
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + lanes_below(mask);
    if (maybe) {
      if (at < cand.cap_each) cand.buf[(size_t)sub * cand.cap_each + at] = Cand{e.t, e.j, list, (uint32_t)l};
      else atomicOr(&ctl->cand_overflow, 1);
    }
  }
};

// The scan pass with blended variates: destinations, pieces and short lists as in k_labor_scan_plain; a list that a layer keeps whole
// goes past the stages where it is short.  Bound by vector instructions (some 27 of 64 entries and layer in stage 1, as many for its
// passers).  A quarter of the papers100M shape: one layer 305 us and 176 now, two layers 315 and 253 (blend_scan.h says what changed).
template <int NF, bool EXACT>
__global__ __launch_bounds__(kWave, NF == 1 ? 7 : NF == 2 ? 6 : NF == 3 ? 5 : 4) void
k_labor_scan_blend(const int32_t* __restrict__ g_indices, const Segment* __restrict__ seg, const uint32_t* __restrict__ thr_all,
                   const PreThr* __restrict__ pthr_all, const float* __restrict__ lim2_all, int64_t n, Dealing deal, FusedKeys keys, uint32_t stage_cap,
                   ScanOut out, Ctl* ctl, int piece_blocks, const Piece* __restrict__ pieces, const uint32_t* __restrict__ piece_count,
                   uint32_t piece_cap, CandOut cand, uint32_t stretch) {
  __shared__ BlendQueue<false> queue[NF];
  const uint32_t lane = (uint32_t)lane_id();
  auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
  auto of64 = [&](int64_t x, int q) { return (int64_t)(((uint64_t)of((uint32_t)((uint64_t)x >> 32), q) << 32) | of((uint32_t)x, q)); };
  BlendScan<NF, false, LaborSink<EXACT>> S;
  S.queue = queue;
  S.cwf = (float)keys.cw;
  S.swf = (float)keys.sw;
  S.sink = LaborSink<EXACT>{out, cand, ctl, stage_cap, 0u, 0u, false, thr_all, n, keys.cw, keys.sw};
#pragma unroll
  for (int l = 0; l < NF; ++l) S.set_keys(l, keys.K[l]);
  if ((int)blockIdx.x < piece_blocks) {
    uint32_t n_pieces = *piece_count;
    if (n_pieces > piece_cap) n_pieces = piece_cap;
    for (uint32_t p = blockIdx.x; p < n_pieces; p += (uint32_t)piece_blocks) {
      const Piece pc = pieces[p];
      const uint32_t list = of(pc.list, 0), q = of(pc.q, 0);
      if (list == kNoPiece) continue;
      const Segment g = seg[list];
      const int64_t beg = of64(g.beg, 0);
      uint32_t len;
      const int64_t j0 = piece_start(of(g.d, 0), of(g.split, 0), q, &len);
      if (j0 < 0) continue;
      S.sink.first = list;  // (every lane has this list's thresholds: slot 0)
      uint32_t a1[NF], a2[NF], b2[NF];
#pragma unroll
      for (int l = 0; l < NF; ++l) {
        const PreThr pt = pthr_all[(int64_t)l * n + list];
        a1[l] = of(pt.a1, 0) | 0xFFFFu;
        a2[l] = of(pt.a2, 0) | 0xFFFFu;
        b2[l] = of(pt.b2, 0) | 0xFFFFu;
        queue[l].keep2[lane] = pt.keep2;
        queue[l].lim2[lane] = lim2_all[(int64_t)l * n + list];
      }
      ListReader<> L(g_indices + beg + j0, len);
      S.collect(L, (uint32_t)j0, 0u, a1, a2, b2);
      S.flush();
    }
    return;
  }
  int each_log2;
  const int64_t w0 = deal.first_list(blockIdx.x - (uint32_t)piece_blocks, &each_log2);
  if (w0 >= n) return;
  const uint32_t n_mine = n - w0 < ((int64_t)1 << each_log2) ? (uint32_t)(n - w0) : 1u << each_log2;
  const uint32_t lanes = 64u >> each_log2, sub = lane & (lanes - 1), number = lane >> (6 - each_log2);
  const int64_t w = w0 + (number < n_mine ? number : n_mine - 1);
  S.sink.owns = true;
  S.sink.first = (uint32_t)w0;
  S.sink.shift = (uint32_t)(6 - each_log2);
  const Segment g = seg[w];
  uint32_t my_a1[NF], my_a2[NF], my_b2[NF];
#pragma unroll
  for (int l = 0; l < NF; ++l) {
    const PreThr pt = pthr_all[(int64_t)l * n + w];
    my_a1[l] = pt.a1 | 0xFFFFu;
    my_a2[l] = pt.a2 | 0xFFFFu;
    my_b2[l] = pt.b2 | 0xFFFFu;
    queue[l].keep2[lane] = pt.keep2;
    queue[l].lim2[lane] = lim2_all[(int64_t)l * n + w];
    queue[l].own[lane] = 0;
  }
  const bool live = number < n_mine && g.split == 0, speaks = live && sub == 0;
  const uint32_t together = each_log2 != 0 ? 2 * lanes : 0;
  if (ballot64(live && g.d <= together && g.d != 0) != 0) {
    const bool mine = live && g.d <= together;
    uint32_t t[2] = {0, 0};
#pragma unroll
    for (int r = 0; r < 2; ++r)
      if (mine && sub + r * lanes < g.d) t[r] = (uint32_t)(g_indices + g.beg)[sub + r * lanes];
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      const bool all = queue[l].keep2[lane] == __builtin_inff();  // (nothing of such a list goes through the stages)
      uint64_t m[4] = {0, 0, 0, 0};
#pragma unroll
      for (uint32_t r = 0; r < 2; ++r) {
        const uint32_t j = sub + r * lanes;
        const bool in = mine && j < g.d;
        if (in && all && j < stage_cap) out.stage[l][(size_t)w * stage_cap + j] = StageEntry{(int32_t)t[r], j};
        m[r] = S.passes(l, t[r], my_a1[l], my_a2[l], my_b2[l]) & ballot64(in && !all);
      }
      if (all && mine && sub == 0) queue[l].own[lane] = g.d;
      const uint32_t both[4] = {t[0], t[1], 0u, 0u};
      S.join(l, both, m, sub, lanes, lane & ~(lanes - 1));
    }
  }
  // A longer list that every layer keeps whole: counted, and as much of it copied as a row holds.
  bool whole = live && g.d > together;
#pragma unroll
  for (int l = 0; l < NF; ++l) whole = whole && queue[l].keep2[lane] == __builtin_inff();
  if (whole) {
    for (uint32_t j = sub; j < g.d && j < stage_cap; j += lanes) {
      const int32_t t = (g_indices + g.beg)[j];
#pragma unroll
      for (int l = 0; l < NF; ++l) out.stage[l][(size_t)w * stage_cap + j] = StageEntry{t, j};
    }
    if (sub == 0) {
#pragma unroll
      for (int l = 0; l < NF; ++l) queue[l].own[lane] = g.d;
    }
  }
  uint64_t todo = ballot64(speaks && g.d > together && !whole);
  if (todo != 0) {
    int at = __builtin_ctzll(todo);
    uint32_t d = of(g.d, at), j0 = 0, a1[NF], a2[NF], b2[NF];
    int64_t beg = of64(g.beg, at);
    auto thresholds = [&]() {
#pragma unroll
      for (int l = 0; l < NF; ++l) { a1[l] = of(my_a1[l], at); a2[l] = of(my_a2[l], at); b2[l] = of(my_b2[l], at); }
    };
    thresholds();
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
        thresholds();
      }
      L = ListReader<>(g_indices + beg + j0, d - j0 < stretch ? d - j0 : stretch);
    }
  }
  S.flush();
  if (speaks) {
#pragma unroll
    for (int l = 0; l < NF; ++l) {
      const uint32_t kept = queue[l].own[lane];
      out.cnt[l][w] = (int32_t)kept;  // (the exact stage adds what it keeps)
      // (one atomic a wave: by 70 thousand lists one at a time, all on one word, a scan of 34 M entries took 0.84 ms, and 0.3 so)
      if (kept > stage_cap) atomicAdd(&ctl->n_overflow, 1);
    }
  }
}

// Stage 3 of the blended path: the exact blend for every candidate the scan kernel appended, one candidate per thread
// (grid-stride; the count is read from device memory).  A kept edge takes the next free slot of its destination's
// staging row.
__global__ __launch_bounds__(kBlock) void k_labor_exact(CandOut cand, const uint32_t* __restrict__ thr_all, int64_t n, int nf, FusedKeys keys,
                                                        uint32_t stage_cap, ScanOut out, Ctl* ctl) {
  uint32_t total = cand.count[blockIdx.y];  // blockIdx.y: the sub-buffer
  if (total > cand.cap_each) total = cand.cap_each;
  const Cand* __restrict__ mine = cand.buf + (size_t)blockIdx.y * cand.cap_each;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < total; i += (uint64_t)gridDim.x * kBlock) {
    const Cand e = mine[i];
    if (e.layer >= (uint32_t)nf || (int64_t)e.list >= n) continue;  // (never: the scan kernel wrote it)
    LayerKeys K = keys.K[0];
    int32_t* cnt = out.cnt[0];
    StageEntry* stage = out.stage[0];
#pragma unroll
    for (int f = 1; f < kMaxFuse; ++f)
      if (e.layer == (uint32_t)f) { K = keys.K[f]; cnt = out.cnt[f]; stage = out.stage[f]; }
    const uint32_t thr = thr_all[(int64_t)e.layer * n + e.list];
    const double n1 = kit_phi_inv_u32(keyed_uniform<false>(K.Ka, (uint32_t)e.t, 0u));
    const double n2 = kit_phi_inv_u32(keyed_uniform<false>(K.Kb, (uint32_t)e.t, 0u));
    const uint32_t R = kit_phi_to_u32(__builtin_fma(keys.cw, n1, keys.sw * n2));
    if (R <= thr) {
      const uint32_t at = (uint32_t)atomicAdd(&cnt[e.list], 1);
      if (at < stage_cap) stage[(size_t)e.list * stage_cap + at] = StageEntry{e.t, e.j};
      else if (at == stage_cap) atomicAdd(&ctl->n_overflow, 1);  // exactly one entry sees the row fill up
    }
  }
}

__global__ void k_enum_redo(Ctl* ctl, uint32_t* piece_count) {
  ctl->cand_overflow = 0;
  *piece_count = 0;
}

__global__ void k_labor_redo(Ctl* ctl, uint32_t* piece_count, uint32_t* cand_count) {  // kCandSub threads
  if (threadIdx.x == 0) {
    ctl->cand_overflow = 0;
    *piece_count = 0;
  }
  cand_count[threadIdx.x] = 0;
}

// staged rows -> the block's edge arrays: 2^LOG2 neighbouring threads per destination, each taking every 2^LOG2-th slot
constexpr int kFillOwnBlock = 1024;  // where a block adds up the counts in front of it: fewer and larger ones
// Four threads per destination where there are many: the rows of 464 thousand destinations 43.6 us with eight, 56 with sixteen, 50 with
// two, 35.9 with four (41.8 and 37.3 before a lane ranked its four slots in one go over the positions).  Sixteen where a block adds up
// the counts in front of it: there it is the wait for memory that counts, and more blocks share the work (264 destinations 7.4 us with
// eight, 6.1; 16,384 of them 9.1 and 7.9), up to the number from which adding up costs more (30 thousand 9.9 and 11.0).
constexpr int kFillLog2 = 2, kFillOwnLog2 = 3, kFillFewLog2 = 4;
constexpr int64_t kFillFew = 20480;
// (edge_limit: entries of col_global / eid; nothing is written beyond them)
template <bool OWN, int BLOCK, int LOG2>
__global__ __launch_bounds__(BLOCK) void k_labor_fill_staged(LayerChunks ch, CountOffsets co, int64_t first, int64_t n_dst, uint32_t stage_cap,
                                                             EdgeOut edges, int64_t edge_limit) {
  __shared__ uint32_t row_j[BLOCK >> LOG2][kWave];  // list positions of one staged row per lane group
  const int64_t idx = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const int64_t w = first + (idx >> LOG2);
  // What is known of the destination is requested ahead of its offset and count, and so is as much of its row as nearly all hold.
  const int64_t w_in = w < n_dst ? w : n_dst - 1;
  const Segment* seg = ch.seg[0];
  const StageEntry* stage = ch.stage[0];
  int64_t start = ch.start[0];
#pragma unroll
  for (int q = 1; q < kMaxFuse; ++q)  // (see chunk_at)
    if (q < ch.n_chunks && w_in >= ch.start[q]) {
      seg = ch.seg[q];
      stage = ch.stage[q];
      start = ch.start[q];
    }
  const int64_t local = w_in - start;
  const StageEntry* __restrict__ row = stage + (size_t)local * stage_cap;
  const int64_t beg = seg[local].beg;
  const int sub = (int)(idx & ((1 << LOG2) - 1));
  constexpr int kPerLane = kWave >> LOG2, kAhead = 16 >> LOG2;
  StageEntry mine[kPerLane];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    const int slot = sub + (i << LOG2);
    mine[i] = row[slot < (int)stage_cap ? slot : 0];
  }
  int32_t c;
  const int64_t o = offset_of<OWN, BLOCK, LOG2>(co, w, n_dst, &c);
  if (w >= n_dst) return;
  if (c > (int32_t)stage_cap) return;  // overflowed row: the overflow pass writes these edges
  // A row may hold its entries in any order (the pieces of a cut list, the lists found from the other side and the
  // blended passes take slots by atomics): an entry's place is its rank by list position.  The lane group (all in one
  // wave) shares the positions through LDS.  The rows that k_labor_scan_plain leaves in list order, those of uncut lists, go the
  // same way: two paths side by side in a wave cost more than ranking a dozen entries.
  uint32_t* js = row_j[threadIdx.x >> LOG2];
#pragma unroll
  for (int i = 0; i < kPerLane; ++i) {
    const int slot = sub + (i << LOG2);
    if (i >= kAhead) mine[i] = StageEntry{0, 0u};
    if (slot < c) {  // (only js[0..c) is read below)
      if (i >= kAhead) mine[i] = row[slot];
      js[slot] = mine[i].j;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int kTogether = kAhead;  // slots of a lane whose ranks are counted together
#pragma unroll
  for (int i0 = 0; i0 < kPerLane; i0 += kTogether) {
    if (sub + (i0 << LOG2) >= c) break;
    uint32_t place[kTogether];
#pragma unroll
    for (int i = 0; i < kTogether; ++i) place[i] = 0;
    for (int q = 0; q < c; ++q) {
      const uint32_t j = js[q];
#pragma unroll
      for (int i = 0; i < kTogether; ++i) place[i] += j < mine[i0 + i].j;
    }
#pragma unroll
    for (int i = 0; i < kTogether; ++i)
      if (sub + ((i0 + i) << LOG2) < c && o + (int64_t)place[i] < edge_limit) put_edge(edges, o, place[i], mine[i0 + i].t, beg + mine[i0 + i].j);
  }
}

// second, ordered scan of the (rare) destinations whose staging row overflowed, writing straight to the edge arrays
template <bool BLEND>
__global__ __launch_bounds__(kBlock) void k_labor_fill_overflow(const int32_t* __restrict__ g_indices, LayerChunks ch, int64_t first, int64_t n_dst,
                                                                LayerKeys K, double cw, double sw, uint32_t stage_cap,
                                                                const int64_t* __restrict__ eptr, int32_t* __restrict__ col_global,
                                                                 int64_t* __restrict__ eid) {
  const int64_t w = first + (int64_t)blockIdx.x * kWavesPerBlock + uniform_wave_in_block();
  if (w >= n_dst) return;
  const int64_t o = eptr[w];
  if (eptr[w + 1] - o <= (int64_t)stage_cap) return;
  const int p = ch.find(w);
  const int64_t local = w - ch.start[p];
  const Segment g = ch.seg[p][local];
  const uint32_t thr = ch.thr[p][local];
  labor_scan_ordered<BLEND>(g_indices, g.beg, g.d, thr, K, cw, sw, [&](uint32_t rank, int32_t t, uint32_t j) {
    // (no tag: this pass comes behind a read-back, and the dedup of such a layer reads keys)
    col_global[o + rank] = t;
    eid[o + rank] = g.beg + j;
  });
}

static void launch_scan_blend(int nf, unsigned blocks, hipStream_t s, const int32_t* indices, const Segment* seg, const uint32_t* thr, const PreThr* pthr,
                              const float* lim2, int64_t n, const Dealing& deal, const FusedKeys& keys, uint32_t cap, const ScanOut& out, Ctl* ctl,
                              int piece_blocks, const Piece* pieces, const uint32_t* piece_count, uint32_t piece_cap,
                              const CandOut& cand /* no buffer: the exact blend in the scan */) {
#define COOP_SCAN_BLEND(NF)                                                                                                                  \
  if (cand.buf != nullptr) { COOP_SCAN_BLEND_AS(NF, false); } else { COOP_SCAN_BLEND_AS(NF, true); }
#define COOP_SCAN_BLEND_AS(NF, EXACT)                                                                                                        \
  COOP_LAUNCH(K_LABOR_COUNT, (k_labor_scan_blend<NF, EXACT>), dim3(blocks), dim3(kWave), 0, s, indices, seg, thr, pthr, lim2, n, deal, keys, cap, out, ctl, \
              piece_blocks, pieces, piece_count, piece_cap, cand, (uint32_t)g_stretch)
  switch (nf) {
    case 1: COOP_SCAN_BLEND(1); break;
    case 2: COOP_SCAN_BLEND(2); break;
    case 3: COOP_SCAN_BLEND(3); break;
    default: COOP_SCAN_BLEND(4); break;
  }
#undef COOP_SCAN_BLEND_AS
#undef COOP_SCAN_BLEND
}
static void launch_scan_plain(int nf, unsigned blocks, hipStream_t s, const int32_t* indices, const Segment* seg, const uint32_t* thr, int64_t n, const Dealing& deal,
                              const FusedKeys& keys, uint32_t cap, const ScanOut& out, Ctl* ctl, int piece_blocks, const Piece* pieces,
                              const uint32_t* piece_count, uint32_t piece_cap) {
#define COOP_SCAN_PLAIN(NF)                                                                                                           \
  COOP_LAUNCH(K_LABOR_COUNT, k_labor_scan_plain<NF>, dim3(blocks), dim3(kWave), 0, s, indices, seg, thr, n, deal, keys, cap, out, ctl, \
              piece_blocks, pieces, piece_count, piece_cap, (uint32_t)g_stretch)
  switch (nf) {
    case 1: COOP_SCAN_PLAIN(1); break;
    case 2: COOP_SCAN_PLAIN(2); break;
    case 3: COOP_SCAN_PLAIN(3); break;
    default: COOP_SCAN_PLAIN(4); break;
  }
#undef COOP_SCAN_PLAIN
}

// One round of resident waves; fewer where there cannot be as many pieces.  (Starting 8,192 that find nothing costs a pass over a few
// hundred lists 2 us.)
constexpr int64_t kPieceWaves = 8192;
// Destinations per wave, as a power of two: products-, papers100M-shaped and dependent steps 677, 1105 and 1043 us by this rule, 677,
// 1103 and 1045 with four in every pass, 680, 1114 and 1046 with eight, 698, 1131 and 1072 with sixteen; the reddit-shaped step with a
// cache, passes of a few thousand lists: 271 by this rule (one), 284 with four.
constexpr int64_t kScanWaves = 16384;
constexpr int kScanEachLog2 = 3;

int labor_layer(LaborState& st, const SampleCtx& cx, int l, const int32_t* dst, int64_t n_dst, coop_block* blk, int64_t edge_cap) {
  const bool defer = edge_cap > 0;
  hipStream_t s = cx.s;
  Alloc& alloc = *cx.alloc;
  if (l == 0) {
    // fuse when every remaining layer fits one scan (GNNs have 2-3 layers); otherwise scan layer by layer
    st.fuse = cx.L <= kMaxFuse && g_fuse_layers != 0;
    uint32_t kmax = 0;
    for (int i = 0; i < cx.L; ++i) kmax = (uint32_t)cx.fanouts[i] > kmax ? (uint32_t)cx.fanouts[i] : kmax;
    // staging rows: room for 2k + 16 kept edges (a row overflows with probability < 1e-8 at k = 10), 32 or 64 entries
    // (what one wave parks in a register pair); a row that overflows is redone by the overflow pass
    st.stage_cap = 2 * (uint64_t)kmax + 16 > 32 ? 64 : 32;
    if (g_stage_cap_override) st.stage_cap = (uint32_t)g_stage_cap_override;
    st.n_pass = 0;
    st.covered = 0;
  }
  const uint32_t cap = st.stage_cap;

  // ---- scan pass over the destinations not covered yet ------------------------------------------------------------
  // Normally the pass evaluates every remaining layer and is recorded.  A pass over only a few lists (the seeds'
  // hop) is not worth a many-layer kernel: it evaluates this layer alone and leaves its destinations to the next pass.
  constexpr int64_t kFuseMinLists = 32768;
  const bool record = st.fuse && (n_dst - st.covered >= kFuseMinLists || l == cx.L - 1 || g_fuse_layers == 2);
  LaborPass local;
  LaborPass& ps = record ? st.pass[st.n_pass] : local;
  ps.first_layer = l;
  ps.start = st.covered;
  ps.n_new = n_dst - ps.start;
  ps.nf = record ? cx.L - l : 1;
  const int64_t n_new = ps.n_new;
  ps.seg = alloc.get<Segment>(n_new, COOP_TAG_SCRATCH);
  ps.thr = alloc.get<uint32_t>(n_new * ps.nf, COOP_TAG_SCRATCH);
  PreThr* pthr = cx.blend ? alloc.get<PreThr>(n_new * ps.nf, COOP_TAG_SCRATCH) : nullptr;
  float* lim2 = cx.blend ? alloc.get<float>(n_new * ps.nf, COOP_TAG_SCRATCH) : nullptr;
  for (int f = 0; f < ps.nf; ++f) {
    ps.stage[f] = alloc.get<StageEntry>(n_new * (int64_t)cap, COOP_TAG_SCRATCH);
    ps.cnt[f] = alloc.get<int32_t>(n_new, COOP_TAG_SCRATCH);
  }
  blk->indptr = alloc.get<int64_t>(n_dst + 1, COOP_TAG_OUTPUT);
  if (alloc.failed) return COOP_E_NOMEM;

  FusedKeys keys{};
  keys.cw = cx.cw;
  keys.sw = cx.sw;
  uint32_t ks[kMaxFuse] = {1, 1, 1, 1};
  for (int f = 0; f < ps.nf; ++f) {
    layer_keys(cx.seed, COOP_LABOR0, l + f, cx.group, keys.K[f].Ka);
    layer_keys(cx.seed, COOP_LABOR0, l + f, cx.group + 1, keys.K[f].Kb);
    ks[f] = (uint32_t)cx.fanouts[l + f];
  }
  // A call on unaligned indices takes memory for neither the queue nor the candidates of the exact blend (programs sized their
  // arenas for such calls when every list was read by one wave, an entry at a time): its queue lies in an array of the layer that is
  // written after the scan, with as many pieces as that holds, and the scan evaluates the exact blend itself.  (A list of 2 million
  // entries among 20 thousand short ones: 82 us with pieces, 1.9 ms without.)
  Piece* pieces = nullptr;
  if (!cx.vec4 && defer) blk->eid = alloc.get<int64_t>(edge_cap, COOP_TAG_OUTPUT);
  if (alloc.failed) return COOP_E_NOMEM;
  // long lists are cut into pieces, which k_segments queues
  int64_t piece_room = 0;
  const Degrees degrees = cx.g->degrees();
  const PieceCut cut = cut_pieces(n_new, degrees, cx.blend, g_piece_len, g_split_min, cx.vec4 ? (int64_t)1 << 30 : defer ? edge_cap : n_dst + 1, &piece_room);
  const uint32_t piece_cap = (uint32_t)piece_room;
  if (cut.len != 0) {
    static_assert(sizeof(Piece) == sizeof(int64_t), "a piece takes the place of an offset or a position");
    pieces = cx.vec4 ? alloc.get<Piece>(piece_cap, COOP_TAG_SCRATCH) : (Piece*)(defer ? blk->eid : blk->indptr);
    if (alloc.failed) return COOP_E_NOMEM;
  }
  // blended variates: stage 3 works from a buffer of the candidates that the fp32 blend left undecided, a few percent
  // of the k kept edges per destination and layer; k / 2 each is ample (a pass that overflows it is redone with more)
  const bool queued = cx.blend && cx.vec4 && n_new > 0;
  int64_t cand_cap = 0;
  uint32_t* cand_count = nullptr;
  if (queued) {
    uint32_t kpass = 1;
    for (int f = 0; f < ps.nf; ++f) kpass = ks[f] > kpass ? ks[f] : kpass;
    cand_cap = g_blend_candidates ? g_blend_candidates : (int64_t)kpass * n_new * ps.nf / 2 + 65536;
    if (cand_cap > ((int64_t)1 << 30)) cand_cap = (int64_t)1 << 30;
    cand_count = alloc.get<uint32_t>(kCandSub, COOP_TAG_SCRATCH);
    if (alloc.failed) return COOP_E_NOMEM;
  }
  // ---- this layer's destinations, piece by piece: a recorded pass covered it as its (l - first_layer)-th layer ------
  if (record) { st.n_pass += 1; st.covered = n_dst; }
  LayerChunks ch{};
  ChunkedI32 counts{};
  int nc = 0;
  auto add_chunk = [&](const LaborPass& q) {
    if (q.n_new == 0) return;  // a pass that scanned nothing (a layer that added no vertex) contributes no piece
    const int f = l - q.first_layer;
    ch.seg[nc] = q.seg;
    ch.thr[nc] = q.thr + (int64_t)f * q.n_new;
    ch.stage[nc] = q.stage[f];
    ch.start[nc] = counts.start[nc] = q.start;
    counts.ptr[nc] = q.cnt[f];
    ++nc;
  };
  for (int p = 0; p < st.n_pass; ++p) add_chunk(st.pass[p]);
  if (!record) add_chunk(local);
  if (nc == 0) { ch.seg[0] = ps.seg; ch.thr[0] = ps.thr; ch.stage[0] = ps.stage[0]; counts.ptr[0] = ps.cnt[0]; nc = 1; }  // n_dst == 0
  ch.n_chunks = counts.n_chunks = nc;

  const bool own = defer && n_dst <= kScanOwn;  // the fill finds its offsets by itself
  // the tiles' sums lie in col_local, which nothing is written to before the dedup
  if (defer) blk->col_local = alloc.get<int32_t>(edge_cap, COOP_TAG_OUTPUT);
  if (alloc.failed) return COOP_E_NOMEM;
  int64_t* sums = defer && sums_ahead(n_dst) && edge_cap >= 2 * kTilesAhead ? (int64_t*)blk->col_local : nullptr;
  bool no_enum = false, used_enum = false;
  for (;;) {
    used_enum = false;
    if (n_new > 0) {
      ScanOut out{};
      for (int f = 0; f < ps.nf; ++f) { out.stage[f] = ps.stage[f]; out.cnt[f] = ps.cnt[f]; }
      CandOut cand{};
      if (queued) {
        cand.cap_each = (uint32_t)((cand_cap + kCandSub - 1) / kCandSub);
        cand.buf = alloc.get<Cand>((int64_t)cand.cap_each * kCandSub, COOP_TAG_SCRATCH);
        cand.count = cand_count;
        if (alloc.failed) return COOP_E_NOMEM;
      }
      // ---- the longest lists from the other side (see k_enum_list) ---------------------------------------------------
      uint32_t kmax_pass = 0;
      for (int f = 0; f < ps.nf; ++f) kmax_pass = ks[f] > kmax_pass ? ks[f] : kmax_pass;
      // (listing and walking cost the same whatever the number of destinations and the shape of the graph: it pays only
      // for a pass over many lists of a graph whose long lists hold a good part (an eighth, here) of the edges; a knob
      // value below the default is for tests and applies always)
      const bool enough = g_enum_degree < kLongListDegree || (n_new >= 65536 && cx.g->long_mass * 8 >= cx.g->n_edges);
      const uint32_t enum_degree = cx.g->symmetric && !cx.blend && !no_enum && kmax_pass <= 64 && enough ? (uint32_t)g_enum_degree : 0u;
      used_enum = enum_degree != 0;
      LongSlot* long_tab = nullptr;
      uint32_t* long_bits = nullptr;
      uint32_t long_mask = 0;
      EnumOut eo{};
      uint32_t u_max[kMaxFuse] = {0, 0, 0, 0}, um_most = 0, list_todo = 0;
      if (enum_degree != 0) {
        // the table of long destinations: twice the number there can be (|E| / D lists are that long, at most), but no
        // more than 65536 slots or a quarter of the destinations, whichever is more: the table then stays in L2, and a
        // pass with more long lists than that is redone the ordinary way
        int64_t most = cx.g->n_edges / enum_degree + 1;
        if (most > n_new) most = n_new;
        const int64_t ceiling = n_new / 4 > 65536 ? n_new / 4 : 65536;
        uint32_t slots = 1024;
        while ((int64_t)slots < 2 * most && (int64_t)slots * 2 <= ceiling) slots <<= 1;
        long_mask = slots - 1;
        constexpr int64_t kBitSlots = kLongBits / 8 / sizeof(LongSlot);
        uint32_t* zeroed = (uint32_t*)alloc.get<LongSlot>(1 + kBitSlots + (int64_t)slots, COOP_TAG_SCRATCH);  // counters, bits, table
        long_bits = (uint32_t*)((LongSlot*)zeroed + 1);
        long_tab = (LongSlot*)zeroed + 1 + kBitSlots;
        // The vertices listed for a layer depend on the layer's keys and fanout only: a later pass that covers the same
        // layer (the pass at layer 2 after the pass at layer 1 that covered layers 1 and 2) walks the same items.
        for (int f = 0; f < ps.nf; ++f) {
          u_max[f] = (uint32_t)(((uint64_t)ks[f] << 32) / ((uint64_t)enum_degree + 1));
          LaborState::Listed* had = l + f < LaborState::kMaxListed ? &st.listed[l + f] : nullptr;
          if (had != nullptr && had->item != nullptr && had->u_max == u_max[f]) {
            eo.item[f] = had->item;
            eo.n_item[f] = had->n;
            eo.item_cap[f] = had->cap;
            continue;
          }
          // items: a listed vertex gives d / kEnumItem + 1 of them; the listed vertices' lists hold |E| u_max / 2^32
          // entries in expectation, and four times that is allowed for (a pass that needs more, because some huge hub is
          // listed, is redone the ordinary way)
          const double expect = (double)cx.g->n_vertices * ((double)u_max[f] + 1.0) / 4294967296.0;  // listed vertices
          const double entries = (double)cx.g->n_edges * ((double)u_max[f] + 1.0) / 4294967296.0;
          const double items = expect + 8.0 * sqrt(expect) + 1024.0 + 4.0 * entries / kEnumItem;
          eo.item_cap[f] = (uint32_t)(items < 268435456.0 ? items : 268435456.0);
          eo.item[f] = alloc.get<EnumItem>(eo.item_cap[f], COOP_TAG_SCRATCH);
          eo.n_item[f] = zeroed + f;
          list_todo |= 1u << f;
          um_most = u_max[f] > um_most ? u_max[f] : um_most;
          if (had != nullptr) *had = LaborState::Listed{eo.item[f], eo.n_item[f], eo.item_cap[f], u_max[f]};
        }
        for (int f = ps.nf; f < kMaxFuse; ++f) { eo.item[f] = eo.item[0]; eo.n_item[f] = eo.n_item[0]; eo.item_cap[f] = 0; }
        if (alloc.failed) return COOP_E_NOMEM;
        fill_u64((uint64_t*)zeroed, (1 + kLongBits / 8 / sizeof(LongSlot) + (int64_t)slots) * (sizeof(LongSlot) / 8), 0, s);
      }
      const Clear clear = take_clear(cx);
#define COOP_SEGMENTS(BLOCK, EACH, SHARED)                                                                                            \
  do {                                                                                                                                \
    const Begin begin = take_begin(cx, blocks_for(n_new, EACH));                                                                      \
    COOP_LAUNCH(K_SEGMENTS, (k_segments<BLOCK, SHARED>), dim3(blocks_for(n_new, EACH)), dim3(BLOCK), 0, s, cx.g->indptr, cx.g->n_vertices,  \
                dst + ps.start, n_new, ps.nf, ks[0], ks[1], ks[2], ks[3], ps.seg, ps.thr, pthr, lim2, cx.cw, cx.sw,                      \
                cx.d_ctl, cut, pieces, piece_cap, cx.d_piece_count + l, out, enum_degree,    \
                long_bits, long_tab, long_mask, clear, begin, cand_count);                                                             \
  } while (0)
      if (n_new >= kSegWideFrom) COOP_SEGMENTS(1024, 1024, false);
      else if (n_new >= kSegSharedBelow || !cx.blend) COOP_SEGMENTS(256, 256, false);
      else COOP_SEGMENTS(3 * kWave, kWave, true);
#undef COOP_SEGMENTS
      if (enum_degree != 0) {
        if (list_todo != 0) {
          const unsigned list_blocks = blocks_for((int64_t)um_most + 1, kEnumListSpan);
          COOP_LAUNCH(K_ENUM_LIST, k_enum_list, dim3(list_blocks, ps.nf), dim3(kListBlock), 0, s, keys, u_max[0], u_max[1], u_max[2], u_max[3],
                      cx.g->n_vertices, cx.g->indptr, eo, cx.d_ctl, list_todo);
        }
        // (three blocks fit a CU: one round of resident blocks strides over the items)
        uint32_t cap_most = 0;
        for (int f = 0; f < ps.nf; ++f) cap_most = eo.item_cap[f] > cap_most ? eo.item_cap[f] : cap_most;
        const int64_t walk_blocks = blocks_for((int64_t)cap_most * 16, kWalkBlock);
        COOP_LAUNCH(K_ENUM_WALK, k_enum_walk, dim3((unsigned)(walk_blocks < 768 ? walk_blocks : 768), ps.nf), dim3(kWalkBlock), 0, s,
                    cx.g->indices, (const uint32_t*)cx.g->rev_pos, (const uint32_t*)long_bits, (const LongSlot*)long_tab, long_mask, cap, out,
                    eo, cx.d_ctl);
      }
      // the piece waves come first in the grid: one round of resident blocks, fewer if there cannot be that many pieces
      int64_t piece_waves = (int64_t)piece_cap < kPieceWaves ? (int64_t)piece_cap : kPieceWaves;
      if (cut.len != 0) {
        const int64_t most = degrees.pieces(n_new, cut.split_min, cut.len);
        if (most < piece_waves) piece_waves = most;
      }
      const uint32_t* pcount = cx.d_piece_count + l;
      // destinations per wave: up to eight, where that leaves kScanWaves waves (the knob overrides, the next power of two)
      int each_log2 = 0;
      if (g_lists_per_wave != 0) while ((1 << each_log2) < g_lists_per_wave) ++each_log2;
      else while (each_log2 < kScanEachLog2 && (n_new >> (each_log2 + 1)) >= kScanWaves) ++each_log2;
      while (each_log2 < 6 && (n_new >> each_log2) > kSliceLists / 2) ++each_log2;  // (no more waves than a launch can have)
      const Dealing deal = deal_lists(n_new, each_log2, g_lists_per_wave != 0 || finer_last(degrees, each_log2, l > 0));
      const unsigned blocks = deal.blocks + (unsigned)piece_waves;
      if (cx.blend)
        launch_scan_blend(ps.nf, blocks, s, cx.g->indices, ps.seg, ps.thr, pthr, lim2, n_new, deal, keys, cap, out, cx.d_ctl, (int)piece_waves,
                          pieces, pcount, piece_cap, cand);
      else
        launch_scan_plain(ps.nf, blocks, s, cx.g->indices, ps.seg, ps.thr, n_new, deal, keys, cap, out, cx.d_ctl, (int)piece_waves, pieces,
                          pcount, piece_cap);
      if (queued) {  // stage 3: the exact blend for the candidates that the scan appended
        // (Blocks for an eighth of what the first covered layer's fanout keeps in every layer, where a few percent are undecided, at most
        // 16 a sub-buffer; the threads stride, so more candidates only take longer.  By the sum of the fanouts it is no better: 300 thousand
        // destinations, fanouts 1 and 25, 25.4 us so and 30.8 with seven times the blocks, 100 thousand and 1, 1, 25 28.8 and 26.6.  With as many blocks as the buffers have room for, 4,096, a launch over 113 thousand destinations
        // and two layers took 19.9 us and one over 463 thousand 19.6, most of it for blocks with nothing to do; now 7.5 and 10.1.)
        const int64_t expected = ((int64_t)ks[0] * n_new * ps.nf) / 8;
        const int64_t each = (expected / kCandSub + kBlock - 1) / kBlock + 1;
        const unsigned blocks = (unsigned)(each < 16 ? each : 16);
        COOP_LAUNCH(K_LABOR_EXACT, k_labor_exact, dim3(blocks, kCandSub), dim3(kBlock), 0, s, cand, ps.thr, n_new, ps.nf, keys, cap, out,
                    cx.d_ctl);
      }
    }

    if (defer) {  // the count stays on the device; an overflow of the candidate buffer is the caller's to notice
      if (sums != nullptr) scan_in_tiles(counts, n_dst, blk->indptr, sums, s);
      else if (!own) scan_tiles(counts, n_dst, blk->indptr, &cx.d_ctl->total_edges, cx.d_ctl, s);
      break;
    }
    const Publish pub = begin_publish(cx.d_ctl, cx.h_ctl);  // the scan's last thread also sends the sizes to the host
    scan_tiles(counts, n_dst, blk->indptr, &cx.d_ctl->total_edges, cx.d_ctl, s, &pub);  // m_l = indptr[n_dst]
    const int rc = wait_ctl(pub, cx.h_ctl, s);
    if (rc != COOP_OK) return rc;
    if (used_enum && cx.h_ctl->cand_overflow != 0) {  // the lists of the listed vertices did not fit: once more, every list scanned
      no_enum = true;
      for (auto& had : st.listed) had = LaborState::Listed{};  // (what was listed may be incomplete)
      hipLaunchKernelGGL(k_enum_redo, dim3(1), dim3(1), 0, s, cx.d_ctl, cx.d_piece_count + l);
      continue;
    }
    if (!queued || cx.h_ctl->cand_overflow == 0) break;
    // the candidate buffer of the exact stage was too small (counts are incomplete): once more with 8 times the room
    if (cand_cap >= ((int64_t)1 << 30)) return COOP_E_CAPACITY;
    cand_cap = cand_cap * 8 < ((int64_t)1 << 30) ? cand_cap * 8 : ((int64_t)1 << 30);
    hipLaunchKernelGGL(k_labor_redo, dim3(1), dim3(kCandSub), 0, s, cx.d_ctl, cx.d_piece_count + l, cand_count);
  }
  const int64_t m = defer ? edge_cap : cx.h_ctl->total_edges;  // entries of the edge arrays
  blk->n_edges = defer ? -1 : m;
  blk->col_global = alloc.get<int32_t>(m, COOP_TAG_OUTPUT);
  if (cx.vec4 || !defer) blk->eid = alloc.get<int64_t>(m, COOP_TAG_OUTPUT);
  if (!defer) blk->col_local = alloc.get<int32_t>(m, COOP_TAG_OUTPUT);
  if (alloc.failed) return COOP_E_NOMEM;

  const EdgeOut edges{blk->col_global, blk->eid, cx.tags};
  if (m > 0 && n_dst > 0) {
    constexpr int64_t kSliceRows = kSliceLists << (6 - kFillLog2);
    const CountOffsets co{counts, blk->indptr, &cx.d_ctl->total_edges, sums};
    if (own && n_dst <= kFillFew)
      COOP_LAUNCH(K_LABOR_FILL, (k_labor_fill_staged<true, kFillOwnBlock, kFillFewLog2>), dim3(blocks_for(n_dst << kFillFewLog2, kFillOwnBlock)),
                  dim3(kFillOwnBlock), 0, s, ch, co, (int64_t)0, n_dst, cap, edges, m);
    else if (own)
      COOP_LAUNCH(K_LABOR_FILL, (k_labor_fill_staged<true, kFillOwnBlock, kFillOwnLog2>), dim3(blocks_for(n_dst << kFillOwnLog2, kFillOwnBlock)),
                  dim3(kFillOwnBlock), 0, s, ch, co, (int64_t)0, n_dst, cap, edges, m);
    else
      for (int64_t b = 0; b < n_dst; b += kSliceRows)
        COOP_LAUNCH(K_LABOR_FILL, (k_labor_fill_staged<false, kBlock, kFillLog2>),
                    dim3(blocks_for((n_dst - b < kSliceRows ? n_dst - b : kSliceRows) << kFillLog2, kBlock)), dim3(kBlock), 0, s, ch, co, b, n_dst,
                    cap, edges, m);
    if (!defer && cx.h_ctl->n_overflow > 0) {
      LayerKeys K{};
      layer_keys(cx.seed, COOP_LABOR0, l, cx.group, K.Ka);
      layer_keys(cx.seed, COOP_LABOR0, l, cx.group + 1, K.Kb);
      for (int64_t b = 0; b < n_dst; b += kSliceLists) {
        const dim3 grid(blocks_for(n_dst - b < kSliceLists ? n_dst - b : kSliceLists, kWavesPerBlock));
        if (cx.blend)
          COOP_LAUNCH(K_LABOR_OVERFLOW, k_labor_fill_overflow<true>, grid, dim3(kBlock), 0, s, cx.g->indices, ch, b, n_dst, K, cx.cw, cx.sw,
                      cap, blk->indptr, blk->col_global, blk->eid);
        else
          COOP_LAUNCH(K_LABOR_OVERFLOW, k_labor_fill_overflow<false>, grid, dim3(kBlock), 0, s, cx.g->indices, ch, b, n_dst, K, cx.cw, cx.sw,
                      cap, blk->indptr, blk->col_global, blk->eid);
      }
    }
  }
  return COOP_OK;
}

}  // namespace coop
