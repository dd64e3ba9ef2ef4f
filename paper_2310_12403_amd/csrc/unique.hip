// Frontier dedup and relabelling (Eq. 2: S^{l+1} = S^l ∪ sampled sources).  Every edge's source vertex gets the FIRST
// position of that vertex in the list [S^l ; col_global]; a vertex is "new" exactly at the edge whose position equals that
// first position (and is not a seed position).  The new-flags are kept as a bit per edge; bit counts per 64-edge word, their
// scan inside a block's stretch and the scan of the stretches' totals give each new vertex its rank, hence its place
// n_dst + rank in S^{l+1}: the order is "S^l, then first appearance in col_global", independent of scheduling.
//
// First positions come from hash tables in LDS: a block owns the keys of one bucket of hash values, and all occurrences of
// a key share a bucket, so the minimum position found there is the global one.  The shortest lists: one block
// does everything (k_uniq_small).  Short lists: every block reads the whole list and picks its keys (k_uniq_filter).  Long lists: a partition brings each bucket's pairs together first.  A bucket
// with more distinct keys than its table serves sends the call to one open-addressing table in HBM (k_uniq_insert).
// The distinct keys are known once the first positions are, so the block that finishes last there sends the sizes to the
// host, and the host's wait and the setup of the next layer run beside the collecting and relabelling kernels.
#include "coop_internal.h"
#include "device_utils.h"

namespace coop {

constexpr uint64_t kEmptySlot = ~0ull;

// multiplicative (Fibonacci) hashing of the key to 32 bits, then multiply-high range reduction onto [0, cap)
__device__ __forceinline__ uint64_t slot_of_key(uint32_t key, uint64_t cap) {
  const uint32_t h = (uint32_t)(((uint64_t)key * 0x9E3779B97F4A7C15ull) >> 32);
  return ((uint64_t)h * cap) >> 32;
}

// (sizes, optional: says the exact number of edges, on the device; m is then the capacity of col)
__global__ __launch_bounds__(kBlock) void k_uniq_insert(const int32_t* __restrict__ dst, int64_t n_dst,
                                                        const int32_t* __restrict__ col, int64_t m, const Ctl* __restrict__ sizes,
                                                        unsigned long long* __restrict__ table, uint64_t cap, Ctl* ctl) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  m = edges_there(sizes, m);
  if (i >= n_dst + m) return;
  const uint32_t key = (uint32_t)(i < n_dst ? dst[i] : col[i - n_dst]);
  const unsigned long long mine = ((unsigned long long)key << 32) | (uint32_t)i;
  uint64_t h = slot_of_key(key, cap);
  for (;;) {
    unsigned long long cur = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (cur == kEmptySlot) {
      cur = atomicCAS(&table[h], (unsigned long long)kEmptySlot, mine);
      if (cur == kEmptySlot) return;  // claimed
    }
    if ((uint32_t)(cur >> 32) == key) {
      // an edge position above the one already recorded cannot lower it: no atomic needed (this is what keeps a
      // hub that shows up in thousands of lists from serialising thousands of atomics on one slot)
      if (i >= n_dst && cur < mine) return;
      const unsigned long long old = atomicMin(&table[h], mine);
      // two positions below n_dst with one key: the destination list holds a vertex twice
      if (i < n_dst && (int64_t)(uint32_t)old < n_dst) atomicOr(&ctl->err_dup, 1);
      return;
    }
    if (++h == cap) h = 0;  // the table is at most half full, so an empty slot or the key is always reached
  }
}

__device__ __forceinline__ uint32_t first_position(const unsigned long long* __restrict__ table, uint64_t cap, uint32_t key) {
  uint64_t h = slot_of_key(key, cap);
  for (;;) {
    const unsigned long long cur = table[h];
    if ((uint32_t)(cur >> 32) == key) return (uint32_t)cur;
    if (cur == kEmptySlot) return 0xFFFFFFFFu;  // not reachable for inserted keys
    if (++h == cap) h = 0;
  }
}

// first[e] = first position of col[e] in [S^l ; col]
__global__ __launch_bounds__(kBlock) void k_uniq_lookup(const int32_t* __restrict__ col, int64_t m, const Ctl* __restrict__ sizes,
                                                        const unsigned long long* __restrict__ table, uint64_t cap,
                                                        uint32_t* __restrict__ first) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  m = edges_there(sizes, m);
  if (e < m) first[e] = first_position(table, cap, (uint32_t)col[e]);
}

// ---- a bucket's table in LDS -------------------------------------------------------------------------------------
// Slots of 8 bytes (key << 32 | position), as in the table in HBM.  The table gives up at `most` distinct keys, with room
// left for one claim per thread under way, so that a probe always reaches an empty slot.  (The reads are relaxed atomics:
// volatile ones would become flat loads.  Keys and positions in separate 32-bit arrays were slower, and so were two or four insertions
// per thread that stay side by side until the last of them has its slot: 45 us for the 1,536 buckets of 5.8 M entries in the place of
// 36.  bucket_insert_many makes only the first tries side by side.)
struct BucketState { uint32_t claimed, full, dup; };
__device__ __forceinline__ uint32_t lds_read(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ uint32_t bucket_insert(unsigned long long* table, uint32_t slots, uint32_t most, uint32_t h, unsigned long long mine,
                                                  uint32_t nd, BucketState* st) {
  const uint32_t key = (uint32_t)(mine >> 32);
  const bool seed_pos = (uint32_t)mine < nd;
  for (;;) {
    unsigned long long cur = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (cur == kEmptySlot) {
      cur = atomicCAS(&table[h], (unsigned long long)kEmptySlot, mine);
      if (cur == kEmptySlot) {
        if (atomicAdd(&st->claimed, 1u) >= most) st->full = 1;
        return h;
      }
    }
    if ((uint32_t)(cur >> 32) == key) {
      if (!seed_pos && cur < mine) return h;  // (a hub that many lists keep lowers its position a few times, not every time)
      const unsigned long long old = atomicMin(&table[h], mine);
      if (seed_pos && (uint32_t)old < nd) st->dup = 1;  // S^l holds a vertex twice
      return h;
    }
    h = (h + 1) & (slots - 1);
  }
}
// N insertions of a thread into a table that cannot fill up (all of the block's together are at most three quarters of its slots).  The
// first tries go side by side and without a look at the slot; what did not find its slot goes on alone, by a step of its key's own (in
// steps of one a wave waits for the longest run of slots that any of its lanes meets).  A try is to be a dozen instructions: nothing is
// asked about a seed's position here (seed_twice tells afterwards), the claimed slots are counted in a register.  (10 thousand entries by
// one block: 49 us in steps of one, 42 with the seeds' question in every try, 10 so.  Buckets of 4,096 pairs: 28.2 us for 1,250 of them
// with a look at every slot first, 25.9 so, 13.7 and 10.3 for 290.)  mine: kEmptySlot for nothing to insert.  Afterwards h[u] is the slot
// of mine[u]'s key; returns the number of slots claimed.
template <int N>
__device__ __forceinline__ uint32_t bucket_insert_many(unsigned long long* table, uint32_t slots, uint32_t (&h)[N], const unsigned long long (&mine)[N]) {
  uint32_t claimed = 0;
  unsigned long long cur[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    cur[u] = mine[u];
    if (mine[u] != kEmptySlot) cur[u] = atomicCAS(&table[h[u]], (unsigned long long)kEmptySlot, mine[u]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t key = (uint32_t)(mine[u] >> 32);
    while (cur[u] != kEmptySlot && (uint32_t)(cur[u] >> 32) != key) {
      h[u] = (h[u] + (key * 0x85EBCA6Bu >> 16 | 1u)) & (slots - 1);
      cur[u] = atomicCAS(&table[h[u]], (unsigned long long)kEmptySlot, mine[u]);
    }
    claimed += cur[u] == kEmptySlot ? 1u : 0u;
    if (mine[u] < cur[u] && cur[u] != kEmptySlot) atomicMin(&table[h[u]], mine[u]);
  }
  uint32_t none = 0;
#pragma unroll
  for (int u = 0; u < N; ++u) none += mine[u] == kEmptySlot ? 1u : 0u;
  return claimed - none;
}
// Is the vertex of list position i a seed that stands in S^l twice?  (`at`: its first position, known by now.)
__device__ __forceinline__ bool seed_twice(uint32_t i, uint32_t at, uint32_t nd) { return i < nd && at != i; }
__device__ __forceinline__ uint32_t bucket_find(const unsigned long long* table, uint32_t slots, uint32_t h, uint32_t key) {
  for (;;) {  // (every key looked up was inserted; an empty slot ends the search regardless)
    const unsigned long long cur = table[h];
    if ((uint32_t)(cur >> 32) == key || cur == kEmptySlot) return (uint32_t)cur;
    h = (h + 1) & (slots - 1);
  }
}

// One thread per block, when the block's part of the first positions is done: adds the distinct keys and counts the block;
// the last one stores the number of new vertices and sends the control block to the host.
__device__ __forceinline__ void bucket_done(Ctl* ctl, const BucketState& st, int64_t n_dst, const Publish& pub) {
  if (st.dup | st.full) {  // (rare: the fence orders the flag before the count)
    if (st.dup) atomicOr(&ctl->err_dup, 1);
    if (st.full) atomicOr(&ctl->uniq_overflow, 1);
    __threadfence();
  }
  uint32_t distinct;
  if (!tally_last(ctl, st.claimed, &distinct)) return;
  const int64_t n_new = (int64_t)distinct - n_dst;
  ctl->total_new = n_new;
  if (pub.h == nullptr) return;
  Ctl c = *ctl;  // (the fields of earlier kernels; those of this one follow)
  c.total_new = n_new;
  c.err_dup = __hip_atomic_load(&ctl->err_dup, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  c.uniq_overflow = __hip_atomic_load(&ctl->uniq_overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  send_ctl(pub.h, pub.ticket, c);
}

// ---- first positions of a short list -----------------------------------------------------------------------------
// Block b reads the whole list and notes, wave by wave, the positions whose key hashes to bucket b; those keys go into the
// block's table, and the edges among them get what the table then says.  One launch in the place of clearing a table,
// inserting and looking up in HBM, and no key's atomic leaves the block (which counts itself once, in bucket_done).
// Reading everything in every block is what it pays for that: ten instructions per key in every block were 12 of the 20 us that a
// list of 180 thousand entries took.  So it is not the edges' sources that are read but their tags, a byte each (EdgeOut::tag, left by
// the kernel that wrote the edges): 16 to a load, and fewer than three instructions for each.  180 thousand entries 20.5 -> 14.5 us,
// 213 thousand 22.5 -> 15.3, 75 thousand 12.4 -> 10.5.
constexpr int kFilterBlock = 1024;
constexpr uint32_t kFilterSlots = 4096;
constexpr uint32_t kFilterFull = kFilterSlots / 4 * 3 - kFilterBlock;  // distinct keys at which a bucket gives up
constexpr uint32_t kFilterList = 256;                   // positions that a wave can note
constexpr int64_t kFilterPairs = 1024;                  // most entries of a bucket in the mean (64 per wave) ...
// ... and at least four buckets: the first wave looks at up to 512 entries of a list of two parts, and with two buckets noted
// 256 to 270 of them on ordinary lists of 1,500 to 2,048 entries, one more than it can (15 us in the place of 12)
constexpr int kFilterLeastLog2 = 2;
// 256 buckets at most: one per CU, and a tag tells no more apart.  (With tables of 8,192 slots and tags 340 thousand entries took 73 us a
// call in the place of 80 by partition, 495 thousand 84 and 85; but where every list keeps one vertex 300 thousand took 162 and 132,
// 520 thousand 247 and 153, all of them from one vertex 458 and 233: the block that has that vertex goes over the whole list.)
constexpr int64_t kFilterMax = 262144;
// Shorter lists are read by their keys: a lane's 16 tags are of entries in a row, so that few lanes have all there is to note
// (1.3 thousand entries 50 us a call, 40 by keys; 11 thousand 41 and 40; 21 thousand 42 either way, 52 thousand 45 and 47).
constexpr int64_t kFilterTaggedFrom = 16384;
constexpr int64_t kShortMax = 65536;                    // entries up to which the kernel also marks the new vertices (k_uniq_relabel_short)
constexpr int kShortWords = (int)(kShortMax / 64) + 1;
__device__ __forceinline__ uint32_t filter_hash(uint32_t key) { return key * 0x9E3779B9u; }
static_assert(kSourceHash == 0x9E3779B9u, "a source's tag is the highest byte of this hash");

template <bool TAGS>
__global__ __launch_bounds__(kFilterBlock) void k_uniq_filter(const int32_t* __restrict__ dst, int64_t n_dst, const int32_t* __restrict__ col,
                                                              const uint8_t* __restrict__ tags, int64_t m, const Ctl* __restrict__ sizes, int log2_buckets,
                                                              uint32_t* __restrict__ first, unsigned long long* __restrict__ bits /* or null */,
                                                              Ctl* ctl, Publish pub) {
  __shared__ unsigned long long table[kFilterSlots];
  __shared__ uint32_t noted[kFilterBlock / kWave][kFilterList];
  __shared__ BucketState st;
  __shared__ uint32_t s_noted, s_overflow;
  __shared__ unsigned long long word[kShortWords];  // the block's bits
  m = edges_there(sizes, m);
  const uint32_t n = (uint32_t)(n_dst + m);  // (below kFilterMax)
  const uint32_t nd = (uint32_t)n_dst;
  const uint32_t n_words = bits != nullptr ? ((n + 63u) >> 6) - (nd >> 6) : 0u;  // (at most kShortWords)
  for (uint32_t i = threadIdx.x; i < n_words; i += kFilterBlock) word[i] = 0;
  for (uint32_t i = threadIdx.x; i < kFilterSlots; i += kFilterBlock) table[i] = kEmptySlot;
  if (threadIdx.x == 0) { st = BucketState{0u, 0u, 0u}; s_noted = 0; s_overflow = 0; }
  __syncthreads();
  auto key_at = [&](uint32_t i) { return (uint32_t)(i < nd ? dst[i] : col[i - nd]); };
  // The first position of edge position i; the edge whose position it is gets its bit.  (The words are clear when the kernel starts.
  // A block's bits are gathered in LDS: an atomic in L2 for each of them, on a few cache lines, made the kernel 4 to 8 us longer
  // where a pass that collects the words takes 5.)
  auto found = [&](uint32_t i, uint32_t at) {
    first[i - nd] = at;
    if (bits != nullptr && at == i) atomicOr(&word[(i >> 6) - (nd >> 6)], 1ull << (i & 63u));
  };
  const uint32_t width = 1u << (32 - log2_buckets), low = blockIdx.x * width;  // the bucket's hashes: low .. low + width - 1 (log2_buckets >= 1)
  auto slot = [&](uint32_t h) { return (h << log2_buckets) >> 20; };           // the hash bits behind those of the bucket
  static_assert(kFilterSlots == 1u << 12, "slot() takes 12 bits");
  // Each part of the list ([S^l], [col]; 256-byte aligned and padded to that) is read in groups of 16 bytes, a few groups per thread
  // and step, the next step's groups requested before this step's are looked at.  take(flags, entry): those of this lane's keys
  // that are in the bucket, and which entry of the part a flag stands for.
  auto fetch = [&](const void* __restrict__ p, uint32_t groups, uint32_t g0, auto& to) {
#pragma unroll
    for (uint32_t u = 0; u < sizeof(to) / sizeof(to[0]); ++u) {
      const uint32_t g = g0 + u * kFilterBlock + threadIdx.x;
      to[u] = reinterpret_cast<const u32x4*>(p)[g < groups ? g : groups - 1];
    }
  };
  auto by_key = [&](const int32_t* __restrict__ p, uint32_t len, auto&& take) {
    constexpr uint32_t U = 4;
    const uint32_t groups = (len + 3) / 4;
    u32x4 next[U];
    if (groups > 0) fetch(p, groups, 0, next);
    for (uint32_t g0 = 0; g0 < groups; g0 += U * kFilterBlock) {
      uint32_t flags = 0;  // bit 4 u + e
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) flags |= filter_hash(next[u][e]) - low < width ? 1u << (4 * u + e) : 0u;
      if (g0 + U * kFilterBlock < groups) fetch(p, groups, g0 + U * kFilterBlock, next);
      take(flags, [&](uint32_t bit) { return (g0 + (bit >> 2) * kFilterBlock + threadIdx.x) * 4 + (bit & 3u); });
    }
  };
  // (Tags: 16 of them to a load, and a stretch of the part for each wave.  Dealt out load by load, 24 thousand entries left seven waves
  // with twice as many as the others, and their lists ran out of room that much earlier.)
  auto by_tag = [&](uint32_t len, auto&& take) {
    constexpr uint32_t U = 2, kWaves = kFilterBlock / kWave;
    const uint32_t groups = (len + 15) / 16, each = (groups + kWaves - 1) / kWaves;
    const uint32_t lo = each * (uint32_t)uniform_wave_in_block(), hi = lo + each < groups ? lo + each : groups;
    const uint32_t mask = ((0xFF00u >> log2_buckets) & 0xFFu) * 0x01010101u, mine = (blockIdx.x << (8 - log2_buckets)) * 0x01010101u;
    u32x4 next[U];
    auto request = [&](uint32_t g0) {
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t g = g0 + u * kWave + lane_id();
        next[u] = reinterpret_cast<const u32x4*>(tags)[g < hi ? g : hi - 1];
      }
    };
    if (lo < hi) request(lo);
    for (uint32_t g0 = lo; g0 < hi; g0 += U * kWave) {
      uint32_t flags = 0;  // bit 8 b + 7 - q: byte b of word q
#pragma unroll
      for (uint32_t q = 0; q < 4 * U; ++q) {
        const uint32_t x = (next[q / 4][q % 4] ^ mine) & mask;  // a zero byte: one of the bucket's
        const uint32_t f = ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu) >> q;
        flags |= g0 + (q / 4) * kWave + lane_id() < hi ? f : 0u;
      }
      if (g0 + U * kWave < hi) request(g0 + U * kWave);
      take(flags, [&](uint32_t bit) {
        const uint32_t q = 7u - (bit & 7u);
        return (g0 + (q >> 2) * kWave + lane_id()) * 16 + (q & 3u) * 4 + (bit >> 3);
      });
    }
  };
  uint32_t* list = noted[uniform_wave_in_block()];
  uint32_t count = 0;  // (the same in every lane)
  auto note = [&](uint32_t len, uint32_t at0) {
    return [&, len, at0](uint32_t flags, auto&& entry) {
      for (;;) {  // a few of the wave's keys: every round notes one of each lane's
        if (ballot64(flags != 0) == 0) break;
        const uint32_t i = entry(flags != 0 ? (uint32_t)__builtin_ctz(flags) : 0u);
        const bool in = flags != 0 && i < len;
        const uint64_t mask = ballot64(in);
        const uint32_t to = count + lanes_below(mask);
        if (in && to < kFilterList) list[to] = at0 + i;
        count += (uint32_t)__popcll(mask);
        flags &= flags - 1;
      }
    };
  };
  by_key(dst, nd, note(nd, 0u));
  if constexpr (TAGS) by_tag(n - nd, note(n - nd, nd));
  else by_key(col, n - nd, note(n - nd, nd));
  if (lane_id() == 0) {
    atomicAdd(&s_noted, count);
    if (count > kFilterList) s_overflow = 1;
  }
  __syncthreads();
  if (s_overflow == 0) {  // every wave goes on with its own list
    constexpr int V = kFilterList / kWave;
    unsigned long long pair[V];
    uint32_t h[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const uint32_t q = (uint32_t)(v * kWave + lane_id());
      const bool in = q < count;
      const uint32_t i = in ? list[q] : 0u;
      const uint32_t key = in ? key_at(i) : 0u;
      h[v] = slot(filter_hash(key));
      pair[v] = in ? ((unsigned long long)key << 32) | i : kEmptySlot;
    }
    const bool fits = s_noted <= kFilterSlots / 4 * 3;  // (the others have their room counted, and seeds that stand there twice reported)
    if (fits) {
      const uint32_t claimed = wave_sum_u32(bucket_insert_many<V>(table, kFilterSlots, h, pair));
      if (lane_id() == 0) atomicAdd(&st.claimed, claimed);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (pair[v] != kEmptySlot && lds_read(&st.full) == 0) h[v] = bucket_insert(table, kFilterSlots, kFilterFull, h[v], pair[v], nd, &st);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (pair[v] == kEmptySlot) continue;
      const uint32_t i = (uint32_t)pair[v], at = (uint32_t)table[h[v]];
      if (i >= nd) found(i, at);
      else if (fits && seed_twice(i, at, nd)) st.dup = 1;
    }
  } else {
    // vertices that very many lists keep: the whole list is read again, twice.  Where most of it is the block's, by its keys, which go
    // from the registers straight to the table; else by its tags, and a key is requested for each that is found.  (235 thousand entries,
    // a fifth of the edges from one vertex: 150 us by keys, 133 by tags, three tenths 179 and 173, four tenths 205 and 213, all 278 and 386;
    // 17 thousand and three tenths 24 and 28.  Where edges lead to vertices by a power law, 80 and 130 thousand entries: 39 and 32, 51 and 40.)
    constexpr uint32_t U = 4;
    auto each = [&](const int32_t* __restrict__ p, uint32_t len, auto&& take) {
      const uint32_t groups = (len + 3) / 4;
      for (uint32_t g0 = 0; g0 < groups; g0 += U * kFilterBlock) {
        u32x4 key[U];
        fetch(p, groups, g0, key);
        uint32_t flags = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) flags |= filter_hash(key[u][e]) - low < width ? 1u << (4 * u + e) : 0u;
        for (; flags != 0; flags &= flags - 1) {
          const uint32_t bit = (uint32_t)__builtin_ctz(flags);
          uint32_t k = 0;
#pragma unroll
          for (uint32_t b = 0; b < 4 * U; ++b) k = bit == b ? key[b / 4][b % 4] : k;
          const uint32_t i = (g0 + (bit >> 2) * kFilterBlock + threadIdx.x) * 4 + (bit & 3u);
          if (i < len) take(i, k);
        }
      }
    };
    auto insert = [&](uint32_t i, uint32_t key) {
      if (lds_read(&st.full) == 0)
        bucket_insert(table, kFilterSlots, kFilterFull, slot(filter_hash(key)), ((unsigned long long)key << 32) | i, nd, &st);
    };
    auto look_up = [&](uint32_t i, uint32_t key) { found(i, bucket_find(table, kFilterSlots, slot(filter_hash(key)), key)); };
    auto tagged = [&](auto&& what) {
      return [&](uint32_t flags, auto&& entry) {
        for (; flags != 0; flags &= flags - 1) {
          const uint32_t i = entry((uint32_t)__builtin_ctz(flags));
          if (i < n - nd) what(nd + i, (uint32_t)col[i]);
        }
      };
    };
    const bool use_tags = TAGS && s_noted <= n / 4;
    each(dst, nd, insert);
    if (use_tags) by_tag(n - nd, tagged(insert));
    else each(col, n - nd, [&](uint32_t i, uint32_t key) { insert(nd + i, key); });
    __syncthreads();
    if (st.full == 0) {
      if (use_tags) by_tag(n - nd, tagged(look_up));
      else each(col, n - nd, [&](uint32_t i, uint32_t key) { look_up(nd + i, key); });
    }
  }
  __syncthreads();
  if (n_words != 0) {
    for (uint32_t i = threadIdx.x - kWave; threadIdx.x >= kWave && i < n_words; i += kFilterBlock - kWave)
      if (word[i] != 0) atomicOr(&bits[i], word[i]);
  }
  if (threadIdx.x == 0) bucket_done(ctl, st, n_dst, pub);
}

// ---- ranks and local ids -----------------------------------------------------------------------------------------
// The new-flags are a bit per position of [S^l ; col]: bit i is set when edge i - n_dst is the first occurrence of its
// vertex.  The rank of such a position among them is kept in three parts: the bits below it in its word, the bits of the
// words in front of it in its block's stretch of positions (one record with the word: looking ranks up is bound by the number
// of scattered requests), and those of the stretches in front (block_prefix).
struct RankView {
  const RankWord* word;   // of the positions from the multiple of 64 at or below n_dst on
  const uint32_t* block_prefix;  // ... or, when n_totals is not 0, the stretches' own totals, which the reader scans
  uint32_t n_blocks;  // when not 0: the stretches are those of the partition's blocks (part_stretch_len of the whole list)
  uint32_t n_totals;
};
constexpr int64_t kCollectStretch = 8192;

// ---- first positions by partition ------------------------------------------------------------------------------
// For long lists the table in HBM costs two dependent random accesses per entry (insert, then look-up), each an
// atomic or a miss of every cache.  The partitioned form touches HBM in streams only: the (key, position) pairs are
// distributed over buckets by the high bits of the key's hash (count, scan, scatter: the classic three-step
// partition, with a counter matrix [bucket][block] so that no atomic leaves a block and every pair has its place
// before it is moved), and a bucket, about kPartPairs pairs, is deduplicated by one block in a table in LDS.
// The scatter orders a tile of the list by bucket and notes, in that order, where every entry went and which entry of the
// tile it is; the first positions are left in the buckets' order, written in streams, and the collecting kernel reads
// them back run by run and puts the tile into list order in LDS.  4-byte stores from the buckets to the places in the list
// cost a partial line each (5.8 M of them 72 us, however they are spread over the XCDs).  For the 5.8 M entries of a last
// papers100M-shaped layer: scatter 38 us (2.8 TB/s), first positions 39 to 41 (84 with the stores to random places), collecting
// with the ranks 24 (20 for two kernels that only made flags and ranks), relabelling 23 (75 MB, 3.3 TB/s).
constexpr int kPartBlock = 1024;        // threads of a counting / scattering block
constexpr int kPartMaxBlocks = 512;     // blocks of those two kernels (two per compute unit)
constexpr int kPartPairs = 4096;        // mean pairs of a bucket
constexpr uint32_t kPartMaxBuckets = 8192;  // counters of a block in LDS: 32 KB
constexpr int kFirstBlock = 1024;       // threads of a bucket's block
constexpr uint32_t kPartSlots = 8192;   // slots of a bucket's table in LDS (64 KB): at most half full when every pair of a
                                        // mean bucket is distinct, a quarter or less with the usual share of repeats
constexpr uint32_t kPartFull = kPartSlots / 4 * 3;  // distinct keys at which a bucket gives up
static_assert(kPartFull + 1 + kFirstBlock < kPartSlots, "a probe must always reach an empty slot");

__device__ __forceinline__ uint32_t hash_of_key(uint32_t key) { return (uint32_t)(((uint64_t)key * 0x9E3779B97F4A7C15ull) >> 32); }
__device__ __forceinline__ uint32_t bucket_of_hash(uint32_t h, uint32_t n_buckets) { return (uint32_t)(((uint64_t)h * n_buckets) >> 32); }
// a bucket's hashes share their high bits: the table slot comes from the low ones, stirred
__device__ __forceinline__ uint32_t table_slot_of_hash(uint32_t h) {
  uint32_t x = h ^ (h >> 16);
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  return x & (kPartSlots - 1);
}

// The stretch of [S^l ; col] that block `block` of `n_blocks` counts and scatters.
__device__ __forceinline__ int64_t part_stretch_len(int64_t n_all, uint32_t n_blocks) {
  const int64_t stretch = (n_all + n_blocks - 1) / n_blocks;
  return (stretch + kPartBlock - 1) / kPartBlock * kPartBlock;
}
__device__ __forceinline__ void part_stretch(int64_t n_all, uint32_t n_blocks, uint32_t block, int64_t* lo, int64_t* hi) {
  const int64_t stretch = part_stretch_len(n_all, n_blocks);
  *lo = (int64_t)block * stretch;
  *hi = *lo + stretch < n_all ? *lo + stretch : n_all;
  if (*lo > n_all) *lo = n_all;
}
// A bucket's pairs are laid out by column, one column per block.  Consecutive blocks run on different XCDs (round
// robin over 8), so the blocks of one XCD take neighbouring columns: a cache line of pairs is then put together in
// one XCD's L2.  (gridDim.x is a multiple of 8.)
__device__ __forceinline__ uint32_t part_column() { return (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3); }

// counts[b * gridDim.x + column] = pairs of this block's stretch that fall into bucket b
__global__ __launch_bounds__(kPartBlock) void k_part_count(const int32_t* __restrict__ dst, int64_t n_dst, const int32_t* __restrict__ col,
                                                           int64_t m, const Ctl* __restrict__ sizes, uint32_t n_buckets,
                                                           uint32_t* __restrict__ counts) {
  extern __shared__ uint32_t tally[];  // [n_buckets]
  m = edges_there(sizes, m);
  int64_t lo, hi;
  part_stretch(n_dst + m, gridDim.x, blockIdx.x, &lo, &hi);
  for (uint32_t b = threadIdx.x; b < n_buckets; b += kPartBlock) tally[b] = 0u;
  __syncthreads();
  constexpr int U = 4;  // independent loads in flight per thread
  for (int64_t base = lo + threadIdx.x; base < hi; base += (int64_t)U * kPartBlock) {
    uint32_t key[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = base + (int64_t)u * kPartBlock;
      key[u] = i < hi ? (uint32_t)(i < n_dst ? dst[i] : col[i - n_dst]) : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + (int64_t)u * kPartBlock < hi) atomicAdd(&tally[bucket_of_hash(hash_of_key(key[u]), n_buckets)], 1u);
  }
  __syncthreads();
  const uint32_t column = part_column();
  for (uint32_t b = threadIdx.x; b < n_buckets; b += kPartBlock) counts[(size_t)b * gridDim.x + column] = tally[b];
}

// The same stretch again: its pairs go to pairs[], bucket b's from place[b * gridDim.x + column] on (place = exclusive
// scan of counts).  A tile of kTilePairs pairs is first ordered by bucket in LDS, so that the pairs of a tile that share a
// bucket leave as one contiguous run written by neighbouring lanes, not as single 8-byte stores.  In the tile's new order,
// every pair's index in pairs[] ("went") and its number in the tile ("which") are kept for k_uniq_collect.
constexpr int kTilePairs = 8 * kPartBlock;
// Where those two lie.  A tile without edges needs neither.  The indices of list position i go to the place in col_local
// that k_uniq_collect fills from them, those of the one tile that begins below n_dst to `head` where they have none there.
struct TileNotes {
  uint32_t* first;  // [m] col_local
  uint32_t* head;   // [kTilePairs]
  uint16_t* which;  // [kTilePairs + m]
  __device__ __forceinline__ uint32_t* went(int64_t i, int64_t n_dst) const { return i >= n_dst ? first + (i - n_dst) : head + (i + kTilePairs - n_dst); }
  __device__ __forceinline__ uint16_t* which_of(int64_t i, int64_t n_dst) const { return which + (i + kTilePairs - n_dst); }
};
// PER: buckets that a thread looks after.  (64 registers, so that two blocks fit a CU.)
template <int PER>
__global__ __launch_bounds__(kPartBlock, PER <= 2 ? 8 : 4) void k_part_scatter(const int32_t* __restrict__ dst, int64_t n_dst, const int32_t* __restrict__ col,
                                                             int64_t m, const Ctl* __restrict__ sizes, uint32_t n_buckets,
                                                             TiledScan<uint32_t> place, unsigned long long* __restrict__ pairs, TileNotes notes) {
  __shared__ unsigned long long staged[kTilePairs];  // the tile's pairs, by bucket: key, bucket (16 bits), number in the tile (16 bits)
  extern __shared__ uint32_t off[];                  // [n_buckets] the tile's tallies, then run starts in the tile
  uint32_t* delta = off + n_buckets;                 // [n_buckets] run start in pairs[] minus run start in the tile
  __shared__ uint32_t wave_total[kPartBlock / kWave];
  m = edges_there(sizes, m);
  int64_t lo, hi;
  part_stretch(n_dst + m, gridDim.x, blockIdx.x, &lo, &hi);
  const uint32_t column = part_column();
  const int lane = lane_id(), wave = wave_in_block();
  constexpr int U = kTilePairs / kPartBlock;
  // A tile's keys are requested before anything else, the next tile's when this one's stand in LDS.
  uint32_t key[U];
  auto fetch = [&](int64_t tile) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = tile + u * kPartBlock + threadIdx.x;
      key[u] = i < hi ? (uint32_t)(i < n_dst ? dst[i] : col[i - n_dst]) : 0u;
    }
  };
  fetch(lo);
  uint32_t cursor[PER];  // next free place of this thread's buckets in this column
#pragma unroll
  for (uint32_t q = 0; q < PER; ++q) {
    const uint32_t b = threadIdx.x * PER + q;
    cursor[q] = b < n_buckets ? place.at((int64_t)b * gridDim.x + column) : 0u;
    if (b < n_buckets) off[b] = 0u;
  }
  __syncthreads();
  for (int64_t tile = lo; tile < hi; tile += kTilePairs) {
    const uint32_t tile_n = (uint32_t)(hi - tile < kTilePairs ? hi - tile : kTilePairs);
    const bool has_edges = tile + tile_n > n_dst;
    uint32_t place_in[U];  // bucket << 16 | rank in the tile's bucket
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t bucket = bucket_of_hash(hash_of_key(key[u]), n_buckets);
      place_in[u] = bucket << 16;
      if ((uint32_t)(u * kPartBlock) + threadIdx.x < tile_n) place_in[u] |= atomicAdd(&off[bucket], 1u);
    }
    __syncthreads();
    {  // tallies -> run starts (exclusive scan over the buckets)
      uint32_t c[PER], sum = 0;
#pragma unroll
      for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t b = threadIdx.x * PER + q;
        c[q] = b < n_buckets ? off[b] : 0u;
        sum += c[q];
      }
      const uint32_t incl = wave_incl_scan(sum);
      if (lane == kWave - 1) wave_total[wave] = incl;
      __syncthreads();
      uint32_t run = incl - sum;
      for (int w = 0; w < wave; ++w) run += wave_total[w];
#pragma unroll
      for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t b = threadIdx.x * PER + q;
        if (b < n_buckets) {
          off[b] = run;
          delta[b] = cursor[q] - run;
          cursor[q] += c[q];
        }
        run += c[q];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = (uint32_t)(u * kPartBlock) + threadIdx.x;
      if (j < tile_n) 
        staged[off[place_in[u] >> 16] + (place_in[u] & 0xFFFFu)] = ((unsigned long long)key[u] << 32) | (place_in[u] & 0xFFFF0000u) | j;
    }
    if (tile + kTilePairs < hi) fetch(tile + kTilePairs);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = (uint32_t)(u * kPartBlock) + threadIdx.x;
      if (j < tile_n) {
        const unsigned long long pr = staged[j];
        const uint32_t to = delta[(uint32_t)pr >> 16] + j;
        pairs[to] = (pr >> 32 << 32) | ((uint32_t)tile + ((uint32_t)pr & 0xFFFFu));  // (positions stay below 2^32)
        if (has_edges) {
          *notes.went(tile + j, n_dst) = to;
          *notes.which_of(tile + j, n_dst) = (uint16_t)pr;
        }
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
      const uint32_t b = threadIdx.x * PER + q;
      if (b < n_buckets) off[b] = 0u;
    }
    __syncthreads();
  }
}

// One bucket per block: first positions of the bucket's keys through a table in LDS; by_place[p << shift] = that of pair p.
// (With shift = 1 by_place is the pairs' own memory: pair p's result takes the place of its position, and nobody else reads
// or writes pair p.  64 registers and 64 KB of LDS: two blocks per CU.)
__global__ __launch_bounds__(kFirstBlock, 8) void k_part_first(const unsigned long long* pairs, TiledScan<uint32_t> place,
                                                               uint32_t G, int64_t n_dst, int64_t n_all, uint32_t* by_place, int shift,
                                                               Ctl* ctl, Publish pub) {
  __shared__ unsigned long long table[kPartSlots];
  __shared__ BucketState st;
  uint32_t lo = place.at((int64_t)blockIdx.x * G), hi = place.at((int64_t)(blockIdx.x + 1) * G);
  if ((int64_t)hi > n_all) hi = (uint32_t)n_all;  // (holds by construction; keeps every access inside the arrays regardless)
  if (lo > hi) lo = hi;
  const uint32_t nd = (uint32_t)n_dst;
  constexpr int U = 5;  // pairs per thread and round, loaded together (a bucket of the mean size and a quarter more in one round)
  static_assert((uint32_t)(U * kFirstBlock) <= kPartFull, "one round cannot fill the table");
  unsigned long long mine[U];
  auto fetch = [&](uint32_t base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = base + u * kFirstBlock + threadIdx.x;
      mine[u] = i < hi ? pairs[i] : kEmptySlot;
    }
  };
  fetch(lo);  // under way while the table is cleared
  for (uint32_t i = threadIdx.x; i < kPartSlots; i += kFirstBlock) table[i] = kEmptySlot;
  if (threadIdx.x == 0) st = BucketState{0u, 0u, 0u};
  __syncthreads();
  uint32_t h[U];
  if (hi - lo <= (uint32_t)(U * kFirstBlock)) {  // the usual bucket
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = table_slot_of_hash(hash_of_key((uint32_t)(mine[u] >> 32)));
    const uint32_t claimed = wave_sum_u32(bucket_insert_many<U>(table, kPartSlots, h, mine));
    if (lane_id() == 0) atomicAdd(&st.claimed, claimed);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = lo + u * kFirstBlock + threadIdx.x;
      if (i >= hi) continue;
      const uint32_t at = (uint32_t)table[h[u]];
      by_place[(size_t)i << shift] = at;
      if (seed_twice((uint32_t)mine[u], at, nd)) st.dup = 1;
    }
    __syncthreads();
  } else {
    for (uint32_t base = lo; base < hi; base += U * kFirstBlock) {
      if (base != lo) fetch(base);
      if (lds_read(&st.full) != 0) break;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (mine[u] == kEmptySlot || lds_read(&st.full) != 0) continue;
        bucket_insert(table, kPartSlots, kPartFull, table_slot_of_hash(hash_of_key((uint32_t)(mine[u] >> 32))), mine[u], nd, &st);
      }
    }
    __syncthreads();
    if (st.full == 0) {
      // (U pairs at a time: with one at a time every load waited for the store before it.  1.7 M pairs of one key 1.61 ms, 1.03 so.)
      for (uint32_t base = lo; base < hi; base += U * kFirstBlock) {
        fetch(base);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (mine[u] == kEmptySlot) continue;
          const uint32_t key = (uint32_t)(mine[u] >> 32);
          by_place[(size_t)(base + u * kFirstBlock + threadIdx.x) << shift] = bucket_find(table, kPartSlots, table_slot_of_hash(hash_of_key(key)), key);
        }
      }
    }
  }
  if (threadIdx.x == 0) bucket_done(ctl, st, n_dst, pub);
}

// List order again, the new-flags and their ranks (see RankView).  GATHER: the first positions lie in by_place and go to
// first[e] (edge order), tile by tile: neighbouring lanes read the runs that the scatter wrote, LDS turns the tile into
// list order.  Else first[e] is there already.  A block takes the stretch that the block of the same number scattered
// (the same XCD, as blocks are dealt to the XCDs in order, and so the columns of by_place that its L2 has seen).
template <bool GATHER>
__global__ __launch_bounds__(kPartBlock, 8) void k_uniq_collect(uint32_t* first, const uint32_t* __restrict__ by_place, int shift,
                                                             TileNotes notes, int64_t m,
                                                             const Ctl* __restrict__ sizes, int64_t n_dst, RankWord* __restrict__ words,
                                                             uint32_t* __restrict__ block_total,
                                                             uint32_t* __restrict__ block_prefix, Ctl* ctl, Publish pub) {
  constexpr int U = kTilePairs / kPartBlock, kWaves = kPartBlock / kWave, kWords = kTilePairs / 64;
  static_assert(kWords == 2 * kWave, "two words per lane of the scanning wave");
  static_assert(kCollectStretch == kTilePairs, "one tile per block when the stretches are not the partition's");
  __shared__ uint32_t in_order[GATHER ? kTilePairs : 1];
  __shared__ uint32_t count[2][kWords];
  __shared__ uint32_t s_last;
  m = edges_there(sizes, m);
  const int64_t n_all = n_dst + m;
  int64_t lo, hi;
  if constexpr (GATHER) {
    part_stretch(n_all, gridDim.x, blockIdx.x, &lo, &hi);
  } else {
    lo = (int64_t)blockIdx.x * kCollectStretch;
    hi = lo + kCollectStretch < n_all ? lo + kCollectStretch : n_all;
  }
  const int lane = lane_id(), wave = wave_in_block();
  const int64_t w0 = n_dst >> 6;  // (the words in front have no bits and are not kept)
  uint32_t run = 0;  // (kept by the first wave)
  int flip = 0;
  for (int64_t tile = lo; tile < hi; tile += kTilePairs, flip ^= 1) {
    const uint32_t tile_n = (uint32_t)(hi - tile < kTilePairs ? hi - tile : kTilePairs);
    uint32_t f[U];
    if (tile + tile_n <= n_dst) continue;  // (no edge in it; the same for the whole block)
    if constexpr (GATHER) {
      uint32_t at[U], to[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t j = (uint32_t)(u * kPartBlock) + threadIdx.x;
        const int64_t i = tile + (j < tile_n ? j : 0u);
        at[u] = *notes.went(i, n_dst);
        to[u] = *notes.which_of(i, n_dst);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) f[u] = by_place[(size_t)at[u] << shift];
#pragma unroll
      for (int u = 0; u < U; ++u) in_order[to[u]] = f[u];  // (a thread behind the tile's end repeats entry 0)
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = (uint32_t)(u * kPartBlock) + threadIdx.x;
      const int64_t i = tile + j;
      const bool edge = j < tile_n && i >= n_dst;
      if constexpr (GATHER) {
        f[u] = in_order[j];
        if (edge) first[i - n_dst] = f[u];
      } else {
        f[u] = 0;
        if (edge) f[u] = first[i - n_dst];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t j = (uint32_t)(u * kPartBlock) + threadIdx.x;
      const int64_t i = tile + j;
      const uint64_t b = ballot64(j < tile_n && i >= n_dst && (int64_t)f[u] == i);
      if (lane == 0) {
        if (j < tile_n && (i >> 6) >= w0) words[(i >> 6) - w0].bits = b;
        count[flip][u * kWaves + wave] = (uint32_t)__popcll(b);
      }
    }
    __syncthreads();  // (two buffers of counts: the next tile's go to the other one while the first wave scans these)
    if (wave == 0) {
      const uint32_t a = count[flip][2 * lane], b = count[flip][2 * lane + 1];
      const uint32_t incl = wave_incl_scan(a + b);
      const uint32_t j = (uint32_t)lane * 128;
      const int64_t w = ((tile + j) >> 6) - w0;
      if (j < tile_n && w >= 0) words[w].before = run + incl - a - b;
      if (j + 64 < tile_n && w + 1 >= 0) words[w + 1].before = run + incl - b;
      run += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    }
  }
  if (block_prefix == nullptr) {  // the relabelling scans the totals
    if (threadIdx.x == 0) block_total[blockIdx.x] = run;
    return;
  }
  if (threadIdx.x == 0) {
    // the exchange has been performed when its result is here; the block counts itself behind it
    const uint32_t old = atomicExch(&block_total[blockIdx.x], run);
    asm volatile("" : : "v"(old) : "memory");
    uint32_t unused;
    s_last = tally_last(ctl, 0u, &unused) ? 1u : 0u;
  }
  __syncthreads();
  if (s_last == 0) return;
  __shared__ uint32_t wave_total[kWaves];
  uint32_t carry = 0;
  for (uint32_t base = 0; base < gridDim.x; base += kPartBlock) {
    const uint32_t b = base + threadIdx.x;
    const uint32_t v = b < gridDim.x ? __hip_atomic_load(&block_total[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    uint32_t incl = wave_incl_scan(v);
    if (lane == kWave - 1) wave_total[wave] = incl;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) incl += wave_total[w];
      all += wave_total[w];
    }
    if (b < gridDim.x) block_prefix[b] = carry + incl - v;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0 && pub.h != nullptr) {
    ctl->total_new = carry;
    Ctl c = *ctl;
    c.total_new = carry;
    send_ctl(pub.h, pub.ticket, c);
  }
}

// col_local and the tail of src_ids; the threads of the first n_dst positions also copy S^l to the front of src_ids.
// col_local holds the first positions and gets the local ids in their place.
// (sizes, optional: says the exact number of edges, on the device; m is then the capacity of col.  The kernel may be
// launched before the host has seen the dedup's error and overflow flags, on first positions that a failed dedup left
// partly unwritten: positions outside [0, n_dst + m) are skipped, so that every access stays inside the arrays whatever
// they are; the caller discards the result in that case.)
constexpr int kRelabelUnroll = 4;  // edges per thread in flight
__global__ __launch_bounds__(kBlock) void k_uniq_relabel(const int32_t* __restrict__ dst, const int32_t* __restrict__ col, int64_t m,
                                                         const Ctl* __restrict__ sizes, int64_t n_dst, RankView rank,
                                                         int32_t* __restrict__ src, int32_t* __restrict__ col_local) {
  m = edges_there(sizes, m);
  // the stretch of a word by multiplication: exact while (positions / 1024) * (stretch / 1024) stays below 2^32
  const int64_t stretch = rank.n_blocks ? part_stretch_len(n_dst + m, rank.n_blocks) : kCollectStretch;
  const uint32_t d = (uint32_t)(stretch >> 10), magic = d <= 1 ? 0u : 0xFFFFFFFFu / d + 1u;
  __shared__ uint32_t prefix[kPartMaxBlocks];
  if (rank.n_totals) {
    __shared__ uint32_t wave_total[kWavesPerBlock];
    static_assert(kPartMaxBlocks == 2 * kBlock, "two totals per thread");
    const uint32_t b = 2 * threadIdx.x;
    const uint32_t t0 = b < rank.n_totals ? rank.block_prefix[b] : 0u, t1 = b + 1 < rank.n_totals ? rank.block_prefix[b + 1] : 0u;
    uint32_t upto = wave_incl_scan(t0 + t1);
    if (lane_id() == kWave - 1) wave_total[wave_in_block()] = upto;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kWavesPerBlock - 1; ++q) upto += q < wave_in_block() ? wave_total[q] : 0u;
    prefix[b] = upto - t0 - t1;
    prefix[b + 1] = upto - t1;
    __syncthreads();
  }
  const int64_t e0 = (int64_t)blockIdx.x * (kBlock * kRelabelUnroll) + threadIdx.x;
#pragma unroll
  for (int u = 0; u < kRelabelUnroll; ++u) {
    const int64_t e = e0 + u * kBlock;
    if (e < n_dst) src[e] = dst[e];
  }
  const uint32_t w0 = (uint32_t)(n_dst >> 6);
  uint32_t f[kRelabelUnroll];
#pragma unroll
  for (int u = 0; u < kRelabelUnroll; ++u) {
    const int64_t e = e0 + u * kBlock;
    f[u] = e < m ? (uint32_t)col_local[e] : 0xFFFFFFFFu;
  }
  RankWord w[kRelabelUnroll];
#pragma unroll
  for (int u = 0; u < kRelabelUnroll; ++u) {
    w[u] = RankWord{0, 0, 0};
    if ((int64_t)f[u] >= n_dst && (int64_t)f[u] < n_dst + m) w[u] = rank.word[(f[u] >> 6) - w0];
  }
#pragma unroll
  for (int u = 0; u < kRelabelUnroll; ++u) {
    const int64_t e = e0 + u * kBlock;
    if ((int64_t)f[u] >= n_dst + m) continue;
    int64_t local = f[u];
    if (local >= n_dst) {
      const uint32_t q = f[u] >> 10, block = d <= 1 ? q : __umulhi(q, magic);
      const uint32_t in_front = rank.n_totals ? prefix[block] : rank.block_prefix[block];
      local = n_dst + in_front + w[u].before + __popcll(w[u].bits & ((1ull << (f[u] & 63)) - 1ull));
      if ((int64_t)f[u] == n_dst + e) src[local] = col[e];
    }
    col_local[e] = (int32_t)local;
  }
}

// The same for the shortest lists, straight from the bits that k_uniq_filter set: every block counts them all, 64 to a word, and keeps
// words and ranks in LDS.  A launch less than with k_uniq_collect in between: calls over 300 to 60 thousand entries 1 to 4 us
// shorter (44.9 and 45.7 us, 51.8 and 55.2), below 300 none.
constexpr int kShortBlock = 1024, kShortEach = 4;
__global__ __launch_bounds__(kShortBlock) void k_uniq_relabel_short(const int32_t* __restrict__ dst, const int32_t* __restrict__ col, int64_t m,
                                                                    const Ctl* __restrict__ sizes, int64_t n_dst,
                                                                    const unsigned long long* __restrict__ bits, int32_t* __restrict__ src,
                                                                    int32_t* __restrict__ col_local) {
  constexpr int kEach = (kShortWords + kShortBlock - 1) / kShortBlock;  // words per thread
  __shared__ unsigned long long word[kEach * kShortBlock];
  __shared__ uint32_t before[kEach * kShortBlock];
  __shared__ uint32_t wave_total[kShortBlock / kWave];
  const int64_t e0 = (int64_t)blockIdx.x * (kShortBlock * kShortEach) + threadIdx.x;
  m = edges_there(sizes, m);
  uint32_t f[kShortEach];
#pragma unroll
  for (int u = 0; u < kShortEach; ++u) {
    const int64_t e = e0 + u * kShortBlock;
    f[u] = e < m ? (uint32_t)col_local[e] : 0xFFFFFFFFu;
    if (e < n_dst) src[e] = dst[e];
  }
  const uint32_t w0 = (uint32_t)(n_dst >> 6), n_words = (uint32_t)((n_dst + m + 63) >> 6) - w0;  // (at most kShortWords)
  uint32_t c[kEach], sum = 0;
#pragma unroll
  for (int q = 0; q < kEach; ++q) {  // words in a row per thread
    const uint32_t w = threadIdx.x * kEach + q;
    const unsigned long long b = w < n_words ? bits[w] : 0ull;
    word[w] = b;
    c[q] = (uint32_t)__popcll(b);
    sum += c[q];
  }
  const uint32_t incl = wave_incl_scan(sum);
  if (lane_id() == kWave - 1) wave_total[wave_in_block()] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int q = 0; q < wave_in_block(); ++q) run += wave_total[q];
#pragma unroll
  for (int q = 0; q < kEach; ++q) {
    before[threadIdx.x * kEach + q] = run;
    run += c[q];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kShortEach; ++u) {
    const int64_t e = e0 + u * kShortBlock;
    if ((int64_t)f[u] >= n_dst + m) continue;  // (also: first positions that a failed dedup left unwritten)
    int64_t local = f[u];
    if (local >= n_dst) {
      const uint32_t w = (f[u] >> 6) - w0;
      local = n_dst + before[w] + __popcll(word[w] & ((1ull << (f[u] & 63)) - 1ull));
      if ((int64_t)f[u] == n_dst + e && local < n_dst + m) src[local] = col[e];
    }
    col_local[e] = (int32_t)local;
  }
}

// ---- the shortest lists in one block ------------------------------------------------------------------------------------
// Everything from the first positions to the local ids, U entries of the list per thread, in one launch in the place of k_uniq_filter
// and k_uniq_relabel_short: nothing goes through memory in between, no other block is counted, and the table has room for all
// entries.  Short of that it waits, for memory twice and for LDS a dozen times; from 4,096 entries on the insertions, all on one CU, are
// what counts (1.3 thousand entries 0.9 us of 4.5, 3.9 thousand 2.2 of 6.0; with room for ten entries per thread, 10 thousand 9.7 of 16).
// Calls over 1.3 and 3.9 thousand entries 5 us shorter than with the two kernels (35.0 -> 30.2, 35.9 -> 30.7), over 6.5 thousand 1,
// over 7.8 thousand none: there it ends.
constexpr int kSmallBlock = 1024;
constexpr int kSmallEach = 8;
constexpr int64_t kSmallMax = 7936;
static_assert(kSmallMax <= (int64_t)kSmallBlock * kSmallEach, "a thread has room for its entries");
template <int U>
__global__ __launch_bounds__(kSmallBlock) void k_uniq_small(const int32_t* __restrict__ dst, int64_t n_dst, const int32_t* __restrict__ col, int64_t m,
                                                            const Ctl* __restrict__ sizes, int32_t* __restrict__ src, int32_t* __restrict__ col_local,
                                                            Ctl* ctl, Publish pub) {
  constexpr uint32_t kSlots = 16384;  // (128 KB of LDS; nobody else wants them)
  static_assert((uint32_t)(U * kSmallBlock) <= kSlots / 4 * 3, "a probe must always reach an empty slot");
  constexpr int kWaves = kSmallBlock / kWave, kWords = U * kWaves;
  __shared__ unsigned long long table[kSlots];
  __shared__ unsigned long long bits[kWords];  // new vertices among 64 entries
  __shared__ uint32_t before[kWords];          // ... and in the words in front
  __shared__ BucketState st;
  const uint32_t nd = (uint32_t)n_dst;
  uint32_t key[U];
  auto fetch = [&](uint32_t n) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = (uint32_t)(u * kSmallBlock) + threadIdx.x;
      key[u] = i < n ? (uint32_t)(i < nd ? dst[i] : col[i - nd]) : 0u;
    }
  };
  fetch((uint32_t)(n_dst + m));  // (as many as there is room for: how many there are is on its way)
  m = edges_there(sizes, m);
  for (uint32_t i = threadIdx.x; i < kSlots; i += kSmallBlock) table[i] = kEmptySlot;
  if (threadIdx.x == 0) st = BucketState{0u, 0u, 0u};
  __syncthreads();
  const uint32_t n = (uint32_t)(n_dst + m);
  unsigned long long mine[U];
  uint32_t h[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = (uint32_t)(u * kSmallBlock) + threadIdx.x;
    h[u] = filter_hash(key[u]) >> (32 - 14);
    mine[u] = i < n ? ((unsigned long long)key[u] << 32) | i : kEmptySlot;
  }
  bucket_insert_many<U>(table, kSlots, h, mine);
  __syncthreads();
  uint32_t f[U];
  const int wave = wave_in_block(), lane = lane_id();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = (uint32_t)(u * kSmallBlock) + threadIdx.x;
    f[u] = i < n ? (uint32_t)table[h[u]] : 0xFFFFFFFFu;
    if (i < n && seed_twice(i, f[u], nd)) st.dup = 1;
    const uint64_t b = ballot64(i >= nd && f[u] == i);
    if (lane == 0) bits[u * kWaves + wave] = b;
  }
  __syncthreads();
  if (wave == 0) {
    constexpr int kEach = (kWords + kWave - 1) / kWave;  // words in a row per lane
    uint32_t c[kEach], sum = 0;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int w = lane * kEach + q;
      c[q] = w < kWords ? (uint32_t)__popcll(bits[w]) : 0u;
      sum += c[q];
    }
    const uint32_t incl = wave_incl_scan(sum);
    uint32_t run = incl - sum;
#pragma unroll
    for (int q = 0; q < kEach; ++q) {
      const int w = lane * kEach + q;
      if (w < kWords) before[w] = run;
      run += c[q];
    }
    if (lane == kWave - 1) {  // the sizes
      Ctl c = *ctl;
      c.total_new = ctl->total_new = incl;
      if (st.dup) c.err_dup = ctl->err_dup = 1;
      if (pub.h != nullptr) send_ctl(pub.h, pub.ticket, c);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = (uint32_t)(u * kSmallBlock) + threadIdx.x;
    if (i >= n) break;
    if (i < nd) {
      src[i] = (int32_t)key[u];
      continue;
    }
    uint32_t local = f[u];
    if (local >= nd) {
      const uint32_t w = f[u] >> 6;
      local = nd + before[w] + (uint32_t)__popcll(bits[w] & ((1ull << (f[u] & 63u)) - 1ull));
      if (f[u] == i) src[local] = (int32_t)key[u];
    }
    col_local[i - nd] = (int32_t)local;
  }
}

__global__ void k_clear_uniq_overflow(Ctl* ctl) { ctl->uniq_overflow = 0; }

static inline unsigned nblocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

int g_unique_mode = 0;  // COOP_TUNE_UNIQUE: 0 automatic, 1 table in HBM, 2 partition whenever it applies, 3 as 2 with buckets 16 times too large

// launches the dedup's kernels up to the one that ranks the new vertices; the sizes are on their way to the host from the
// kernel that finds the first positions on.  col_local serves as the array of first positions (edge order).
enum UniqPath { kByFilter, kByPartition, kByTable, kInOneBlock };
static int unique_launch(const int32_t* dst, int64_t n_dst, const int32_t* col_global, int64_t m, const Ctl* sizes, int32_t* col_local,
                         int32_t* spare, UniqueWork* w, UniqPath path, Alloc& alloc, Ctl* d_ctl, Ctl* h_ctl, hipStream_t s) {
  const int64_t n_all = n_dst + m;
  uint32_t* first = (uint32_t*)col_local;
  w->pub = begin_publish(d_ctl, h_ctl);
  w->path = path;
  uint32_t collect_blocks = (uint32_t)((n_all + kCollectStretch - 1) / kCollectStretch);
  const uint32_t* by_place = nullptr;
  int shift = 0;
  TileNotes notes{};
  w->part_blocks = 0;
  w->n_totals = 0;
  if (path == kInOneBlock) {  // (the relabelling too; spare becomes src_ids)
    if (n_all <= 4 * kSmallBlock)
      COOP_LAUNCH(K_UNIQ_FILTER, k_uniq_small<4>, dim3(1), dim3(kSmallBlock), 0, s, dst, n_dst, col_global, m, sizes, spare, col_local, d_ctl, w->pub);
    else
      COOP_LAUNCH(K_UNIQ_FILTER, k_uniq_small<kSmallEach>, dim3(1), dim3(kSmallBlock), 0, s, dst, n_dst, col_global, m, sizes, spare, col_local, d_ctl,
                  w->pub);
    return COOP_OK;
  }
  if (path == kByFilter) {
    int log2_buckets = kFilterLeastLog2;
    while ((kFilterPairs << log2_buckets) < n_all) ++log2_buckets;
    unsigned long long* bits = w->bits ? (unsigned long long*)w->words : (unsigned long long*)nullptr;
    const uint8_t* tags = w->tagged ? (const uint8_t*)spare : nullptr;
    COOP_LAUNCH(K_UNIQ_FILTER, (tags != nullptr ? k_uniq_filter<true> : k_uniq_filter<false>), dim3(1u << log2_buckets), dim3(kFilterBlock), 0, s, dst,
                n_dst, col_global, tags, m, sizes, log2_buckets, first, bits, d_ctl, w->pub);
  } else if (path == kByPartition) {
    const int64_t n_buckets = w->n_buckets;
    const int64_t by_size = (n_all + 4 * kPartBlock - 1) / (4 * kPartBlock);
    const uint32_t G = (uint32_t)(by_size < kPartMaxBlocks ? (by_size + 7) / 8 * 8 : kPartMaxBlocks);  // a multiple of 8
    const int64_t n_counts = n_buckets * G;
    uint32_t* counts = alloc.get<uint32_t>(n_counts, COOP_TAG_SCRATCH);
    uint32_t* place = alloc.get<uint32_t>(n_counts + 1, COOP_TAG_SCRATCH);
    unsigned long long* pairs = alloc.get<unsigned long long>(n_all, COOP_TAG_SCRATCH);
    notes = TileNotes{first, alloc.get<uint32_t>(kTilePairs, COOP_TAG_SCRATCH), alloc.get<uint16_t>(kTilePairs + m, COOP_TAG_SCRATCH)};
    void* tmp = alloc.get<char>((int64_t)scan_tmp_bytes(n_counts), COOP_TAG_SCRATCH);
    if (alloc.failed) return COOP_E_NOMEM;
    // the first positions, in the buckets' order: into the caller's spare array, else (8-byte steps instead of 4) over the pairs
    uint32_t* firsts = spare ? (uint32_t*)spare : (uint32_t*)pairs;
    shift = spare ? 0 : 1;
    const size_t lds = (size_t)n_buckets * sizeof(uint32_t);
    COOP_LAUNCH(K_PART_COUNT, k_part_count, dim3(G), dim3(kPartBlock), lds, s, dst, n_dst, col_global, m, sizes, (uint32_t)n_buckets, counts);
    const TiledScan<uint32_t> places = scan_u32_tiled(counts, n_counts, place, tmp, d_ctl, s);
    static_assert(kPartMaxBuckets <= 65536 && kTilePairs <= 65536, "a staged pair has 16 bits for either");
    static_assert(kPartMaxBuckets <= 8 * kPartBlock, "a thread of the scatter looks after eight buckets at most");
    if (n_buckets <= 2 * kPartBlock)
      COOP_LAUNCH(K_PART_SCATTER, k_part_scatter<2>, dim3(G), dim3(kPartBlock), 2 * lds, s, dst, n_dst, col_global, m, sizes, (uint32_t)n_buckets,
                  places, pairs, notes);
    else
      COOP_LAUNCH(K_PART_SCATTER, k_part_scatter<8>, dim3(G), dim3(kPartBlock), 2 * lds, s, dst, n_dst, col_global, m, sizes, (uint32_t)n_buckets,
                  places, pairs, notes);
    COOP_LAUNCH(K_PART_FIRST, k_part_first, dim3((unsigned)n_buckets), dim3(kFirstBlock), 0, s, pairs, places, G, n_dst, n_all, firsts, shift, d_ctl,
                w->pub);
    if (hipGetLastError() != hipSuccess) return COOP_E_HIP;  // (a launch that did not happen would leave places or firsts unwritten)
    by_place = firsts;
    collect_blocks = w->part_blocks = G;
  } else {
    // at most half full; an even number of slots (the clear uses 16-byte stores)
    const int64_t cap = 2 * n_all + 1024;
    unsigned long long* table = alloc.get<unsigned long long>(cap, COOP_TAG_SCRATCH);
    if (alloc.failed) return COOP_E_NOMEM;
    if (n_all > 0) {
      fill_u64((uint64_t*)table, cap, kEmptySlot, s);
      COOP_LAUNCH(K_UNIQ_INSERT, k_uniq_insert, dim3(nblocks(n_all)), dim3(kBlock), 0, s, dst, n_dst, col_global, m, sizes, table, (uint64_t)cap,
                  d_ctl);
    }
    if (m > 0)
      COOP_LAUNCH(K_UNIQ_FLAG, k_uniq_lookup, dim3(nblocks(m)), dim3(kBlock), 0, s, col_global, m, sizes, table, (uint64_t)cap, first);
  }
  if (m > 0 && !(path == kByFilter && w->bits)) {
    uint32_t* totals = alloc.get<uint32_t>(2 * (int64_t)collect_blocks, COOP_TAG_SCRATCH);
    if (alloc.failed) return COOP_E_NOMEM;
    // Up to kPartMaxBlocks stretches every block of the relabelling scans their totals for itself, in the place of the block that finishes
    // last here, behind two atomics per block (120 thousand, 1 and 2.4 M entries: this kernel 6.1, 11.3 and 23.0 us -> 4.5, 9.3 and 20.6,
    // the relabelling 18.1 -> 19.3 for the longest).  Only the fallback can have more.
    static_assert(kFilterMax <= kCollectStretch * kPartMaxBlocks, "a short list has no more stretches than that");
    w->n_totals = path != kByTable ? (uint32_t)collect_blocks : 0u;
    uint32_t* const prefix = path != kByTable ? nullptr : totals + collect_blocks;
    w->block_prefix = prefix ? prefix : totals;
    // (the table in HBM does not count its keys: there the ranks bring the number of new vertices, and the sizes leave with them)
    const Publish pub = path == kByTable ? w->pub : Publish{};
    if (by_place)
      COOP_LAUNCH(K_UNIQ_COLLECT, k_uniq_collect<true>, dim3(collect_blocks), dim3(kPartBlock), 0, s, first, by_place, shift, notes, m, sizes, n_dst,
                  w->words, totals, prefix, d_ctl, pub);
    else
      COOP_LAUNCH(K_UNIQ_COLLECT, k_uniq_collect<false>, dim3(collect_blocks), dim3(kPartBlock), 0, s, first, by_place, shift, notes, m, sizes, n_dst,
                  w->words, totals, prefix, d_ctl, pub);
  } else if (path == kByTable && launch_publish(w->pub, s) != COOP_OK) {
    return COOP_E_HIP;
  }
  return COOP_OK;
}

int unique_prepare(int64_t n_dst, int64_t m, bool deferred, UniqueWork* w, Alloc& alloc) {
  const int64_t n_all = n_dst + m;
  const int64_t n_words = (n_all + 63) / 64 - (n_dst >> 6);
  w->words = alloc.get<RankWord>(n_words, COOP_TAG_SCRATCH);
  if (alloc.failed) return COOP_E_NOMEM;
  // by partition from kFilterMax entries on, as long as a block's counters fit LDS
  const int64_t pairs_per_bucket = g_unique_mode == 3 ? 16 * kPartPairs : kPartPairs;
  w->n_buckets = (n_all + pairs_per_bucket - 1) / pairs_per_bucket;
  // two bucket blocks fit a CU: a last round of a few blocks is spread over the others, which grow by an eighth at most.  (One
  // round: lists of 2.2 and 2.3 M entries 20.5 us for the first positions, with the last round 23.4; two: 4.4 and 4.6 M 27.2
  // and 28.1; from three rounds on half a us more there, a bucket of more than 4,096 pairs reading them twice, and one to
  // three less in the scatter, which has fewer buckets: 7.0 M 40.5 and 43.4.)
  const int64_t whole_rounds = w->n_buckets / 512 * 512;
  if (whole_rounds > 0 && n_all <= whole_rounds * (pairs_per_bucket + pairs_per_bucket / 8)) w->n_buckets = whole_rounds;
  const bool by_partition = m > 0 && w->n_buckets <= kPartMaxBuckets && g_unique_mode != 1 && (g_unique_mode >= 2 || n_all >= kFilterMax);
  const bool by_filter = !by_partition && g_unique_mode != 1 && n_all > 0 && n_all < kFilterMax;
  w->tagged = deferred && by_filter && n_all >= kFilterTaggedFrom;
  const bool small = deferred && by_filter && n_all <= kSmallMax;
  w->path = by_partition ? kByPartition : small ? kInOneBlock : by_filter ? kByFilter : kByTable;
  const bool bits = by_filter && !small && n_all <= kShortMax;
  w->clear = bits ? (uint64_t*)w->words : nullptr;
  w->n_clear = bits ? n_words : 0;
  return COOP_OK;
}

int unique_front_launch(const int32_t* dst, int64_t n_dst, const int32_t* col_global, int64_t m, const Ctl* sizes, int32_t* col_local,
                        int32_t* spare, UniqueWork* w, Alloc& alloc, Ctl* d_ctl, Ctl* h_ctl, hipStream_t s) {
  // (Words that nobody has cleared on the way, the list's length having been unknown, are left to k_uniq_collect: a launch as well,
  // and 2 us less than clearing them here.)
  w->bits = w->n_clear != 0 && w->clear == nullptr;
  return unique_launch(dst, n_dst, col_global, m, sizes, col_local, spare, w, (UniqPath)w->path, alloc, d_ctl, h_ctl, s);
}

int unique_front_finish(const int32_t* dst, int64_t n_dst, const int32_t* col_global, int64_t m, const Ctl* sizes, int32_t* col_local,
                        UniqueWork* w, Alloc& alloc, Ctl* d_ctl, Ctl* h_ctl, hipStream_t s, bool* redone) {
  *redone = false;
  int rc = wait_ctl(w->pub, h_ctl, s);
  if (rc != COOP_OK) return rc;
  if (w->path != kByTable && h_ctl->uniq_overflow != 0) {  // a bucket's table overflowed: once more through the table in HBM
    hipLaunchKernelGGL(k_clear_uniq_overflow, dim3(1), dim3(1), 0, s, d_ctl);
    rc = unique_launch(dst, n_dst, col_global, m, sizes, col_local, nullptr, w, kByTable, alloc, d_ctl, h_ctl, s);
    if (rc != COOP_OK) return rc;
    rc = wait_ctl(w->pub, h_ctl, s);
    if (rc != COOP_OK) return rc;
    *redone = true;
  }
  w->n_new = m > 0 ? h_ctl->total_new : 0;
  return COOP_OK;
}

int unique_back(const int32_t* dst, int64_t n_dst, const int32_t* col_global, int64_t m, const Ctl* sizes, const UniqueWork& w,
                int32_t* col_local, int32_t* src, hipStream_t s) {
  const int64_t n_threads = m > n_dst ? m : n_dst;
  const RankView rank{w.words, w.block_prefix, w.part_blocks, w.n_totals};
  if (w.path == kInOneBlock) return COOP_OK;
  if (n_threads > 0 && w.path == kByFilter && w.bits)
    COOP_LAUNCH(K_UNIQ_RELABEL, k_uniq_relabel_short, dim3((unsigned)((n_threads + kShortBlock * kShortEach - 1) / (kShortBlock * kShortEach))),
                dim3(kShortBlock), 0, s, dst, col_global, m, sizes, n_dst, (const unsigned long long*)w.words, src, col_local);
  else if (n_threads > 0)
    COOP_LAUNCH(K_UNIQ_RELABEL, k_uniq_relabel, dim3(nblocks((n_threads + kRelabelUnroll - 1) / kRelabelUnroll)), dim3(kBlock), 0, s, dst, col_global, m, sizes, n_dst, rank, src, col_local);
  return COOP_OK;
}

}  // namespace coop
