// How the lists of a pass are dealt to the waves that look at them.  No GPU in here: a test runs it on the CPU.
#pragma once
#include "pieces.h"

namespace coop {

// Block b of n, renumbered so that an XCD (blocks are dealt to the eight in turn) takes runs of 32 neighbouring numbers: what
// neighbours read, records and offsets, then shares the cache lines of one L2.  (A bijection of 0 .. n - 1.)
COOP_HOST_DEVICE uint32_t xcd_runs(uint32_t b, uint32_t n) {
  const uint32_t whole = n & ~255u;
  return b < whole ? (b & ~255u) | ((b & 7u) << 5) | ((b >> 3) & 31u) : b;
}

// Neighbouring lists for each one-wave block, a quarter as many for the last blocks (`finer`), so that the waves end more nearly
// together (eight lists are some 35 us of a wave's time on the reddit shape, and without this the number of waves in flight fell for the
// last 25 us of 132).  The last 16,384 lists, two for each of the 8,192 waves that the chip holds: steps of the reddit shape 647 -> 641
// us, papers100M 1,098 -> 1,085, dependent batches 1,034 -> 1,025; with 8,192 lists 643, 1,090 and 1,027, with 32,768 642, 1,083 and
// 1,026, with 65,536 650 and more, for starting a wave costs as well.
constexpr int64_t kTailLists = 16384;
constexpr int kTailShift = 2;
struct Dealing {
  uint32_t head, blocks;     // of `blocks` blocks the first `head` take 2^head_log2 lists each, the others 2^tail_log2
  int head_log2, tail_log2;
  COOP_HOST_DEVICE int64_t first_list(uint32_t b, int* each_log2) const {
    const bool in_head = b < head;
    *each_log2 = in_head ? head_log2 : tail_log2;
    const uint32_t at = in_head ? xcd_runs(b, head) : xcd_runs(b - head, blocks - head);
    return ((int64_t)(in_head ? 0u : head) << head_log2) + ((int64_t)at << *each_log2);
  }
};
inline Dealing deal_lists(int64_t n, int each_log2, bool finer) {
  Dealing d{0, 0, each_log2, each_log2};
  if (finer) d.tail_log2 = each_log2 > kTailShift ? each_log2 - kTailShift : 0;
  const int64_t tail = d.tail_log2 == each_log2 ? 0 : n / 2 < kTailLists ? n / 2 : kTailLists;
  d.head = (uint32_t)((n - tail) >> each_log2);
  const int64_t rest = n - ((int64_t)d.head << each_log2);
  d.blocks = d.head + (uint32_t)((rest + ((int64_t)1 << d.tail_log2) - 1) >> d.tail_log2);
  return d;
}
// Finer for the last ones?  Only where most lists keep a wave busy one after the other.  A wave of 2^e lists looks at those of up to
// 128 >> e entries together, so that its time does not depend on how many there are, and starting more waves is all that it comes to:
// the scan of 70 thousand lists of 10 entries, four to a wave, 9.5 us, with the last ones dealt one by one 13.2, with dependent variates
// 193 and 492.  From twice that length on it gains: 140 thousand lists of 32 entries, eight to a wave, 29.1 -> 25.9 (LABOR-0), 59.7 ->
// 56.1 (NS), of 16, or 1 to 31, 10.3 -> 11.1 and 24.4 -> 21.2.  Four to a wave it is the lists' different lengths that it is for: 70
// thousand of 64 entries 18.1 -> 18.8, of 256 23.9 -> 23.9 (NS 37.1 -> 36.4), the products-shaped step 637 -> 628.  Two to a wave: 40
// thousand of 256 entries 16.9 and 17.5, NS 25.5 and 25.9, of 32 entries 9.4 and 12.2, 23.5 and 23.9: never.
inline bool finer_last(const Degrees& g, int each_log2, bool of_edges) { return each_log2 >= 2 && g.most_have(256 >> each_log2, of_edges); }

}  // namespace coop
