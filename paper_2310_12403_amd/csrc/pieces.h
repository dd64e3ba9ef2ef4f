// How a LABOR-0 pass cuts its long lists into pieces, and the room that their queue needs.  No GPU in here: the host decides, the
// kernels ask PieceCut, and a test runs all of it on the CPU.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define COOP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define COOP_HOST_DEVICE inline
#endif

namespace coop {

constexpr int kPieceLenAuto = -1;   // COOP_TUNE_PIECE_LEN: as long as is best, that is ...
constexpr int kPieceLen = 4096;     // ... so many entries ...
constexpr int kFewPieceLen = 1024;  // ... and so many in passes over fewer than kFewLists lists
constexpr int64_t kFewLists = 16384;
constexpr uint32_t kNoBound = 0xFFFFFFFFu;
constexpr uint32_t kMostPiecesOfAList = 1u << 20;  // keeps the sum over the 1,024 lists of a block at 2^30

// Lists longer than split_min are queued in pieces of about len entries, of each list no more than it has pieces of whole_len and
// `extra` (kNoBound: as many as there are).  len == 0: nothing is queued.
struct PieceCut {
  uint32_t split_min = 0, len = 0, whole_len = 0, extra = kNoBound;
  COOP_HOST_DEVICE uint32_t pieces(uint32_t d) const {
    uint32_t np = (d - 1) / len + 1;
    if (extra != kNoBound) {
      const uint32_t most = (d - 1) / whole_len + 1 + extra;
      np = np < most ? np : most;
    }
    return np < kMostPiecesOfAList ? np : kMostPiecesOfAList;
  }
  // their length: equal, a multiple of 4
  COOP_HOST_DEVICE uint32_t each(uint32_t d) const { return ((d - 1) / pieces(d) + 4u) & ~3u; }
};
// Where piece q of a list of d entries in pieces of `each` starts, and its length.  (Below 0: nowhere.  Rounding the length up can
// leave the last slots of a very long list empty.)
COOP_HOST_DEVICE int64_t piece_start(uint32_t d, uint32_t each, uint32_t q, uint32_t* length) {
  const uint64_t j0 = (uint64_t)q * each;
  if (j0 >= d) return -1;
  *length = d - (uint32_t)j0 < each ? d - (uint32_t)j0 : each;
  return (int64_t)j0;
}

// What is known of a graph's degrees: census[k] lists have at least 2^k and fewer than 2^(k+1) entries (null: nobody looked).
struct Degrees {
  int64_t n_edges;
  const int64_t* census;
  int64_t n_vertices = 0;
  // do most vertices, or, of_edges, most of those that an edge leads to in a graph with every edge both ways, have at least `len` entries
  // (a power of two)?  Of a graph that nobody looked at: does the mean list?
  bool most_have(int64_t len, bool of_edges) const {
    if (census == nullptr) return n_edges >= len * n_vertices;
    int64_t lists = 0, shorter = 0;
    for (int k = 0; k < 32; ++k) {
      if ((int64_t)1 << k >= len) lists += census[k];
      else shorter += census[k] * ((int64_t)3 << k) / 2;
    }
    return of_edges ? 2 * shorter <= n_edges : 2 * lists >= n_vertices;
  }
  // at most so many of n distinct lists have more than split_min entries ...
  int64_t longer(int64_t n, uint32_t split_min) const {
    int64_t most = n_edges / ((int64_t)split_min + 1);
    if (census != nullptr) {
      int64_t there = 0;
      for (int k = 31; k >= 0 && ((int64_t)2 << k) - 1 > (int64_t)split_min; --k) there += census[k];
      most = there < most ? there : most;
    }
    return n < most ? n : most;
  }
  // ... and those have at most so many pieces of len
  int64_t pieces(int64_t n, uint32_t split_min, uint32_t len) const {
    const int64_t lists = longer(n, split_min);
    if (lists == 0) return 0;
    const int64_t by_edges = n_edges / len + lists;  // (a list of d entries has at most d / len + 1)
    if (census == nullptr) return by_edges;
    int64_t by_census = 0, left = lists;
    for (int k = 31; k >= 0 && left > 0; --k) {
      const int64_t n_k = census[k] < left ? census[k] : left;
      by_census += n_k * ((((int64_t)2 << k) - 2) / len + 1);
      left -= n_k;
    }
    return by_census < by_edges ? by_census : by_edges;
  }
};

// piece_len, split_set: the knobs (0: never cut, kPieceLenAuto: automatic; 0: automatic).  room_most: what the caller has room for at most.  *room: entries of
// the queue, enough for all pieces of distinct destinations (a queue that room_most keeps shorter may leave lists whole).
//
// Lists longer than split_min go to the piece waves, which come first in the grid.  With independent variates that is for the
// lists worth cutting (twice the piece length).  The blended scan costs three times as much per entry, and a wave that meets a few
// lists of several thousand entries late in the kernel keeps it waiting: there every list above 2,048 entries goes first, whole if
// it is shorter than two pieces (papers100M-shaped, kappa 16: scan 1.44 -> 1.32 ms; no difference with independent variates).
//
// A pass over fewer than kFewLists lists does not fill the chip with them and ends when its longest list does: those are cut into
// pieces that one step of a wave's requests covers, as far as the queue has room for that, which stays as long as pieces of
// kPieceLen make it.  (64 seeds, three layers 147 -> 142 us, 1,024 seeds 117 -> 114, both with pieces of 1,024; of 512 144 and
// 115.)  What pieces of kPieceLen leave free by the degrees that were counted at registration is shared out among the lists, so
// that none stays whole: that costs far more than fine pieces give (20 destinations and a list of 2 million entries that are
// nearly all of the graph's 49 us, left whole 1,575).  A graph that nobody looked at has nothing to share out.
inline PieceCut cut_pieces(int64_t n_new, const Degrees& g, bool blend, int piece_len, int split_set, int64_t room_most, int64_t* room) {
  PieceCut cut;
  *room = 0;
  if (piece_len == 0 || n_new <= 0) return cut;
  const bool automatic = piece_len == kPieceLenAuto;
  cut.len = cut.whole_len = (uint32_t)(automatic ? kPieceLen : piece_len);
  cut.split_min = split_set != 0 ? (uint32_t)split_set : (blend && cut.len >= 2048u ? 2048u : 2u * cut.len);
  const int64_t room_lists = g.n_edges / (int64_t)cut.split_min + 1;
  const int64_t enough = g.n_edges / (int64_t)cut.len + (n_new < room_lists ? n_new : room_lists) + 1;
  *room = enough < room_most ? enough : room_most;
  if (n_new < kFewLists && automatic && split_set == 0) {
    const PieceCut fine{2 * kFewPieceLen, kFewPieceLen, kPieceLen, kNoBound};
    const int64_t lists = g.longer(n_new, fine.split_min), spare = *room - g.pieces(n_new, fine.split_min, kPieceLen);
    if (g.pieces(n_new, fine.split_min, kFewPieceLen) <= *room) {
      cut = fine;
    } else if (spare >= 0) {
      cut = fine;
      cut.extra = (uint32_t)(spare / lists);
    }
  }
  if (g.longer(n_new, cut.split_min) == 0) {  // (no list is that long: nothing is queued)
    *room = 0;
    return PieceCut{};
  }
  return cut;
}

}  // namespace coop
