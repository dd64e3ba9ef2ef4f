"""How a LABOR-0 pass cuts its long lists into pieces (csrc/pieces.h), compiled for the CPU: whatever lists a pass meets, the queue
has room for all of their pieces, so that no list is left to a single wave."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_12403_amd", "csrc")
SHIM = r"""
#include "pieces.h"
using namespace coop;
extern "C" int64_t queue_of(const uint32_t* degree, int64_t n, int64_t n_edges, const int64_t* census, int blend, int piece_len, int split_set,
                            int64_t room_most, int64_t* room, int64_t* shortest, int64_t* longest, int64_t* uncovered) {
  const PieceCut cut = cut_pieces(n, Degrees{n_edges, census}, blend != 0, piece_len, split_set, room_most, room);
  int64_t total = 0;
  *shortest = (int64_t)1 << 40; *longest = 0; *uncovered = 0;
  for (int64_t i = 0; i < n; ++i) {
    const uint32_t d = degree[i];
    if (cut.len == 0 || d <= cut.split_min) {
      if (piece_len != 0 && d > *longest) *longest = d;  // one wave's
      continue;
    }
    const uint32_t np = cut.pieces(d);
    total += np;
    int64_t at = 0;
    for (uint32_t q = 0; q < np; ++q) {
      uint32_t len = 0;
      const int64_t j0 = piece_start(d, cut.each(d), q, &len);
      if (j0 < 0) continue;
      if (j0 != at || len == 0 || (j0 & 3)) *uncovered += 1;
      at = j0 + len;
      if (len > *longest) *longest = len;
    }
    if (at != d) *uncovered += 1;
    const int64_t mean = d / np;
    if (mean < *shortest) *shortest = mean;
  }
  return total;
}
extern "C" int64_t most_pieces(int64_t n, int64_t n_edges, const int64_t* census, uint32_t split_min, uint32_t len) {
  return Degrees{n_edges, census}.pieces(n, split_min, len);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    open(src, "w").write(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib])
    so = C.CDLL(lib)
    so.queue_of.restype = so.most_pieces.restype = C.c_int64

    def queue_of(graph, taken, census=True, blend=False, piece_len=-1, split_set=0, room_most=1 << 30):
        """graph: all degrees; taken: those of the destinations.  (room, pieces, mean length of the finest cut, longest stretch)"""
        graph, taken = np.ascontiguousarray(graph, dtype=np.int64), np.ascontiguousarray(taken, dtype=np.uint32)
        counts = np.bincount(np.log2(np.maximum(graph[graph > 0], 1)).astype(np.int64), minlength=32).astype(np.int64)
        out = [C.c_int64() for _ in range(4)]
        total = so.queue_of(taken.ctypes.data_as(C.c_void_p), C.c_int64(len(taken)), C.c_int64(int(graph.sum())),
                            counts.ctypes.data_as(C.c_void_p) if census else None, int(blend), piece_len, split_set, C.c_int64(room_most),
                            *[C.byref(o) for o in out])
        assert out[3].value == 0, "a list is not covered by its pieces"
        return out[0].value, total, out[1].value, out[2].value
    queue_of.lib = so
    return queue_of


def hubs(n, each, rest, seed=0):
    return np.concatenate([np.full(n, each), np.random.default_rng(seed).integers(0, 25, rest)])


GRAPHS = {
    "one hub": (hubs(1, 2000000, 50000), 21),
    "a hundred hubs": (hubs(100, 200000, 200000), 3000),
    "a thousand hubs": (hubs(1000, 20000, 200000), 3000),
    "lists around the border": (hubs(3000, 2049, 10000), 3000),
    "lists twice the border": (hubs(2000, 4097, 10000), 16383),
    "hubs of two lengths": (np.concatenate([hubs(50, 300000, 100000), np.full(2000, 2500)]), 5000),
    "all lists long": (np.random.default_rng(1).integers(3000, 9000, 8000), 8000),
}


@pytest.mark.parametrize("blend", [False, True])
@pytest.mark.parametrize("census", [True, False])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_the_queue_holds_every_piece(rule, name, census, blend):
    graph, n = GRAPHS[name]
    taken = np.sort(graph)[::-1][:n]                   # distinct destinations, the longest lists among them
    room, total, _, longest = rule(graph, taken, census, blend)
    assert total <= room
    assert longest <= 8192, "a list of that length is one wave's"
    whole = int(graph.sum()) // 4096 + min(n, int(graph.sum()) // (2048 if blend else 8192) + 1) + 1
    assert room <= whole                               # (no more memory than pieces of 4,096 ask for)


def test_random_graphs(rule):
    rng = np.random.default_rng(5)
    for case in range(300):
        size = int(rng.integers(10, 5000))
        graph = np.exp(rng.uniform(0, np.log(10.0 ** rng.uniform(1, 6)), size)).astype(np.int64)
        n = int(rng.integers(1, min(size, 16383) + 1))
        taken = rng.permutation(graph)[:n] if case % 2 else np.sort(graph)[::-1][:n]
        blend, census = bool(rng.integers(2)), bool(rng.integers(2))
        for piece_len, split_set in ((-1, 0), (-1, 500), (4096, 0), (256, 0), (512, 1000), (4096, 64)):
            room, total, _, _ = rule(graph, taken, census, blend, piece_len, split_set)
            assert total <= room, (case, piece_len, split_set)
        counts = np.bincount(np.log2(np.maximum(graph, 1)).astype(np.int64), minlength=32).astype(np.int64)
        for split, length in ((2048, 1024), (2048, 4096), (300, 256)):
            most = rule.lib.most_pieces(C.c_int64(n), C.c_int64(int(graph.sum())), counts.ctypes.data_as(C.c_void_p), split, length)
            assert int((-(-taken[taken > split] // length)).sum()) <= most


def test_few_ordinary_lists_are_cut_finely(rule):
    """A power law such as the configurations have: pieces of about 1,024, and all of them find room."""
    d = (np.arange(150000) + 300.0) ** -0.9
    graph = np.minimum(d * 7.7e6 / d.sum(), 30000).astype(np.int64)
    assert graph.max() > 2048
    for n in (24, 300, 3000, 16383):
        room, total, finest, longest = rule(graph, np.sort(graph)[::-1][:n])
        assert total <= room and 600 <= finest <= 1024 and longest <= 2048, (n, room, total, finest, longest)
    assert rule(graph, np.sort(graph)[::-1][:16384])[3] <= 8192


def test_what_the_caller_has_room_for(rule):
    """Unaligned indices: the queue lies in an array of a size of its own."""
    graph = hubs(10, 500000, 20000)
    for room_most in (5, 600, 1300, 4500):
        room, total, _, _ = rule(graph, np.sort(graph)[::-1][:300], room_most=room_most)
        assert room <= room_most
        assert total <= room or room_most < 1221 + 10   # (fewer entries than pieces of 4,096: lists may stay whole)


@pytest.mark.parametrize("blend", [False, True])
def test_a_length_that_was_asked_for(rule, blend):
    """4,096 asked for is 4,096 in small passes too, with the queue that belongs to it."""
    for name, (graph, n) in GRAPHS.items():
        taken = np.sort(graph)[::-1][:n].astype(np.int64)
        room, total, _, longest = rule(graph, taken, blend=blend, piece_len=4096)
        long = taken[taken > (2048 if blend else 8192)]
        assert total == int((-(-long // 4096)).sum()), name
        assert total <= room
