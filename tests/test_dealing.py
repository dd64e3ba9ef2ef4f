"""How the lists of a pass are dealt to one-wave blocks (csrc/dealing.h), compiled for the CPU: every list once, and no more blocks than
the lists are worth."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_12403_amd", "csrc")
SHIM = r"""
#include "dealing.h"
using namespace coop;
extern "C" int64_t blocks_of(int64_t n, int each_log2, int finer, uint8_t* taken) {
  const Dealing d = deal_lists(n, each_log2, finer != 0);
  for (uint32_t b = 0; taken != nullptr && b < d.blocks; ++b) {
    int log2 = 0;
    const int64_t w0 = d.first_list(b, &log2);
    if (w0 >= n) return -1;
    for (int64_t w = w0; w < w0 + ((int64_t)1 << log2) && w < n; ++w) taken[w] += 1;
  }
  return d.blocks;
}
extern "C" int64_t out_of_place(int64_t n, int each_log2) {
  const Dealing d = deal_lists(n, each_log2, false);
  int64_t bad = 0;
  for (uint32_t b = 0; b < (uint32_t)(n >> each_log2); ++b) {
    int log2 = 0;
    bad += d.first_list(b, &log2) != (int64_t)xcd_runs(b, (uint32_t)(n >> each_log2)) << each_log2;
  }
  return bad;
}
extern "C" int finer(int64_t n_edges, const int64_t* census, int64_t n_vertices, int each_log2, int of_edges) {
  return finer_last(Degrees{n_edges, census, n_vertices}, each_log2, of_edges != 0);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("dealing")
    src, out = str(d / "shim.cpp"), str(d / "shim.so")
    open(src, "w").write(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", out])
    so = C.CDLL(out)
    so.blocks_of.restype = so.out_of_place.restype = C.c_int64
    return so


def sizes():
    rng = np.random.default_rng(0)
    return [1, 2, 3, 7, 8, 9, 32767, 32768, 32769, 65535, 131071, 131072, 131073] + [int(x) for x in np.exp(rng.uniform(0, 13, 60))]


@pytest.mark.parametrize("finer", [0, 1])
@pytest.mark.parametrize("each_log2", range(7))
def test_every_list_once(lib, each_log2, finer):
    for n in sizes():
        taken = np.zeros(n, dtype=np.uint8)
        blocks = lib.blocks_of(C.c_int64(n), each_log2, finer, taken.ctypes.data_as(C.c_void_p))
        assert blocks > 0 and (taken == 1).all(), n
        least = -(-n // (1 << each_log2))
        if not finer:
            assert blocks == least, n
        else:
            assert least <= blocks <= least + min(n, 16384 + (1 << each_log2)), n


def test_an_even_dealing_is_one_run(lib):
    """Where no list is dealt finer the neighbours that an XCD takes are those of the whole pass, not of two halves."""
    for n in sizes():
        for each_log2 in range(4):
            assert lib.out_of_place(C.c_int64(n), each_log2) == 0, (n, each_log2)


def asked(lib, degrees, each_log2, of_edges, census=True):
    degrees = np.asarray(degrees, dtype=np.int64)
    counts = np.bincount(np.floor(np.log2(np.maximum(degrees[degrees > 0], 1))).astype(np.int64), minlength=32).astype(np.int64)
    return bool(lib.finer(C.c_int64(int(degrees.sum())), counts.ctypes.data_as(C.c_void_p) if census else None, C.c_int64(len(degrees)), each_log2,
                          int(of_edges)))


@pytest.mark.parametrize("census", [True, False])
@pytest.mark.parametrize("of_edges", [False, True])
def test_short_lists_start_no_more_waves(lib, of_edges, census):
    """Lists that a wave looks at together, 128 >> each_log2 entries at most, take the same time however many there are."""
    for each_log2 in range(4):
        together = 128 >> each_log2
        for d in (1, 7, 10, together // 2, together):
            assert not asked(lib, np.full(5000, d), each_log2, of_edges, census), (each_log2, d)
        assert not asked(lib, np.random.default_rng(1).integers(0, together + 1, 5000), each_log2, of_edges, census)
        for d in (2 * together, 5 * together):
            assert asked(lib, np.full(5000, d), each_log2, of_edges, census) == (each_log2 >= 2), (each_log2, d)


def test_a_power_law_by_what_its_edges_lead_to(lib):
    """Most lists are short and most edges lead to long ones: the seeds' pass is dealt by the former, the later ones by the latter."""
    d = (np.arange(300000) + 30.0) ** -0.9
    degrees = np.maximum(d * 9e6 / d.sum(), 1).astype(np.int64)
    for each_log2 in (2, 3):
        assert not asked(lib, degrees, each_log2, False) and asked(lib, degrees, each_log2, True)
