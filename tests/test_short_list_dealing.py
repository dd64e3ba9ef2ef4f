"""The dedup of short lists gives every bucket of keys a block, whose waves note the positions of the bucket's keys in lists of
fixed length; a wave that has more to note sends its block over the whole list again.  This deals lists of distinct and of
repeated keys out as the kernel does, on the CPU and with the kernel's own constants, and checks that ordinary ones do not
come near that length."""
import os
import re

import numpy as np
import pytest

_SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_12403_amd", "csrc", "unique.hip")


def constants():
    text = open(_SRC).read()
    found = re.findall(r"constexpr (?:int|uint32_t|int64_t) (kFilter[A-Za-z0-9]+) = ([0-9]+)[;u]", text)
    k = {name: int(v) for name, v in found}
    k["hash"] = int(re.search(r"filter_hash\(uint32_t key\) { return key \* (0x[0-9A-F]+)u", text).group(1), 16)
    return k


def most_noted(keys, n_dst, k):
    log2 = k["kFilterLeastLog2"]
    while (k["kFilterPairs"] << log2) < len(keys):
        log2 += 1
    bucket = ((keys.astype(np.uint64) * np.uint64(k["hash"])) & np.uint64(0xFFFFFFFF)) >> np.uint64(32 - log2)
    at = np.concatenate([np.arange(n_dst), np.arange(len(keys) - n_dst)])    # each part is dealt out from its own beginning
    wave = at // 256 % (k["kFilterBlock"] // 64)                             # a wave's load takes 64 groups of four keys
    noted = np.zeros((1 << log2, k["kFilterBlock"] // 64), dtype=np.int64)
    np.add.at(noted, (bucket.astype(np.int64), wave), 1)
    return noted.max()


@pytest.mark.parametrize("n_dst,fanout", [(256, 5), (400, 4), (512, 3), (682, 2), (1024, 1), (24, 10), (1000, 3), (2047, 1), (300, 40), (4352, 1),
                                          (16000, 1), (20000, 5), (43000, 5)])
def test_waves_have_room(n_dst, fanout):
    k = constants()
    n = n_dst * (fanout + 1)
    assert n < k["kFilterMax"]
    rng = np.random.default_rng(n)
    for _ in range(10):
        distinct = rng.permutation(300000)[:n]
        sources = np.concatenate([distinct[:n_dst], rng.choice(distinct, n - n_dst)])   # and edges that share sources
        for keys in (distinct, sources):
            assert most_noted(keys, n_dst, k) <= 0.8 * k["kFilterList"]
