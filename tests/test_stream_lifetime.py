"""Memory that the binding takes from torch for work on a stream other than torch's current one: torch hands it out again as soon as the
last tensor over it goes, unless it has been told of that stream."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2310_12403_amd as P
from paper_2310_12403_amd import binding


class Buffer:
    """What _take gets from torch.empty, on the host, noting the streams it is recorded on."""
    made = []

    def __init__(self, nbytes):
        self.memory = (C.c_uint8 * nbytes)()
        self.streams = []
        Buffer.made.append(self)

    def data_ptr(self):
        return C.addressof(self.memory)

    def record_stream(self, stream):
        self.streams.append(stream)


class Stream:
    def __init__(self, idle=True):
        self.cuda_stream, self.idle = id(self), idle

    def record_event(self):
        return self

    def query(self):
        return self.idle


@pytest.fixture
def buffers(monkeypatch):
    Buffer.made = []
    monkeypatch.setattr(binding.torch, "empty", lambda n, **kw: Buffer(n))
    monkeypatch.setattr(binding, "_torch_stream", lambda stream: stream)
    return Buffer.made


@pytest.mark.parametrize("queued,idle", [(True, True), (True, False), (False, True)])
def test_torch_is_told_of_a_stream_that_is_still_at_work(buffers, queued, idle):
    """... when the last block of a call goes, or of a call that has failed; not of one that is through with the call."""
    side = Stream(idle)
    al = binding._SampleAllocator(torch.device("cpu"), side)
    assert all(binding._take(al.key, n, 0) for n in (1, 256, 5000))
    if queued:
        al.called()
    assert [b.streams for b in buffers] == [[]] * 3
    del al
    assert [b.streams for b in buffers] == [[] if queued and idle else [side]] * 3
    del buffers[:]
    al = binding._SampleAllocator(torch.device("cpu"))     # (torch's current stream: the memory is that one's)
    assert binding._take(al.key, 256, 0)
    al.called()
    del al
    assert [b.streams for b in buffers] == [[]]


def test_memory_that_outlives_a_call(buffers):
    """A cache's, a graph's: every stream is recorded, once for what it has been told of."""
    al = binding._TorchAllocator(torch.device("cpu"))
    one, two = Stream(), Stream()
    assert all(binding._take(al.key, n, 0) for n in (1, 256))
    for stream in (one, None, one, two, one, two):
        al.used_on(stream)
    assert [b.streams for b in buffers] == [[one, two]] * 2
    assert binding._take(al.key, 4096, 0)
    al.used_on(two)
    assert buffers[2].streams == [two]


@pytest.mark.gpu
@pytest.mark.parametrize("sampler", [P.COOP_NS, P.COOP_LABOR0, P.COOP_RW])
def test_blocks_dropped_while_the_stream_is_at_work(sampler):
    """What a call on another stream took does not come back from torch before that stream has got there."""
    n = 2000
    rng = np.random.default_rng(3)
    indptr = torch.arange(0, 20 * n + 1, 20, dtype=torch.int64).cuda()
    indices = torch.from_numpy(rng.integers(0, n, 20 * n).astype(np.int32)).cuda()
    g = P.coop_graph_load(indptr, indices, P.COOP_VALIDATE)
    seeds = torch.arange(700, dtype=torch.int32).cuda()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def call():
        return P.coop_sample_rw(g, seeds, (5, 5), 2, 8, 0.5, stream=side) if sampler == P.COOP_RW else \
            P.coop_sample(g, seeds, (5, 5), sampler, stream=side)
    blocks = call()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)        # (a tenth of a second, or two seconds by a slow clock)
        done = torch.cuda.Event()
        done.record()
        if blocks[0]._alloc.done is not None:
            blocks[0]._alloc.done.record()    # (as if the call's own work took that long)
    held = {t.untyped_storage().data_ptr(): t.untyped_storage().nbytes() for t in blocks[0]._alloc.tensors.values()}
    del blocks
    again = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for nbytes in held.values() for _ in range(2)]
    assert not done.query(), "the sleep ended too early for this to say anything"
    assert not held.keys() & {t.untyped_storage().data_ptr() for t in again}
    side.synchronize()
