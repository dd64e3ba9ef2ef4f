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


@pytest.fixture
def buffers(monkeypatch):
    Buffer.made = []
    monkeypatch.setattr(binding.torch, "empty", lambda n, **kw: Buffer(n))
    monkeypatch.setattr(binding, "_torch_stream", lambda stream: stream)
    return Buffer.made


def test_a_callback_tells_torch_of_the_stream(buffers):
    side = object()
    for kind in (binding._TorchAllocator, binding._SampleAllocator):
        del buffers[:]
        al = kind(torch.device("cpu"), side)
        assert all(binding._take(al.key, n, 0) for n in (1, 256, 5000))
        assert [b.streams for b in buffers] == [[side]] * 3
        other = object()
        al.used_on(other)       # a later call on memory that outlives the first one (a cache's, a graph's)
        assert [b.streams[1:] for b in buffers] == [[other]] * 3
        al.used_on(None)        # (torch's current stream: the memory is that one's)
        assert all(len(b.streams) == 2 for b in buffers)
        del buffers[:]
        al = kind(torch.device("cpu"))
        assert binding._take(al.key, 256, 0) and buffers[0].streams == []


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
    held = {t.untyped_storage().data_ptr(): t.untyped_storage().nbytes() for t in blocks[0]._alloc.tensors.values()}
    del blocks
    again = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for nbytes in held.values() for _ in range(2)]
    assert not done.query(), "the sleep ended too early for this to say anything"
    assert not held.keys() & {t.untyped_storage().data_ptr() for t in again}
    side.synchronize()
