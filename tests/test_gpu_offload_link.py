"""Offload and prefetch over the link: pinned and pageable host memory, staging buffers and host buffers
that are not 16-byte aligned, streams that end at every byte of a 16-byte chunk, small streams and some of
16 MB, one stream and two, and several tensors through one workspace and one size word while their copies
wait.  The oracle's streams, and nothing beside them."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"


def round_trip(x, expect, pinned=True, stage_offset=0, host_offset=0, one_stream=False, size_pinned=True):
    n, w = x.numel(), x.element_size()
    compute = torch.cuda.Stream()
    copy = compute if one_stream else torch.cuda.Stream()
    cap = zvc.zvc_max_compressed_bytes(n, w)
    stage = torch.zeros(cap + 64, dtype=torch.uint8, device=DEV)[stage_offset:stage_offset + cap]
    room = torch.full((cap + 64,), 0x5A, dtype=torch.uint8, pin_memory=pinned)
    host = room[host_offset:host_offset + cap]
    h_bytes = torch.zeros(1, dtype=torch.int64, pin_memory=size_pinned)
    ws = zvc.new_workspace(n, w, DEV)
    torch.cuda.synchronize()
    nbytes = zvc.zvc_offload(x, stage, host, h_bytes, ws, compute, copy)
    copy.synchronize()
    assert nbytes == expect.size == int(h_bytes[0])
    assert np.array_equal(host[:nbytes].numpy(), expect)
    assert bool((room[:host_offset] == 0x5A).all()) and bool((room[host_offset + nbytes:] == 0x5A).all())
    stage.fill_(0xCD)
    out = torch.zeros_like(x)
    torch.cuda.synchronize()
    zvc.zvc_prefetch(host, nbytes, stage, out, ws, copy, compute)
    compute.synchronize()
    assert np.array_equal(raw_bytes(out), raw_bytes(x))
    assert bool((stage[nbytes:] == 0xCD).all())


@pytest.mark.parametrize("w", [4, 2])
def test_every_end_of_a_stream(oracle, w):
    n = 9000 + 33
    for kept in range(700, 700 + 16 // w):
        x = torch.zeros(n, dtype={4: torch.float32, 2: torch.bfloat16}[w])
        x[torch.randperm(n, generator=torch.Generator().manual_seed(kept))[:kept]] = 1.5
        expect = oracle.compress_stream(raw_bytes(x), w)
        say("end w=%d stream bytes %d" % (w, expect.size))
        round_trip(x.to(DEV), expect, one_stream=kept % 2 == 0)


@pytest.mark.parametrize("how", [dict(pinned=False), dict(size_pinned=False), dict(pinned=False, size_pinned=False),
                                 dict(stage_offset=4), dict(host_offset=4), dict(host_offset=16), dict(host_offset=1),
                                 dict(stage_offset=8, pinned=False, one_stream=True)])
def test_memory_of_every_kind(oracle, how):
    x = random_tensor(70001, 4, 0.4, seed=3)
    expect = oracle.compress_stream(raw_bytes(x), 4)
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipPeekAtLastError() == 0
    say("offload %r" % (how,))
    round_trip(x, expect, **how)
    assert hip.hipPeekAtLastError() == 0


@pytest.mark.parametrize("n,w,density", [(4400000, 4, 0.9), (4400000, 4, 0.95), (9000000, 2, 0.92), (20000, 4, 1.0)])
def test_large_streams(oracle, n, w, density):
    """Streams just below and above 16 MB, and a dense small one."""
    x = random_tensor(n, w, density, seed=n)
    expect = oracle.compress_stream(raw_bytes(x), w)
    say("large n=%d w=%d stream bytes %d" % (n, w, expect.size))
    round_trip(x, expect)


def test_several_tensors_while_their_copies_wait(oracle):
    """The copy stream is kept busy; size word, workspace and streams are shared, staging and host
    buffers are each tensor's own."""
    compute, copy = torch.cuda.Stream(), torch.cuda.Stream()
    xs = [random_tensor(n, 4, d, seed=n) for n, d in ((300000, 0.2), (1000, 1.0), (700001, 0.6), (33, 0.5))]
    caps = [zvc.zvc_max_compressed_bytes(x.numel(), 4) for x in xs]
    stages = [torch.zeros(c, dtype=torch.uint8, device=DEV) for c in caps]
    hosts = [torch.zeros(c, dtype=torch.uint8, pin_memory=True) for c in caps]
    h_bytes = torch.zeros(1, dtype=torch.int64, pin_memory=True)
    ws = zvc.new_workspace(700001, 4, DEV)
    busy = torch.randn(4096, 4096, device=DEV)
    torch.cuda.synchronize()
    say("copies that wait")
    with torch.cuda.stream(copy):
        for _ in range(20):
            busy = busy @ busy * 1e-3
    sizes = [zvc.zvc_offload(x, s, h, h_bytes, ws, compute, copy) for x, s, h in zip(xs, stages, hosts)]
    copy.synchronize()
    for x, h, size in zip(xs, hosts, sizes):
        expect = oracle.compress_stream(raw_bytes(x), 4)
        assert size == expect.size and np.array_equal(h[:size].numpy(), expect)


def test_memory_that_is_pinned_but_not_coherent(oracle):
    """hipHostMalloc with hipHostMallocNonCoherent: the size and the stream are the host's to read once the
    call and the copy stream are done, the stream is the GPU's to read as the host left it; one buffer for
    several tensors, whose lines a cache may still hold from the one before."""
    hip = ctypes.CDLL("libamdhip64.so")
    cap = zvc.zvc_max_compressed_bytes(400000, 4)
    room = ctypes.c_void_p()
    assert hip.hipHostMalloc(ctypes.byref(room), ctypes.c_size_t(cap + 64), ctypes.c_uint(0x80000000)) == 0
    try:
        both = torch.frombuffer((ctypes.c_uint8 * (cap + 64)).from_address(room.value), dtype=torch.uint8)
        h_bytes, host = both[:8].view(torch.int64), both[64:]
        compute, copy = torch.cuda.Stream(), torch.cuda.Stream()
        ws = zvc.new_workspace(400000, 4, DEV)
        stage = zvc.new_compressed_buffer(400000, 4, DEV)
        for n, density in ((400000, 0.3), (400000, 0.9), (70001, 0.5), (399999, 0.1)):
            x = random_tensor(n, 4, density, seed=n + 1).to(DEV)
            expect = oracle.compress_stream(raw_bytes(x), 4)
            say("not coherent n=%d stream bytes %d" % (n, expect.size))
            h_bytes[0] = 0                            # (a size that was not seen is at worst an empty stream)
            torch.cuda.synchronize()
            nbytes = zvc.zvc_offload(x, stage, host, h_bytes, ws, compute, copy)
            copy.synchronize()
            assert nbytes == expect.size and np.array_equal(host[:nbytes].numpy(), expect)
            # what the host writes there comes back: the same tensor with its first word changed
            first = int(np.flatnonzero(raw_bytes(x).view(np.uint32))[0])
            host[4 * -(-n // 32):4 * -(-n // 32) + 4] = torch.tensor([1, 2, 3, 4], dtype=torch.uint8)
            out = torch.zeros_like(x)
            torch.cuda.synchronize()
            zvc.zvc_prefetch(host, nbytes, stage, out, ws, copy, compute)
            compute.synchronize()
            want = raw_bytes(x).copy().view(np.uint32)
            want[first] = 0x04030201
            assert np.array_equal(raw_bytes(out).view(np.uint32), want)
    finally:
        torch.cuda.synchronize()
        assert hip.hipHostFree(room) == 0
