"""Outputs that begin anywhere in a 128-byte line: from 8 MB on the decoder's pieces then begin at the first line, in the
middle of a mask, and the first wave writes what lies before; smaller ones are written as they lie.  Every offset; sizes around
the shift, a mask, a wave's piece, a workgroup, and (two launches) around a chunk of the pre-pass; streams that end early."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor
from tests.test_gpu_unaligned import assert_guard, guarded

pytestmark = pytest.mark.gpu
DEV = "cuda"
LINE, PIECE = 128, 4096


MB = 1 << 20
CHUNK = 131072                                   # elements of a chunk of the pre-pass


def every_offset(w):
    """(elements, first element, density) of outputs in whole lines, at every offset that is written so: one launch where
    the output is not 16-byte aligned, two where it is not 64-byte aligned (128 in the largest outputs of 32 bits)."""
    line, step = LINE // w, 16 // w
    one, two = 8 * MB // w + 77, 45 * MB // w + 77
    return ([(one, first, 0.5) for first in range(line) if first % step] +
            [(two, first, 0.5) for first in range(0, line, step) if first * w % 64] +
            [(257 * MB // w + 5, 64 // w, 0.1)] * (w == 4))


def chunk_edges(w):
    """Two launches, a shift of one element, of almost a line and on both sides of a mask."""
    line, chunks = LINE // w, 57 * MB // w // CHUNK + 1
    return [(chunks * CHUNK + more, first, (0.3, 0.7, 0.05)[k % 3])
            for k, first in enumerate((1, line // 2 - 1, line // 2 + 1, line - 1, line - 16 // w))
            for more in ((0, 1) if k % 2 else (-first, line - first))]


def early_ends(w):
    """(elements, first element, stored elements that are missing): as it lies, one launch with 4 waves and 8, two launches."""
    return [(5000, 3, 1), (5000, 3, 700), (PIECE // w + 20, 1, 5), (40, 1, 12), (9 * MB // w, 5, 1000), (36 * MB // w + 9, 7, 3000),
            (57 * MB // w + 3, 1, 1), (57 * MB // w + 3, 5, 5000), (57 * MB // w + 3, LINE // w - 3, 3 * MB // w)]


def decode(x, oracle, offset, label, cut=0, stream=None):
    n, w = x.numel(), x.element_size()
    host = raw_bytes(x)
    if stream is None:
        stream = oracle.compress_stream(host, w)
    comp = torch.from_numpy(stream).to(DEV)
    base, out = guarded(n, x.dtype, offset)
    say("%s n=%d w=%d offset %d cut %d" % (label, n, w, offset, cut))
    zvc.zvc_decompress(comp, stream.size - cut * w, out, zvc.new_workspace(n, w, DEV))
    torch.cuda.synchronize()
    expect = host
    if cut:                                   # the last `cut` stored elements decode as zero
        expect = host.copy().view(np.uint32 if w == 4 else np.uint16)
        expect[np.flatnonzero(expect)[-cut:]] = 0
        expect = expect.view(np.uint8)
    assert np.array_equal(raw_bytes(out), expect), label
    assert_guard(base, n, offset, label)


@pytest.mark.parametrize("w", [4, 2])
def test_every_offset(oracle, w):
    per, line = PIECE // w, LINE // w
    for offset in range(line):
        shift = -offset % line
        sizes = {1, shift, shift + 1, 33, per, per + shift, 4 * per + shift + 1, 9 * per + (offset * 37) % per}
        for k, n in enumerate(sorted(sizes - {0})):
            x = random_tensor(n, w, (0.4, 1.0, 0.05)[(offset + k) % 3], seed=n + offset)
            decode(x, oracle, offset, "shift %d" % shift)


@pytest.mark.parametrize("w", [4, 2])
def test_every_offset_in_whole_lines(oracle, w):
    made = {}
    for n, first, density in every_offset(w):
        if n not in made:
            x = random_tensor(n, w, density, seed=n)
            made = {n: (x, oracle.compress_stream(raw_bytes(x), w))}
        decode(made[n][0], oracle, first, "whole lines", stream=made[n][1])


@pytest.mark.parametrize("w", [4, 2])
def test_chunk_edges(oracle, w):
    for n, first, density in chunk_edges(w):
        decode(random_tensor(n, w, density, seed=n + first), oracle, first, "chunk edge")


@pytest.mark.parametrize("w", [4, 2])
def test_many_chunks_and_both_orders(oracle, w):
    """More chunks than the workgroups add up themselves, and the interleaved order."""
    for n, density, offset in ((1025 * CHUNK + 5, 0.04, 3), ((77 << 20) // w + 1, 0.04, 5), ((77 << 20) // w + 1, 0.5, 7),
                               ((77 << 20) // w + 1, 0.9, LINE // w - 5)):
        decode(random_tensor(n, w, density, seed=n), oracle, offset, "large")


@pytest.mark.parametrize("w", [4, 2])
def test_streams_that_end_early(oracle, w):
    for n, offset, cut in early_ends(w):
        decode(random_tensor(n, w, 0.6, seed=n), oracle, offset, "early end", cut)
