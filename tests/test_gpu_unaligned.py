"""Outputs and inputs that begin at any element of a larger buffer: every offset
modulo 16 bytes, sizes at the edges of a lane's 16 bytes, a wave's 4 KB and a
workgroup's 16 KB, and one size that takes the scan, one that takes two launches.  Bit exact
against the oracle; the bytes around the output keep their values."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.decoder_routes import elements
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"
GUARD = 64
TILE_BYTES = 64 << 10      # the largest tile: no load of an encoder reaches further past the tensor's end


def guarded(n, dtype, offset):
    """A buffer of n + offset + GUARD elements filled with 0x5A bytes and the view that begins at `offset`."""
    base = torch.empty(offset + n + GUARD, dtype=dtype, device=DEV)
    base.view(torch.uint8).fill_(0x5A)
    return base, base[offset:offset + n]


def assert_guard(base, n, offset, label):
    w = base.element_size()
    image = raw_bytes(base)
    assert (image[:offset * w] == 0x5A).all() and (image[(offset + n) * w:] == 0x5A).all(), label


def sizes(w):
    lane, wave = 16 // w, 4096 // w
    return [1, lane - 1, lane, lane + 1, wave - 1, wave, wave + 1, 4 * wave - 1, 4 * wave + 1, 9 * wave + 3 * lane + 1]


@pytest.mark.parametrize("w,offset", [(4, k) for k in (1, 2, 3)] + [(2, k) for k in range(1, 8)])
def test_decoders_at_every_output_offset(oracle, w, offset):
    for n in sizes(w) + [elements("scan8", w) + 2, elements("two", w, offset) + 2]:
        x = random_tensor(n, w, 0.45, seed=n + offset)
        host = raw_bytes(x)
        ws = zvc.new_workspace(n, w, DEV)
        comp = torch.from_numpy(np.ascontiguousarray(oracle.compress_stream(host, w))).to(DEV)
        say("unaligned decode n=%d w=%d offset=%d" % (n, w, offset))
        base, out = guarded(n, x.dtype, offset)
        zvc.zvc_decompress(comp, comp.numel(), out, ws)
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), host), "planar n=%d" % n
        assert_guard(base, n, offset, "planar n=%d" % n)
        for window in (1024, 4096, 65536):
            stream, table = oracle.window_compress(host, w, window // w)
            d_stream = torch.from_numpy(np.ascontiguousarray(stream)).to(DEV)
            d_table = torch.from_numpy(table.astype(np.int64)).to(DEV)
            base, out = guarded(n, x.dtype, offset)
            zvc.zvc_window_decompress(d_stream, d_stream.numel(), d_table, n, 0, len(table) - 1, out,
                                      window_bytes=window)
            torch.cuda.synchronize()
            assert np.array_equal(raw_bytes(out), host), "window %d n=%d" % (window, n)
            assert_guard(base, n, offset, "window %d n=%d" % (window, n))


def encoder_sizes(w):
    """Edges of a chunk, a wave's and a workgroup's part of the smallest tile, and a ragged size in each
    of the larger tiles' ranges (whose last wave holds 1 element, or all but 1)."""
    chunk, wave, tile = 256 // w, 4096 // w, 16384 // w
    small = [1, chunk - 1, chunk, chunk + 1, wave - 1, wave, wave + 1, tile - 1, tile, tile + 1, 3 * tile + wave + 3]
    return small + ([(25 << 20) // 4 + 1, (41 << 20) // 4 - 1, (160 << 20) // 4 + 1] if w == 4 else
                    [(65 << 20) // 2 + 1, (65 << 20) // 2 - 1])


@pytest.mark.parametrize("w,offset", [(4, 0), (4, 1), (2, 0), (2, 1), (2, 2)])
def test_encoders_at_every_tile_edge(oracle, w, offset):
    """The tensor's neighbours in its buffer are not zero, up to a whole tile past its end: what lies
    there, and before its beginning, must not count."""
    for n in encoder_sizes(w):
        dense = random_tensor(n + offset + TILE_BYTES // w, w, 1.0, seed=n + offset)
        inner = random_tensor(n, w, 0.4, seed=n + offset + 1)
        dense[offset:offset + n] = inner
        x = dense[offset:offset + n]
        host = raw_bytes(inner)
        say("encode n=%d w=%d offset=%d" % (n, w, offset))
        expect = oracle.compress_stream(host, w)
        ws = zvc.new_workspace(n, w, DEV)
        out = torch.zeros(zvc.zvc_max_compressed_bytes(n, w) + GUARD, dtype=torch.uint8, device=DEV)
        size = torch.zeros(1, dtype=torch.int64, device=DEV)
        zvc.zvc_compress(x, out, size, ws)
        got = out.cpu().numpy()
        assert int(size.item()) == expect.size and np.array_equal(got[:expect.size], expect), "planar n=%d" % n
        assert not got[expect.size:].any(), "planar n=%d: written past the stream" % n
        zvc.zvc_compressed_size(x, size.zero_(), ws)
        assert int(size.item()) == expect.size, "size n=%d" % n
        stream, table = oracle.window_compress(host, w, 4096 // w)
        d_table = torch.zeros(len(table), dtype=torch.int64, device=DEV)
        zvc.zvc_window_compress(x, out, d_table, size, ws)
        assert np.array_equal(out[:len(stream)].cpu().numpy(), stream), "windowed n=%d" % n
        assert d_table.cpu().numpy().astype(np.uint64).tolist() == table.tolist(), "windowed n=%d" % n
