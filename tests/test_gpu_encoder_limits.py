"""The encoder at the sizes where its kernels change (16 or 32 KB tiles, half of a tile's staging before its
count or all of it), at 10 MB, and its tile's queues filled to the last byte: whole tiles, a word less and a
word more, at densities from nothing to everything, in each mode and at either alignment of 16-bit
elements.  The oracle's streams, and nothing written past them."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_encoder_shapes import stretches
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"
MB = 1 << 20
LIMITS = {("plain", 4): (10 * MB, 14 * MB, 48 * MB), ("relu", 4): (10 * MB, 14 * MB, 48 * MB),
          ("windowed", 4): (10 * MB, 38 * MB),
          ("plain", 2): (10 * MB, 20 * MB, 48 * MB), ("relu", 2): (10 * MB, 20 * MB, 48 * MB),
          ("windowed", 2): (10 * MB, 120 * MB)}


def check(oracle, mode, x, label):
    n, w = x.numel(), x.element_size()
    host = raw_bytes(x)
    say("%s %s n=%d w=%d ptr%%4=%d" % (label, mode, n, w, x.data_ptr() % 4))
    ws = zvc.new_workspace(n, w, DEV)
    out = torch.full((zvc.zvc_max_compressed_bytes(n, w) + 64,), 0xCD, dtype=torch.uint8, device=DEV)
    size = torch.full((1,), -1, dtype=torch.int64, device=DEV)
    if mode == "windowed":
        expect, table = oracle.window_compress(host, w, 4096 // w)
        d_table = torch.zeros(len(table), dtype=torch.int64, device=DEV)
    else:
        expect = (oracle.relu_compress_stream if mode == "relu" else oracle.compress_stream)(host, w)
    for _ in range(2):                                # the second call finds the workspace as the first left it
        if mode == "windowed":
            zvc.zvc_window_compress(x, out, d_table, size, ws)
            assert np.array_equal(d_table.cpu().numpy().astype(np.uint64), table), label
        elif mode == "relu":
            zvc.zvc_relu_compress(x, out, size, ws)
        else:
            zvc.zvc_compress(x, out, size, ws)
        got = out.cpu().numpy()
        assert int(size.item()) == expect.size, label
        assert np.array_equal(got[:expect.size], expect), label
        assert (got[expect.size:] == 0xCD).all(), "%s: written past the stream" % label
    if mode == "plain":
        zvc.zvc_compressed_size(x, size, ws)
        assert int(size.item()) == expect.size, label


@pytest.mark.parametrize("w,offset", [(4, 0), (2, 0), (2, 1)])
@pytest.mark.parametrize("mode", ["plain", "relu", "windowed"])
def test_both_sides_of_every_limit(oracle, mode, w, offset):
    for limit in LIMITS[mode, w]:
        for n in (limit // w - 1, limit // w, limit // w + 1):
            _, x = stretches(n, w, offset, seed=n + offset)
            check(oracle, mode, x, "limit %d MB" % (limit // MB))


@pytest.mark.parametrize("w,offset", [(4, 0), (4, 1), (2, 0), (2, 1)])
@pytest.mark.parametrize("mode", ["plain", "relu", "windowed"])
def test_queues_from_empty_to_full(oracle, mode, w, offset):
    tile = 16384 // w
    for n in (tile, 3 * tile - 1, 3 * tile, 3 * tile + 1, 40 * tile + 33):
        for density in (0.0, 0.5, 0.97, 1.0):
            x = random_tensor(n + offset, w, density, seed=n + w)[offset:]
            if mode == "relu":
                x = x.abs()                           # (dense in the stream as well)
            base = torch.empty(n + offset, dtype=x.dtype, device=DEV)
            base[offset:] = x
            check(oracle, mode, base[offset:], "density %.2f" % density)
