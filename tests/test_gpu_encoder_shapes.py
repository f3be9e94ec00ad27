"""Every shape of the encoder's tile, in each mode, against the oracle: tensors on both sides of each size
at which the tile changes, ragged (the last wave holds one element, or all but one), with empty, sparse and
dense stretches of up to several tiles, at a 4-byte boundary and (16-bit elements) at an odd half dword,
with a tile of non-zeros before and behind the tensor."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say

pytestmark = pytest.mark.gpu
DEV = "cuda"
DTYPES = {4: torch.int32, 2: torch.int16}
TILE_BYTES = 64 << 10
MB = 1 << 20
# bytes from which a larger tile is taken: 16 -> 32 KB, 32 -> 64 KB
LIMITS = {("plain", 4): (14 * MB, 160 * MB), ("relu", 4): (14 * MB, 160 * MB), ("windowed", 4): (38 * MB,),
          ("plain", 2): (48 * MB,), ("relu", 2): (48 * MB,), ("windowed", 2): (120 * MB,)}


def stretches(n, w, offset, seed):
    """(buffer, tensor): words of either sign; stretches of 500 to 60,000 elements, empty, all non-zero, or between."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    guard = TILE_BYTES // w
    base = torch.randint(1, 2 ** (8 * w - 1), (guard + offset + n + guard,), generator=g, device=DEV, dtype=torch.int32)
    x = base[guard + offset:guard + offset + n]
    lengths = rng.integers(500, 60000, size=n // 20000 + 100)
    assert lengths.sum() >= n
    density = torch.from_numpy(rng.choice([0.0, 0.02, 0.4, 0.4, 0.9, 1.0], size=lengths.size)).to(DEV, torch.float32)
    keep = torch.repeat_interleave(density, torch.from_numpy(lengths).to(DEV))[:n]
    x *= torch.rand(n, generator=g, device=DEV) < keep
    x *= 1 - 2 * (torch.rand(n, generator=g, device=DEV) < 0.3).to(torch.int32)
    base = base.to(DTYPES[w])
    return base, base[guard + offset:guard + offset + n]


@pytest.mark.parametrize("w,offset", [(4, 0), (2, 0), (2, 1)])
@pytest.mark.parametrize("mode", ["plain", "relu", "windowed"])
def test_both_sides_of_every_tile_limit(oracle, mode, w, offset):
    for limit in LIMITS[mode, w]:
        for n in (limit // w - 1, limit // w + 1, limit // w + 70001):
            base, x = stretches(n, w, offset, seed=n + offset)
            assert x.data_ptr() % 4 == w * offset % 4
            host = raw_bytes(x)
            say("%s n=%d w=%d offset=%d" % (mode, n, w, offset))
            ws = zvc.new_workspace(n, w, DEV)
            out = torch.full((zvc.zvc_max_compressed_bytes(n, w) + 64,), 0xCD, dtype=torch.uint8, device=DEV)
            size = torch.full((1,), -1, dtype=torch.int64, device=DEV)
            if mode == "windowed":
                expect, table = oracle.window_compress(host, w, 4096 // w)
                d_table = torch.zeros(len(table), dtype=torch.int64, device=DEV)
                zvc.zvc_window_compress(x, out, d_table, size, ws)
                assert np.array_equal(d_table.cpu().numpy().astype(np.uint64), table), "n=%d" % n
            elif mode == "relu":
                expect = oracle.relu_compress_stream(host, w)
                zvc.zvc_relu_compress(x, out, size, ws)
            else:
                expect = oracle.compress_stream(host, w)
                zvc.zvc_compress(x, out, size, ws)
            got = out.cpu().numpy()
            assert int(size.item()) == expect.size, "n=%d" % n
            assert np.array_equal(got[:expect.size], expect), "n=%d" % n
            assert (got[expect.size:] == 0xCD).all(), "n=%d: written past the stream" % n
            del base, x, out, ws
