"""Window decoders where a window, a part of one or a group can end: tails of every kind, windows
that are nothing but masks, streams and outputs at every offset modulo 16 bytes, ranges of one
window.  The oracle's streams, bit for bit, and nothing beside the output."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor
from tests.test_gpu_unaligned import assert_guard, guarded

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("window", [1024, 2048, 4096, 8192, 16384, 32768, 65536])
def test_window_ends(oracle, window, w):
    per = window // w
    tails = [1, 31, 32, 33, per // 2 - 1, per // 2 + 1, per - 32, per - 1, per]
    for k, tail in enumerate(tails):
        n = (1 + 5 * (k % 2)) * per + tail            # few windows, and more than a workgroup's waves take
        density = (0.0, 0.02, 0.5, 1.0)[k % 4]
        x = random_tensor(n, w, density, seed=n + w)
        if k % 3 == 2:
            x[per // 3:per] = 0                       # a window whose bytes are nearly all in its first third
        host = raw_bytes(x)
        stream, table = oracle.window_compress(host, w, per)
        offset, out_offset = k * 7 % (16 // w), k * 5 % (16 // w)         # in elements
        room = torch.zeros(stream.size + 64, dtype=torch.uint8, device=DEV)
        d_stream = room[offset * w:offset * w + stream.size]
        d_stream.copy_(torch.from_numpy(np.ascontiguousarray(stream)))
        d_table = torch.from_numpy(table.astype(np.int64)).to(DEV)
        windows = len(table) - 1
        for first, count in ((0, windows), (windows - 1, 1), (windows // 2, windows - windows // 2)):
            say("window=%d w=%d n=%d d=%.2f windows %d+%d offsets %d %d" % (window, w, n, density, first, count,
                                                                           offset, out_offset))
            lo, hi = first * per, min(n, (first + count) * per)
            base, out = guarded(hi - lo, x.dtype, out_offset)
            zvc.zvc_window_decompress(d_stream, stream.size, d_table, n, first, count, out, window_bytes=window)
            torch.cuda.synchronize()
            assert np.array_equal(raw_bytes(out), host[lo * w:hi * w]), "n=%d windows %d+%d" % (n, first, count)
            assert_guard(base, hi - lo, out_offset, "n=%d windows %d+%d" % (n, first, count))
