"""The window decoder's walk over masks: streams that end early, window sizes and
numbers of windows on both sides of where the kernels change, the extremes of
density (a group of one word, a group of 33), against a walk written out in numpy."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"


def walk(stream, table, n, w, per, end):
    """What the decoder gives for the first `end` bytes of a stream: a mask that is not wholly there is
    empty, an element that is not wholly there is zero."""
    out = np.zeros(n, dtype={2: np.uint16, 4: np.uint32}[w])
    for k in range(len(table) - 1):
        p, hi = min(int(table[k]), end), min(int(table[k + 1]), end)
        for g in range(k * per // 32, -(-min(n, (k + 1) * per) // 32)):
            if p + 4 > hi:
                break
            mask = int(stream[p:p + 4].view("<u4")[0])
            p += 4
            for b in range(32):
                if mask >> b & 1:
                    if p + w <= hi:
                        out[32 * g + b] = stream[p:p + w].view(out.dtype)[0]
                    p += w
    return out


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("window", [1024, 2048, 4096, 8192, 65536])
def test_streams_that_end_early(oracle, window, w):
    per = window // w
    n = 2 * per + per // 3 + 7
    for density in (0.03, 0.5, 1.0):
        x = random_tensor(n, w, density, seed=window + w)
        stream, table = oracle.window_compress(raw_bytes(x), w, per)
        stream = np.ascontiguousarray(stream)
        d_stream = torch.from_numpy(stream).to(DEV)
        d_table = torch.from_numpy(table.astype(np.int64)).to(DEV)
        total = int(table[-1])
        for end in {total, total - w, total // 2 // w * w, total // 5 // w * w + w, 8, 4, 0}:
            say("early end window=%d w=%d d=%.2f end=%d of %d" % (window, w, density, end, total))
            out = torch.empty(n, dtype=x.dtype, device=DEV)
            out.view(torch.uint8).fill_(0xEE)
            zvc.zvc_window_decompress(d_stream, end, d_table, n, 0, len(table) - 1, out, window_bytes=window)
            torch.cuda.synchronize()
            want = walk(stream, table, n, w, per, end)
            assert np.array_equal(raw_bytes(out), want.view(np.uint8)), "end=%d" % end
