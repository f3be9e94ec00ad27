"""Where the tensor can end inside a tile of the windowed encoder: in, before and behind a group, a chunk, a
1 KB unit, a step and a wave's part, in both tile sizes.  Room for masks is left for whole chunks and given
back, so the stream, its size and the table are compared with the oracle's, and nothing is written behind."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"
ENDS = (0, 256, 1024, 2048, 4096, 8192)        # bytes: tile, chunk, unit, step, a wave's 16 chunks, its 32


@pytest.mark.parametrize("w,tile,floor", [(4, 16384, 0), (2, 16384, 0), (4, 32768, 38 << 20), (2, 32768, 120 << 20)])
def test_tensor_ends_anywhere_in_a_tile(oracle, w, tile, floor):
    for k, end in enumerate(ENDS):
        for j, more in enumerate((-33, -1, 1, 31, 32, 64)):
            if floor and (k + j) % 3:
                continue
            n = (floor + 2 * tile + end) // w + more
            x = random_tensor(n, w, (0.4, 1.0, 0.03)[(k + j) % 3], seed=n)
            say("w=%d n=%d" % (w, n))
            stream, table = oracle.window_compress(raw_bytes(x), w, 1024 // w)
            out = torch.full((zvc.zvc_max_compressed_bytes(n, w) + 64,), 0xCD, dtype=torch.uint8, device=DEV)
            offsets = torch.zeros(len(table), dtype=torch.int64, device=DEV)
            size = torch.zeros(1, dtype=torch.int64, device=DEV)
            zvc.zvc_window_compress(x, out, offsets, size, zvc.new_workspace(n, w, DEV), window_bytes=1024)
            got = out.cpu().numpy()
            assert int(size.item()) == stream.size
            assert np.array_equal(got[:stream.size], stream) and (got[stream.size:] == 0xCD).all()
            assert np.array_equal(offsets.cpu().numpy().astype(np.uint64), table)
