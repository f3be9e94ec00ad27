"""The count-only pass reads whole 16-byte chunks around a tensor that begins or ends inside one: what lies
before and after it in memory is non-zero and must not count.  Every first element of a chunk; sizes around a
chunk, a group and a workgroup's 32 KB."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("w", [4, 2])
def test_neighbours_in_memory_are_not_counted(w):
    dtype, per, tile = (torch.int32 if w == 4 else torch.int16), 16 // w, 32768 // w
    rng = np.random.default_rng(w)
    ws = zvc.new_workspace(3 * tile, w, DEV)
    size = torch.zeros(1, dtype=torch.int64, device=DEV)
    for first in range(per):
        for n in {1, 2, per - first, per, per + 1, 32, 33, tile - first - 1, tile - first, tile - first + 1, tile, 2 * tile + 5}:
            say("first=%d n=%d w=%d" % (first, n, w))
            host = rng.integers(0, 3, n).astype(np.int32 if w == 4 else np.int16)
            room = torch.full((4 * per + n,), -1, dtype=dtype, device=DEV)
            x = room[per + first:per + first + n]
            assert x.data_ptr() % 16 == first * w
            x.copy_(torch.from_numpy(host))
            zvc.zvc_compressed_size(x, size, ws)
            assert size.item() == 4 * -(-n // 32) + w * int(np.count_nonzero(host))
