"""The scan's words in the workspace stay from one call to the next and are told apart by the calls' tags:
calls of many sizes, in every mode, one after the other on one workspace, each against the oracle.  The
numbers of tiles (16 and 32 KB) lie on both sides of a pair of counts, of a load of the wave and of a block,
and every number follows a larger and a smaller one; with the default patience and with none."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import assert_parity, raw_bytes, say
from tests.test_gpu_parity import random_tensor

pytestmark = pytest.mark.gpu
DEV = "cuda"
TILES = (1, 512, 2, 513, 127, 1, 1025, 130, 3, 511, 1024, 128, 129, 514)


def elements(tiles, w, windowed):
    """A tensor of that many tiles, the last one ragged (32 KB tiles from the sizes that take them)."""
    small = (38 if windowed else 14) << 20 if w == 4 else (120 if windowed else 48) << 20
    tile = 16384 if tiles * 16384 <= small else 32768
    return tiles * tile // w - 77 if tile == 16384 or (tiles - 1) * tile >= small else None


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("patience", [None, 0])
def test_calls_of_many_sizes_on_one_workspace(oracle, w, patience):
    ws = zvc.new_workspace(1025 * 32768 // w, w, DEV)
    if patience is not None:
        zvc.zvc_workspace_set_lookback_patience(ws, patience)
    for k, tiles in enumerate(TILES):
        for windowed in (False, True):
            n = elements(tiles, w, windowed)
            if n is None:
                continue
            x = random_tensor(n, w, (0.3, 0.0, 1.0, 0.6)[k % 4], seed=n + k)
            if not windowed:
                assert_parity(x, oracle, "%d tiles" % tiles, ws)      # decodes as well, up to 1024 tiles in one launch
                continue
            say("%d tiles windowed n=%d w=%d" % (tiles, n, w))
            stream, table = oracle.window_compress(raw_bytes(x), w, 4096 // w)
            out, size = zvc.new_compressed_buffer(n, w, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
            offsets = torch.zeros(len(table), dtype=torch.int64, device=DEV)
            zvc.zvc_window_compress(x, out, offsets, size, ws)
            assert int(size.item()) == stream.size and np.array_equal(out[:stream.size].cpu().numpy(), stream)
            assert np.array_equal(offsets.cpu().numpy().astype(np.uint64), table)


@pytest.mark.parametrize("w", [4, 2])
def test_calls_that_name_a_part_of_the_workspace(oracle, w):
    """A call may be told of no more of the workspace than it needs: the words of larger calls lie past that part."""
    large, small = 300 * 16384 // w - 5, 7 * 16384 // w + 3
    ws = zvc.new_workspace(large, w, DEV)
    part = ws[:zvc.zvc_workspace_bytes(small, w)]
    for k, n in enumerate((large, small, large, small, small, large, large)):
        assert_parity(random_tensor(n, w, 0.4, seed=n + k), oracle, "call %d" % k, part if n == small else ws)
