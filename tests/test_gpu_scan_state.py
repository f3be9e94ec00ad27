"""The scan's words in the workspace stay from one call to the next and are told apart by the calls' numbers:
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
            windowed_parity(x, oracle, ws, "%d tiles" % tiles)


def windowed_parity(x, oracle, ws, label, expect=None):
    n, w = x.numel(), x.element_size()
    say("%s windowed n=%d w=%d" % (label, n, w))
    stream, table = expect or oracle.window_compress(raw_bytes(x), w, 4096 // w)
    out, size = zvc.new_compressed_buffer(n, w, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    offsets = torch.zeros(len(table), dtype=torch.int64, device=DEV)
    zvc.zvc_window_compress(x, out, offsets, size, ws)
    assert int(size.item()) == stream.size and np.array_equal(out[:stream.size].cpu().numpy(), stream), label
    assert np.array_equal(offsets.cpu().numpy().astype(np.uint64), table), label


@pytest.mark.parametrize("w,large_mb,small_mb", [(4, 37, 0.1), (2, 37, 0.1), (4, 37, 3), (2, 37, 2), (4, 200, 10), (4, 500, 46)])
def test_calls_that_name_a_part_of_the_workspace(oracle, w, large_mb, small_mb):
    """A call may be told of no more of the workspace than it needs (the decoder of these sizes: every workgroup by
    itself, a scan of 4 or 8 waves, two launches).  It touches nothing behind that part, where words of larger calls lie,
    and what it leaves inside does not disturb them."""
    large, small = int(large_mb * (1 << 20)) // w - 5, int(small_mb * (1 << 20)) // w + 3
    big, little = random_tensor(large, w, 0.4, seed=large), random_tensor(small, w, 0.999, seed=small)
    expect = oracle.window_compress(raw_bytes(big), w, 4096 // w)
    ws = zvc.new_workspace(large, w, DEV)
    part = zvc.zvc_workspace_bytes(small, w)
    for k in range(3):
        windowed_parity(big, oracle, ws, "large %d" % k, expect)
        behind = ws[part:].clone()
        assert behind.any()
        assert_parity(little, oracle, "named part %d" % k, ws[:part])
        if k == 1:
            windowed_parity(little, oracle, ws[:part], "named part %d" % k)
        torch.cuda.synchronize()
        assert torch.equal(ws[part:], behind)


def header(ws):
    """The words that the scan keeps about the calls so far (number, prefixes, limit), and the wide calls' number."""
    return ws[:48].view(torch.int64)


@pytest.mark.parametrize("patience", [None, 0])
@pytest.mark.parametrize("w", [4, 2])
def test_wide_counts(oracle, w, patience):
    """Calls that may meet counts with their own number from before: here all words have it.  Such a call
    takes counts of 64 bits.  Tiles on both sides of a load of the wave and of a block, every scan decoder."""
    mb = 1 << 20
    sizes = [k * 16384 // w - 7 for k in (2, 3, 64, 65, 129, 511, 513, 600)] + [k * mb // w + 5 for k in (3, 9, 15, 33)]
    ws = zvc.new_workspace(max(sizes), w, DEV)
    if patience is not None:
        zvc.zvc_workspace_set_lookback_patience(ws, patience)
    calls = 0

    def old_counts():
        state = header(ws)[1].item() & 0xFFFFFFFF       # number and prefixes as they are, a limit of one tile
        header(ws)[1] = 1 << 32 | state
        counts = ws[8576:]                              # behind the header
        word = 1 << 31 | (state & 0x7FFF) << 16 | 1 << 15 | 77
        counts[:counts.numel() // 4 * 4].view(torch.int32).fill_(word - (1 << 32))

    for k, n in enumerate(sizes):
        x = random_tensor(n, w, (0.3, 1.0, 0.6)[k % 3], seed=n)
        host = raw_bytes(x)
        expect = oracle.compress_stream(host, w)
        comp, size, out = zvc.new_compressed_buffer(n, w, DEV), torch.zeros(1, dtype=torch.int64, device=DEV), torch.empty_like(x)
        say("wide n=%d w=%d patience %s" % (n, w, patience))
        old_counts()
        zvc.zvc_compress(x, comp, size, ws)
        assert int(size.item()) == expect.size and np.array_equal(comp[:expect.size].cpu().numpy(), expect)
        old_counts()
        zvc.zvc_decompress(comp, expect.size, out, ws)
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), host)
        calls += 1 + (n > 655360)                       # (up to 80 KB of masks decode without a scan)
        assert header(ws)[5].item() == calls
        old_counts()
        windowed_parity(x, oracle, ws, "wide")
        calls += 1
        assert header(ws)[5].item() == calls
    assert patience is None or zvc.zvc_workspace_self_help_count(ws) > 0


def test_more_calls_than_a_count_tells_apart(oracle):
    """2^15 small calls between two large ones: the second has the first one's number in 15 bits."""
    w, large = 4, 300 * 16384 // 4
    ws = zvc.new_workspace(large, w, DEV)
    x, y = random_tensor(large, w, 0.4, seed=1), random_tensor(large, w, 0.7, seed=2)
    small = random_tensor(5000, w, 0.5, seed=3)
    comp, size = zvc.new_compressed_buffer(large, w, DEV), torch.zeros(1, dtype=torch.int64, device=DEV)
    for gap in (0, (1 << 15) - 1, (1 << 15) - 1):
        say("%d small calls" % gap)
        for _ in range(gap):
            zvc.zvc_compress(small, comp, size, ws)
        x, y = y, x
        expect = oracle.compress_stream(raw_bytes(x), w)
        zvc.zvc_compress(x, comp, size, ws)
        assert int(size.item()) == expect.size and np.array_equal(comp[:expect.size].cpu().numpy(), expect)
    assert header(ws)[5].item() > 0
