"""Both sides of every size at which the decoder changes (workgroups that count the masks before their own, the
scan in workgroups of 4 and 8 waves, two launches), and sizes around a wave's and a workgroup's part in each,
at 16-byte boundaries and at an odd element; streams whose masks are only 4-byte aligned."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.decoder_routes import elements
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor
from tests.test_gpu_unaligned import assert_guard, guarded

pytestmark = pytest.mark.gpu
DEV = "cuda"
KB, MB = 1 << 10, 1 << 20


def limits(w):
    return [m * 8 for m in (48 * KB, 80 * KB)] + [k // w for k in (9 * MB // 2, 8 * MB, 16 * MB, 32 * MB, 44 * MB, 56 * MB, 76 * MB)]


@pytest.mark.parametrize("w", [4, 2])
def test_both_sides_of_every_limit(oracle, w):
    wave = 4096 // w
    for k, limit in enumerate(limits(w)):
        for j, n in enumerate((limit - 4 * wave - 1, limit - 1, limit, limit + 1, limit + 33, limit + 8 * wave + 31)):
            x = random_tensor(n, w, (0.4, 0.05, 1.0)[(j + k) % 3], seed=n)
            host = raw_bytes(x)
            stream = oracle.compress_stream(host, w)
            room = torch.zeros(stream.size + 16, dtype=torch.uint8, device=DEV)
            comp = room[4 * (j % 3):4 * (j % 3) + stream.size]
            comp.copy_(torch.from_numpy(stream))
            offset = (0, 1, 16 // w, 5)[j % 4]
            base, out = guarded(n, x.dtype, offset)
            say("w=%d n=%d offset %d" % (w, n, offset))
            zvc.zvc_decompress(comp, stream.size, out, zvc.new_workspace(n, w, DEV))
            torch.cuda.synchronize()
            assert np.array_equal(raw_bytes(out), host), "n=%d" % n
            assert_guard(base, n, offset, "n=%d" % n)


@pytest.mark.parametrize("w", [4, 2])
def test_small_streams_that_end_early(oracle, w):
    """What the masks ask for past the stream's end decodes as zero."""
    for n, cut in ((1000, 3), (4096 // w * 5 + 7, 900), (48 * KB * 8 + 100, 20000), (75 * KB * 8, 100000)):
        x = random_tensor(n, w, 0.5, seed=n)
        expect = raw_bytes(x).copy().view(np.uint32 if w == 4 else np.uint16)
        stream = oracle.compress_stream(raw_bytes(x), w)
        expect[np.flatnonzero(expect)[-cut:]] = 0
        out = torch.empty_like(x)
        say("w=%d n=%d cut %d" % (w, n, cut))
        zvc.zvc_decompress(torch.from_numpy(stream).to(DEV), stream.size - cut * w, out, zvc.new_workspace(n, w, DEV))
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), expect.view(np.uint8)), "n=%d" % n


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("route", ["scan4", "scan8", "scan4 large"])
@pytest.mark.parametrize("w", [4, 2])
def test_dense_streams(oracle, w, route, first):
    """The kernels that read the stored elements with the streaming hint: three quarters of them stored, and all."""
    for size, density in ((elements(route, w), 0.77), (elements(route, w) + (2 * MB // w if route == "scan4" else 77), 1.0)):
        x = random_tensor(size, w, density, seed=size)
        host = raw_bytes(x)
        stream = oracle.compress_stream(host, w)
        base, out = guarded(size, x.dtype, first)
        say("w=%d n=%d density %g" % (w, size, density))
        zvc.zvc_decompress(torch.from_numpy(stream).to(DEV), stream.size, out, zvc.new_workspace(size, w, DEV))
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), host), "n=%d" % size
        assert_guard(base, size, first, "n=%d" % size)
