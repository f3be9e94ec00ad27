"""The decoders on both sides of the sizes and densities at which the order of the workgroups changes:
planar outputs around 64 and 400 MB, windows of 1, 2 and 4 KB around 150, 250, 400 and 600 MB, 32- and 16-bit
elements, outputs on a 16-byte boundary and not.  The decoded tensor is the one that was compressed
(whose stream other tests compare with the oracle's), and nothing beside it is written."""
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda"
MB = 1 << 20
GUARD = 64


def tensor(n, w, density, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randint(1, 2 ** (8 * w - 1), (n,), generator=g, device=DEV, dtype=torch.int32)
    x *= torch.rand(n, generator=g, device=DEV) < density
    return x if w == 4 else x.to(torch.int16)


def room(n, w, offset):
    base = torch.empty(offset + n + GUARD, dtype={4: torch.int32, 2: torch.int16}[w], device=DEV)
    base.view(torch.uint8).fill_(0x5A)
    return base, base[offset:offset + n]


def check(base, out, x, offset):
    assert torch.equal(out, x)
    rest = torch.cat([base[:offset], base[offset + x.numel():]]).view(torch.uint8)
    assert bool((rest == 0x5A).all())


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("limit", [64 * MB, 400 * MB])
@pytest.mark.parametrize("density", [0.04, 0.2, 0.6])
def test_planar(w, limit, density):
    for n, offset in ((limit // w - 1, 0), (limit // w, 3), (limit // w + 1, 0), (limit // w + 70001, 1)):
        x = tensor(n, w, density, seed=n + w)
        ws = zvc.new_workspace(n, w, DEV)
        comp = zvc.new_compressed_buffer(n, w, DEV)
        size = torch.zeros(1, dtype=torch.int64, device=DEV)
        zvc.zvc_compress(x, comp, size, ws)
        base, out = room(n, w, offset)
        say("planar n=%d w=%d density=%.2f offset=%d" % (n, w, density, offset))
        zvc.zvc_decompress(comp, int(size.item()), out, ws)
        check(base, out, x, offset)


@pytest.mark.parametrize("w,density,limit", [(4, 0.04, 150 * MB), (4, 0.12, 600 * MB), (2, 0.25, 400 * MB),
                                             (4, 0.4, 250 * MB), (2, 0.6, 150 * MB), (2, 0.04, 150 * MB)])
def test_windows(w, density, limit):
    for window in (1024, 2048, 4096):
        per = window // w
        windows = limit // window + 3
        n = windows * per - 37
        x = tensor(n, w, density, seed=window + w)
        ws = zvc.new_workspace(n, w, DEV)
        comp = zvc.new_compressed_buffer(n, w, DEV)
        table = torch.zeros(windows + 1, dtype=torch.int64, device=DEV)
        size = torch.zeros(1, dtype=torch.int64, device=DEV)
        zvc.zvc_window_compress(x, comp, table, size, ws, window_bytes=window)
        for first, count, offset in ((0, windows, 0), (2, windows - 5, 1), (3, windows - 3, 0)):
            lo, hi = first * per, min(n, (first + count) * per)
            base, out = room(hi - lo, w, offset)
            say("windows of %d: %d+%d w=%d density=%.2f offset=%d" % (window, first, count, w, density, offset))
            zvc.zvc_window_decompress(comp, int(size.item()), table, n, first, count, out, window_bytes=window)
            check(base, out, x[lo:hi], offset)
