"""The decoder's staging and expansion at its edges: streams that end anywhere among a wave's
16-byte chunks and 1 KB loads, value areas at every offset modulo 16 bytes, tensors that end at
every element of a lane's 16 bytes.  All decoders, against numpy: what is not there is zero."""
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


@pytest.mark.parametrize("route", ["direct4", "scan8", "two"])
@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("density", [0.1, 0.6, 1.0])
def test_streams_cut_short_at_every_edge(oracle, w, density, route):
    n = elements(route, w)
    x = random_tensor(n, w, density, seed=n + w)
    host = raw_bytes(x).view({2: np.uint16, 4: np.uint32}[w])
    stream = np.ascontiguousarray(oracle.compress_stream(raw_bytes(x), w))
    G = (n + 31) // 32
    stored = (stream.size - 4 * G) // w
    rank = np.cumsum(host != 0)                       # an element is there if its rank is at most `kept`
    chunk, load = 16 // w, 1024 // w
    edges = {0, 1, chunk - 1, chunk, chunk + 1, load - 1, load, load + 1, 2 * load + 1, 3 * load - 1, 4 * load,
             4 * load + 1, stored - 1, stored, stored - load, stored // 2}
    ws = zvc.new_workspace(n, w, DEV)
    room = torch.empty(stream.size + 32, dtype=torch.uint8, device=DEV)
    for k, kept in enumerate(sorted(e for e in edges if 0 <= e <= stored)):
        offset = 4 * (k % 4)                          # of the compressed buffer, in bytes
        comp = room[offset:offset + stream.size]
        comp.copy_(torch.from_numpy(stream))
        say("cut n=%d w=%d d=%.1f kept=%d of %d offset=%d" % (n, w, density, kept, stored, offset))
        base, out = guarded(n, x.dtype, 0)
        zvc.zvc_decompress(comp, 4 * G + w * kept + k % w, out, ws)        # (a part of an element is none)
        torch.cuda.synchronize()
        want = np.where(rank <= kept, host, 0).astype(host.dtype)
        assert np.array_equal(raw_bytes(out), want.view(np.uint8)), "kept=%d" % kept
        assert_guard(base, n, 0, "kept=%d" % kept)


@pytest.mark.parametrize("w", [4, 2])
def test_tensors_that_end_anywhere_in_a_step(oracle, w):
    step, lane = 4096 // w, 16 // w
    for extra in list(range(1, 2 * lane + 1)) + [step // 4 - 1, step // 4, step // 4 + 1, step - lane - 1, step - 1, step]:
        n = 4 * step + extra
        x = random_tensor(n, w, 0.5, seed=n)
        comp = torch.from_numpy(np.ascontiguousarray(oracle.compress_stream(raw_bytes(x), w))).to(DEV)
        ws = zvc.new_workspace(n, w, DEV)
        say("end n=%d w=%d" % (n, w))
        base, out = guarded(n, x.dtype, 0)
        zvc.zvc_decompress(comp, comp.numel(), out, ws)
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), raw_bytes(x)), "n=%d" % n
        assert_guard(base, n, 0, "n=%d" % n)
