"""The window decoder's walk over masks: streams that end early, window sizes on both
sides of where the kernels change, one window and thousands, the extremes of
density (a group of one word, a group of 33), against a walk written out in numpy."""
import numpy as np
import pytest
import torch

from paper_1705_01626_amd import zvc
from tests.gpu_util import raw_bytes, say
from tests.test_gpu_parity import random_tensor
from tests.test_gpu_unaligned import assert_guard, guarded

pytestmark = pytest.mark.gpu
DEV = "cuda"


def walk(stream, table, n, w, per, end):
    """What the decoder gives for the first `end` bytes of a stream: a mask that is not wholly there is
    empty, an element that is not wholly there is zero.  What is there, is up to the end of the window, or of
    the 4 KB of windows that are decoded together, and no more than those can need; a window that does not
    begin in it has nothing."""
    out = np.zeros(n, dtype={2: np.uint16, 4: np.uint32}[w])
    table = [min(int(o), end) for o in table]
    windows = len(table) - 1
    together = max(1, 4096 // (per * w))
    for k in range(windows):
        first = k // together * together
        lo, hi = table[first], table[min(first + together, windows)]
        hi = min(max(lo, hi), lo + together * per // 32 * (4 + 32 * w))
        p = table[k] if lo <= table[k] <= hi else hi
        for g in range(k * per // 32, -(-min(n, (k + 1) * per) // 32)):
            if p + 4 > hi:
                break
            mask = int(stream[p:p + 4].view("<u4")[0])
            p += 4
            for b in range(32):
                if mask >> b & 1:
                    if p + w <= hi and 32 * g + b < n:
                        out[32 * g + b] = stream[p:p + w].view(out.dtype)[0]
                    p += w
    return out


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("window", [1024, 2048, 4096, 8192, 16384, 32768, 65536])
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
        half, fifth = total // 2 // w * w, total // 5 // w * w
        # whole words, and ends inside an element or a mask
        for end in {total, total - w, half, fifth + w, 8, 4, 0,
                    total - 1, total - 2, total - 3, half + 1, half + 3, fifth + 2, 9, 6, 3}:
            say("early end window=%d w=%d d=%.2f end=%d of %d" % (window, w, density, end, total))
            out = torch.empty(n, dtype=x.dtype, device=DEV)
            out.view(torch.uint8).fill_(0xEE)
            zvc.zvc_window_decompress(d_stream, end, d_table, n, 0, len(table) - 1, out, window_bytes=window)
            torch.cuda.synchronize()
            want = walk(stream, table, n, w, per, end)
            assert np.array_equal(raw_bytes(out), want.view(np.uint8)), "end=%d" % end


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("window", [1024, 2048, 4096, 8192, 16384, 32768, 65536])
def test_damaged_streams_and_tables(oracle, window, w):
    """Random bytes, sparse and dense ones, as the stream, and random numbers as the table (odd ones among
    them, ends before beginnings, beyond the stream): the walk's result, and nothing beside the output."""
    per = window // w
    n = 5 * per + per // 3 + 7
    rng = np.random.default_rng(window + w)
    x = random_tensor(n, w, 0.5, seed=window + w)
    stream, table = oracle.window_compress(raw_bytes(x), w, per)
    total = stream.size
    noise = rng.integers(0, 256, size=total, dtype=np.uint8)
    thin = noise & rng.integers(0, 256, size=total, dtype=np.uint8) & rng.integers(0, 256, size=total, dtype=np.uint8)
    empty = np.where(rng.random(total) < 0.02, noise, 0).astype(np.uint8)
    inside = np.sort(rng.integers(0, total, size=len(table)))
    cases = [(s, table, end) for s in (noise, thin, empty, np.full(total, 255, np.uint8)) for end in (total, total - 5)]
    cases += [(stream, t, total) for t in (inside, inside // 4 * 4, rng.permutation(inside),
                                           rng.integers(0, 1 << 62, size=len(table)))]
    cases += [(noise, inside, total - 1)]
    for k, (s, t, end) in enumerate(cases):
        s, t = np.ascontiguousarray(s), t.astype(np.int64)
        say("damaged window=%d w=%d case %d" % (window, w, k))
        base, out = guarded(n, x.dtype, 0)
        zvc.zvc_window_decompress(torch.from_numpy(s).to(DEV), end, torch.from_numpy(t).to(DEV), n, 0, len(t) - 1, out,
                                  window_bytes=window)
        torch.cuda.synchronize()
        assert np.array_equal(raw_bytes(out), walk(s, t, n, w, per, end).view(np.uint8)), "case %d" % k
        assert_guard(base, n, 0, "case %d" % k)


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("window", [16384, 32768, 65536])
def test_windows_of_mixed_density(oracle, window, w):
    """Dense, empty and middling stretches inside a window: equal shares of its bytes are very unequal
    shares of its groups (one wave's share can be most of the window)."""
    per = window // w
    rng = np.random.default_rng(window + w)
    n = 7 * per + per // 2 + 3
    host = rng.integers(1, 2 ** (8 * w - 1), size=n, dtype=np.int64).astype({2: np.int16, 4: np.int32}[w])
    at, kinds = 0, (0.0, 1.0, 0.0, 0.02, 0.6)
    for k in range(200):
        run = int(rng.integers(per // 20, per))
        host[at:at + run] *= rng.random(len(host[at:at + run])) < kinds[k % len(kinds)]
        at += run
    x = torch.from_numpy(host)
    stream, table = oracle.window_compress(raw_bytes(x), w, per)
    d_stream = torch.from_numpy(np.ascontiguousarray(stream)).to(DEV)
    d_table = torch.from_numpy(table.astype(np.int64)).to(DEV)
    say("mixed density window=%d w=%d" % (window, w))
    out = torch.empty(n, dtype=x.dtype, device=DEV)
    out.view(torch.uint8).fill_(0xEE)
    zvc.zvc_window_decompress(d_stream, d_stream.numel(), d_table, n, 0, len(table) - 1, out, window_bytes=window)
    torch.cuda.synchronize()
    assert np.array_equal(raw_bytes(out), raw_bytes(x))


@pytest.mark.parametrize("window,w,most", [(16384, 4, 2048), (16384, 2, 768), (32768, 2, 1536), (65536, 2, 1792)])
def test_many_windows_and_the_last_alone(window, w, most):
    """Hundreds of large windows, whose workgroups share the CUs, with and without the ragged last one, and
    that one alone: the same elements (which the GPU's own encoder compressed; its streams are compared with
    the oracle's elsewhere)."""
    per = window // w
    n = (most + 1) * per - 37
    g = torch.Generator(device=DEV).manual_seed(window + w)
    x = torch.randint(1, 2 ** (8 * w - 1), (n,), generator=g, device=DEV, dtype=torch.int32)
    x = (x * (torch.rand(n, generator=g, device=DEV) < 0.4)).to({2: torch.int16, 4: torch.int32}[w])
    ws = zvc.new_workspace(n, w, DEV)
    comp = zvc.new_compressed_buffer(n, w, DEV)
    table = torch.zeros(most + 2, dtype=torch.int64, device=DEV)
    size = torch.zeros(1, dtype=torch.int64, device=DEV)
    zvc.zvc_window_compress(x, comp, table, size, ws, window_bytes=window)
    for first, count in ((0, most), (0, most + 1), (most, 1)):
        say("window=%d w=%d windows %d+%d" % (window, w, first, count))
        lo, hi = first * per, min(n, (first + count) * per)
        out = torch.full((hi - lo,), -1, dtype=x.dtype, device=DEV)
        zvc.zvc_window_decompress(comp, int(size.item()), table, n, first, count, out, window_bytes=window)
        assert torch.equal(out, x[lo:hi])
