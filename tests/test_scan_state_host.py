"""The arithmetic of the scan's state in the workspace, on the CPU and from the library's own source: which words
pass for a call's counts, over more calls than a count's 15 bits tell apart, which prefixes a call leaves, and that every call's
state lies in the bytes that the workspace's size promises.  Far beyond the sizes that a test can decode."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_1705_01626_amd import build as zvc_build
from paper_1705_01626_amd import zvc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = 458752                                  # tiles from which on a block is longer than 512: 896 prefixes
MOST = 896


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    where = tmp_path_factory.mktemp("scan_state")
    out, fake = str(where / "scan_state.so"), str(where / "fake.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", zvc_build.ROCM_INCLUDE,
                    "-o", fake, os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True)
    subprocess.run([zvc_build.HIPCC, "-x", "hip", "--offload-host-only", "-fuse-cuid=none", "-O1", "-std=c++17", "-fPIC", "-c", "-w",
                    "-I", os.path.join(ROOT, "include"), "-o", out + ".o", os.path.join(ROOT, "tests", "scan_state_host.cpp")], check=True)
    # (there is no device code in it, so the symbol that stands for that has to come from somewhere)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,--defsym=__hip_fatbin=0", "-o", out, out + ".o", fake, "-Wl,-rpath," + str(where),
                    os.path.join(os.path.dirname(zvc_build.ROCM_INCLUDE), "lib", "libamdhip64.so")], check=True)
    lib = ctypes.CDLL(out)
    u64 = ctypes.c_ulonglong
    lib.host_header_bytes.restype = lib.host_scan_bytes.restype = ctypes.c_size_t
    lib.host_scan_bytes.argtypes = [ctypes.c_size_t, ctypes.c_int]
    lib.host_narrow_count.restype = ctypes.c_uint
    lib.host_passes_as.argtypes = lib.host_in_halves.argtypes = lib.host_from_halves.argtypes = [u64]
    lib.host_wide_count.restype = lib.host_in_halves.restype = lib.host_from_halves.restype = u64
    lib.host_wide_count.argtypes = [u64, ctypes.c_uint, ctypes.c_int]
    lib.host_prefix_call.argtypes = [ctypes.c_char_p, ctypes.c_uint]
    return lib


NUMBERS = [0, 1, 2, 3, 255, 32767, 32768, (1 << 31) - 1, 1 << 31, (1 << 32) + 1, (1 << 45) - 1]
KEPT = [(kept, owner) for kept in (0, 1, 0x4000) for owner in (0, 1)]


def test_no_word_passes_for_another_kind(host):
    """Counts of 32 bits in either half of 8 bytes, counts of 64, and what the decoder's pre-pass keeps in the same
    bytes: sums of at most a chunk's 131072 elements, prefixes in halves, zero at first."""
    for kept, owner in KEPT:
        for call in (0, 1, 16383, 16384, 32767):
            narrow = host.host_narrow_count(call, kept, owner)
            assert narrow & 0x7FFF == kept and (narrow >> 16) & 0x7FFF == call
            for word in (narrow, narrow << 32, narrow << 32 | narrow):
                assert host.host_passes_as(word) == 1
        for number in NUMBERS:
            wide = host.host_wide_count(number, kept, owner)
            assert wide & 0x7FFF == kept and host.host_passes_as(wide) == 2
    assert len({host.host_wide_count(number, 0, 0) for number in NUMBERS}) == len(NUMBERS)
    for sums in (0, 1, 131072, 131072 << 32 | 131072):
        assert host.host_passes_as(sums) == 0
    for prefix in (0, 1, (1 << 30) - 1, 1 << 30, (1 << 31) + 5, (1 << 32) - 1, (1 << 45) - 1):
        assert host.host_passes_as(host.host_in_halves(prefix)) == 0
        assert host.host_from_halves(host.host_in_halves(prefix)) == prefix


TERM = 1 << 14


def test_no_call_takes_an_older_count_for_its_own(host):
    """Calls whose numbers are the same in the 15 bits of a count, with smaller ones in between that leave its words
    where they are."""
    def run(tiles, slots=64):
        wide = ctypes.c_int(0)
        assert host.host_calls((ctypes.c_uint * len(tiles))(*tiles), len(tiles), slots, ctypes.byref(wide)) == -1
        return wide.value
    # equal calls, and calls of two sizes in turn, have no need for wide counts but at a term's beginning
    assert run([40] * (5 * TERM)) == 0
    assert run([40, 3] * (5 * TERM // 2)) <= 4 and run([3, 40] * (5 * TERM // 2)) <= 4
    # the same number again after two terms, and everything around it
    for gap in (TERM - 1, TERM, 2 * TERM - 2, 2 * TERM - 1, 2 * TERM, 4 * TERM - 1, 4 * TERM):
        for before in (0, 1, TERM - 1, TERM):
            assert run([1] * before + [60] + [1] * gap + [60] + [2] * gap + [30, 60, 31]) > 0 or gap < TERM
    rng = random.Random(3)
    for _ in range(6):
        tiles = []
        while len(tiles) < 12 * TERM:
            tiles += [rng.choice((1, 2, 5, 17, 33, 64))] * rng.choice((1, 1, 2, 30, TERM // 2, TERM - 1, TERM, 2 * TERM - 1, 2 * TERM))
        run(tiles)


def test_block_length(host):
    sizes = {t + d for t in (1, 511, 512, LIMIT, 2 * LIMIT, 4 * LIMIT, 1024 * LIMIT) for d in (-1, 0, 1, 511, 512, 1023, 1024)}
    for tiles in sorted(sizes | {0x7FFFFFFF}):
        shift = host.host_block_shift(tiles)
        assert shift >= 9 and tiles >> shift <= MOST
        assert shift == 9 or tiles >> (shift - 1) > MOST


def test_prefixes_that_calls_leave(host):
    """After every call the header holds its prefixes and no others: calls of more and fewer tiles in turn, with
    blocks of one length and of several."""
    rng = random.Random(5)
    edges = [1, 2, 63, 511, 512, 513, 1024, 64 * 512, 65 * 512 + 3, LIMIT - 1, LIMIT, LIMIT + 511, LIMIT + 512, LIMIT + 1024,
             2 * LIMIT, 2 * LIMIT + 1024, 3 * LIMIT]
    header = ctypes.create_string_buffer(host.host_header_bytes())
    first_line = 256
    def prefixes():
        words = memoryview(header.raw[first_line:first_line + 128 * 64]).cast("Q")
        return [words[16 * line + 2 + k] for line in range(64) for k in range(14)]
    for call, tiles in enumerate(edges + edges[::-1] + [rng.choice(edges) for _ in range(120)]):
        shift = host.host_block_shift(tiles)
        assert host.host_prefix_call(header, tiles) == tiles >> shift
        got = prefixes()
        want = [(1 + call % 2) << 62 | ((b + 1) << shift) - 1 for b in range(tiles >> shift)]
        assert got[:len(want)] == want and not any(got[len(want):]), "call %d of %d tiles" % (call, tiles)
        assert int.from_bytes(header.raw[8:16], "little") & 0xFFFFFFFF == len(want) << 15 | (call + 1)


@pytest.mark.parametrize("w", [4, 2])
def test_the_workspace_holds_every_calls_state(host, w):
    tile = 16384 // w
    sizes = [k * tile + d for k in (0, 1, 7, 8, 15, 16, 31, 32, 33, 63, 64, 65, 8191, 8192, 8193, 10 ** 6) for d in (-1, 0, 1, 31, 32)]
    for n in [n for n in sizes if n >= 0]:
        assert host.host_header_bytes() + host.host_scan_bytes(n, w) <= zvc.zvc_workspace_bytes(n, w), n
