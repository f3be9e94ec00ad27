"""What the library asks of the HIP runtime, call by call, written down by a stand-in for the runtime
(fake_hip.cpp) in a child process: which streams work and copies go to, and which events order them.
No GPU needed."""
import os
import re
import subprocess
import sys

import pytest

from paper_1705_01626_amd import build as zvc_build
from tests import test_gpu_shifted_output as shifted
from tests.decoder_routes import ROUTES, elements

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPUTE, COPY = 0x1000, 0x2000
IN, STAGE, WS, HOST, OUT = 1 << 41, 1 << 42, 1 << 43, 1 << 44, 1 << 45
CHILD = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
fake.fake_log.restype = ctypes.c_char_p
lib.zvc_max_compressed_bytes.restype = lib.zvc_workspace_bytes.restype = ctypes.c_size_t
size = ctypes.c_uint64(0)
def call(name, *args):
    wide = [ctypes.c_size_t(a) if isinstance(a, int) else a for a in args]
    status = getattr(lib, name)(*wide)
    assert status == 0, (name, status)
def worst(n, w):
    return lib.zvc_max_compressed_bytes(ctypes.c_size_t(n), w)
def room(n, w):
    return lib.zvc_workspace_bytes(ctypes.c_size_t(n), w)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", zvc_build.ROCM_INCLUDE,
                    "-o", out, os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True)
    return out


def run(fake, code):
    """The stand-in's lines for `code`, split into words and key=value pairs."""
    done = subprocess.run([sys.executable, "-c", CHILD + code + "\nprint(fake.fake_log().decode())", fake,
                           zvc_build.ensure_built()], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stderr[-2000:]
    lines = []
    for line in done.stdout.splitlines():
        words = line.split()
        if words:
            lines.append((words[0], {k: int(v) for k, v in re.findall(r"(\w+)=(-?\d+)", line)}, words[-1]))
    return lines


# Flags under which an event does not order everything before it, or not for the host.
DISABLE_SYSTEM_FENCE, RELEASE_TO_DEVICE = 0x20000000, 0x40000000

OFFLOAD = """
n, w = %d, %d
fake.fake_host_memory(%d)
fake.fake_written(ctypes.byref(size), %d)
call('zvc_offload', %d, n, w, %d, worst(n, w), %d, worst(n, w), ctypes.addressof(size), %d, room(n, w), %d, %d)
"""
PREFETCH = """
n, w = %d, %d
fake.fake_host_memory(%d)
call('zvc_prefetch', %d, %d, n, w, %d, worst(n, w), %d, %d, room(n, w), %d, %d)
"""


@pytest.mark.parametrize("n,w,pinned", [(100001, 4, 1), (100001, 2, 1), (100001, 4, 0), (20 << 20, 4, 1)])
def test_order_of_an_offload(fake, n, w, pinned):
    """The host waits for an event that releases to the whole system, recorded behind the encoder on
    `compute`; the stream goes to `copy` after that wait."""
    nbytes = 4 * -(-n // 32) + w * (n // 5)
    lines = run(fake, OFFLOAD % (n, w, pinned, nbytes, IN, STAGE, HOST, WS, COMPUTE, COPY))
    kinds = [k for k, _, _ in lines]
    made = {v["event"]: v["flags"] for k, v, _ in lines if k == "create"}
    assert kinds.count("synchronize") == 1
    wait = kinds.index("synchronize")
    record = kinds.index("record")
    event = lines[wait][1]["event"]
    assert lines[record][1] == {"event": event, "stream": COMPUTE} and record < wait
    assert made[event] & (DISABLE_SYSTEM_FENCE | RELEASE_TO_DEVICE) == 0
    encoder = [i for i, (k, v, name) in enumerate(lines) if k == "launch" and "compress_kernel" in name]
    assert len(encoder) == 1 and encoder[0] < record and lines[encoder[0]][1]["stream"] == COMPUTE
    assert all(i > wait for i, (k, v, _) in enumerate(lines) if v.get("stream") == COPY)


@pytest.mark.parametrize("n,w,pinned", [(100001, 4, 1), (100001, 2, 1), (100001, 4, 0), (20 << 20, 4, 1)])
def test_order_of_a_prefetch(fake, n, w, pinned):
    """`compute` waits for an event that is recorded behind the copy on `copy` and that orders what
    lies before it; the decoder's launches come behind that wait.  One stream needs no event."""
    nbytes = 4 * -(-n // 32) + w * (n // 5)
    lines = run(fake, PREFETCH % (n, w, pinned, HOST, nbytes, STAGE, OUT, WS, COPY, COMPUTE))
    kinds = [k for k, _, _ in lines]
    made = {v["event"]: v["flags"] for k, v, _ in lines if k == "create"}
    record, wait = kinds.index("record"), kinds.index("wait")
    event = lines[wait][1]["event"]
    assert lines[wait][1] == {"event": event, "stream": COMPUTE}
    assert lines[record][1] == {"event": event, "stream": COPY} and record < wait
    assert made[event] & DISABLE_SYSTEM_FENCE == 0
    assert all(i < record for i, (k, v, _) in enumerate(lines) if k in ("launch", "copy") and v["stream"] == COPY)
    assert all(i > wait for i, (k, v, _) in enumerate(lines) if k == "launch" and v["stream"] == COMPUTE)
    one = run(fake, PREFETCH % (n, w, pinned, HOST, nbytes, STAGE, OUT, WS, COMPUTE, COMPUTE))
    assert not [k for k, _, _ in one if k in ("record", "wait", "synchronize")]


@pytest.mark.parametrize("n,w,pinned", [(8192, 4, 1), (100001, 2, 1), (100001, 4, 0), (20 << 20, 4, 1)])
def test_copies_are_the_runtimes(fake, n, w, pinned):
    """The stream crosses the link by one copy of the runtime, on `copy` and of exactly its size, and no
    kernel runs there: a kernel would wait for compute units that the program's own work holds, and keep
    them from it.  The size comes by a copy only where the GPU cannot write it."""
    nbytes = 4 * -(-n // 32) + w * (n // 5)
    out = run(fake, OFFLOAD % (n, w, pinned, nbytes, IN, STAGE, HOST, WS, COMPUTE, COPY))
    back = run(fake, PREFETCH % (n, w, pinned, HOST, nbytes, STAGE, OUT, WS, COPY, COMPUTE))
    assert not [v for k, v, _ in out + back if k == "launch" and v["stream"] == COPY]
    assert [v for k, v, _ in out if k == "copy" and v["stream"] == COPY] == [
        {"stream": COPY, "to": HOST, "from": STAGE, "bytes": nbytes}]
    assert [v for k, v, _ in back if k == "copy"] == [{"stream": COPY, "to": STAGE, "from": HOST, "bytes": nbytes}]
    assert [v["bytes"] for k, v, _ in out if k == "copy" and v["stream"] == COMPUTE] == ([] if pinned else [8])


ENCODERS = {
    "compress": "call('zvc_compress', %d, n, w, %d, worst(n, w), %d, %d, room(n, w), 0)" % (IN, OUT, HOST, WS),
    "relu": "call('zvc_relu_compress', %d, n, w, %d, worst(n, w), %d, %d, room(n, w), 0)" % (IN, OUT, HOST, WS),
    "windowed": "call('zvc_window_compress', %d, n, w, 4096, %d, worst(n, w), %d, %d, %d, room(n, w), 0)"
                % (IN, OUT, HOST, HOST + 64, WS),
}
MB = 1 << 20


@pytest.mark.parametrize("mode,w,nbytes,tile,early", [
    # half of the staging behind the count: 16-bit tiles where the call is one short chain of tiles
    ("compress", 2, 4 * MB, 16384, 1), ("compress", 2, 12 * MB, 16384, 1), ("relu", 2, 17 * MB, 16384, 1),
    ("compress", 2, 24 * MB, 16384, 0), ("compress", 2, 64 * MB, 32768, 0),
    # 32 KB tiles from 48 MB of 16-bit elements on
    ("compress", 2, 47 * MB, 16384, 0), ("compress", 2, 49 * MB, 32768, 0), ("relu", 2, 49 * MB, 32768, 0),
    # fp32: all but the large ones
    ("compress", 4, 4 * MB, 16384, 1), ("relu", 4, 20 * MB, 32768, 1), ("compress", 4, 40 * MB, 32768, 1),
    ("compress", 4, 64 * MB, 32768, 0), ("relu", 4, 80 * MB, 32768, 0), ("compress", 4, 300 * MB, 65536, 0),
])
def test_encoder_by_size(fake, mode, w, nbytes, tile, early):
    """The tile and the order of staging and count that measure best at a size (the measurements stand
    beside the rules)."""
    lines = run(fake, "n, w = %d, %d\n%s" % (nbytes // w, w, ENCODERS[mode]))
    (kind, values, name), = lines
    assert kind == "launch"
    got = re.search(r"compress_kernelILi(\d)ELi(\d+)ELi(\d)ELb(\d)ELb(\d)ELb(\d)ELb(\d)E", name).groups()
    got_w, chunks, waves, relu, windowed, _, got_early = map(int, got)
    assert (got_w, relu, windowed) == (w, mode == "relu", mode == "windowed")
    assert (chunks * waves * 256, got_early) == (tile, early)
    assert values["grid"] == -(-nbytes // tile)


WINDOW_DECODE = """
n, w, window = %d, %d, %d
windows = -(-n * w // window)
call('zvc_window_decompress', %d, 4 * -(-n // 32) + int(w * n * %f), %d, n, w, window, 0, windows, %d, 0)
"""


@pytest.mark.parametrize("w,window,nbytes,density,interleaved", [
    # sparse streams of 32-bit elements: the order in which the XCDs write next to each other, from 150 MB up
    (4, 1024, 784 * MB, 0.05, 1), (4, 2048, 784 * MB, 0.05, 1), (4, 4096, 784 * MB, 0.05, 1), (4, 1024, 200 * MB, 0.02, 1),
    (4, 1024, 130 * MB, 0.05, 0), (2, 1024, 300 * MB, 0.05, 0), (2, 4096, 784 * MB, 0.05, 0),
    # between a twelfth and a fifth only the largest, and earlier the denser
    (4, 1024, 400 * MB, 0.12, 0), (4, 1024, 784 * MB, 0.12, 1), (2, 2048, 784 * MB, 0.12, 1), (4, 2048, 300 * MB, 0.25, 0),
    (2, 1024, 450 * MB, 0.25, 1), (4, 4096, 200 * MB, 0.4, 0), (4, 4096, 300 * MB, 0.4, 1), (2, 2048, 160 * MB, 0.6, 1),
    (4, 2048, 130 * MB, 0.6, 0), (4, 1024, 66 * MB, 0.9, 1), (2, 4096, 60 * MB, 0.9, 0),
])
def test_order_of_window_decoding(fake, w, window, nbytes, density, interleaved):
    """In which order the windows are dealt out to the XCDs (the measurements stand beside the rule)."""
    lines = run(fake, WINDOW_DECODE % (nbytes // w, w, window, STAGE, density, HOST, OUT))
    (kind, values, name), = lines
    assert kind == "launch" and "window_decode_kernelILi%d" % w in name
    assert values["choice"] == interleaved
    assert values["lds"] == 0


DECODE = """
n, w = %d, %d
call('zvc_decompress', %d, 4 * -(-n // 32) + int(w * n * %f), n, w, %d, %d, room(n, w), 0)
"""


@pytest.mark.parametrize("w", [4, 2])
@pytest.mark.parametrize("nbytes,density,interleaved,seven", [
    (60 * MB, 0.6, 0, 0), (66 * MB, 0.6, 1, 1), (66 * MB, 0.05, 1, 0), (300 * MB, 0.2, 0, 0), (300 * MB, 0.3, 0, 1),
    (450 * MB, 0.2, 1, 0), (784 * MB, 0.02, 1, 0), (784 * MB, 0.15, 1, 0), (784 * MB, 0.2, 1, 1), (784 * MB, 1.0, 1, 1),
])
def test_order_and_occupancy_of_decoding(fake, w, nbytes, density, interleaved, seven):
    """Large planar outputs: the order of the parts, and eight workgroups per CU or seven."""
    lines = run(fake, DECODE % (nbytes // w, w, STAGE, density, OUT, WS))
    launched = [(v, name) for k, v, name in lines if "17decompress_kernelILi%d" % w in name]
    assert len(launched) == 1 and len(lines) == 2
    values = launched[0][0]
    assert (values["choice"], values["lds"] > 0) == (interleaved, bool(seven))


ROUTE = re.compile(r"(?:decompress_(direct|scan)_kernelILi(\d)ELN.*?OutputE(\d)ELi(\d)E(?:Lb(\d)E)?|17decompress_kernelILi(\d)ELi\d+ELN.*?OutputE(\d)E)")
OUTPUTS = ("aligned", "loose", "shifted")


def routes(fake, calls):
    """How the planar decoder takes each of the calls (elements, width, the output's first element, density):
    direct4 | direct8 | scan4 | scan8 | two, and how it writes."""
    code = "".join("n, w = %d, %d\ncall('zvc_decompress', %d, 4 * -(-n // 32) + w * int(n * %f), n, w, %d, %d, room(n, w), 0)\n"
                   % (n, w, STAGE, density, OUT + first * w, WS) for n, w, first, density in calls)
    found = []
    for _, _, name in run(fake, code):
        got = ROUTE.search(name)
        if got is None:
            assert "mask_prefix_kernel" in name          # the first of two
            continue
        one, w, output, waves, hint, two_w, two_output = got.groups()
        found.append((one + waves if one else "two", OUTPUTS[int(output or two_output)]))
        assert int(w or two_w) == calls[len(found) - 1][1]
        if one == "scan":                                # dense streams are read with the streaming hint
            assert hint == "%d" % (calls[len(found) - 1][3] >= 0.75)
    assert len(found) == len(calls)
    return found


@pytest.mark.parametrize("w", [4, 2])
def test_decoder_by_size(fake, w):
    """Both sides of every limit of the planar decoder (the measurements stand beside the rules)."""
    masks = 8 * 1024                                     # elements per KB of masks
    aligned = [(48 * masks, "direct4"), (48 * masks + 32, "direct8"), (80 * masks, "direct8"), (80 * masks + 32, "scan4"),
               (9 * MB // 2 // w - 1, "scan4"), (9 * MB // 2 // w, "scan8"), (32 * MB // w, "scan8"), (32 * MB // w + 1, "scan4"),
               (44 * MB // w - 1, "scan4"), (44 * MB // w, "two")]
    for density in (0.05, 0.5, 0.9):
        assert routes(fake, [(n, w, 0, density) for n, _ in aligned]) == [(route, "aligned") for _, route in aligned]
    odd = [(n, route, "loose" if n * w < 8 * MB else "shifted") for n, route in aligned[:-1]] + [
        (8 * MB // w - 1, "scan8", "loose"), (8 * MB // w, "scan8", "shifted"), (44 * MB // w, "scan4", "shifted"),
        (56 * MB // w - 1, "scan4", "shifted")]
    for density in (0.05, 0.5, 0.9):
        limit = 76 if density == 0.9 else 56
        more = [(limit * MB // w - 1, "scan4", "shifted"), (limit * MB // w, "two", "shifted")]
        assert routes(fake, [(n, w, 1, density) for n, _, _ in odd + more]) == [(route, out) for _, route, out in odd + more]
    # whole 16 bytes that are no line: as they lie in one launch, in two only whole 64 bytes (128 in the largest fp32 outputs)
    for first, small, large in ((16 // w, "shifted", "shifted"), (64 // w, "aligned", "shifted" if w == 4 else "aligned"),
                                (128 // w, "aligned", "aligned")):
        assert routes(fake, [(43 * MB // w, w, first, 0.5), (60 * MB // w, w, first, 0.5), (256 * MB // w, w, first, 0.5)]) == [
            ("scan4", "aligned"), ("two", small), ("two", large)]


@pytest.mark.parametrize("w", [4, 2])
def test_sizes_of_the_decoder_tests(fake, w):
    """The sizes that the GPU tests use for a kernel take that kernel."""
    for first in (0, 1, 16 // w):
        for density in (0.05, 0.6, 1.0):
            calls = [(elements(route, w, first, density > 0.7), w, first, density) for route in ROUTES]
            assert [route for route, _ in routes(fake, calls)] == [route.split()[0] for route in ROUTES]


@pytest.mark.parametrize("w", [4, 2])
def test_sizes_of_the_shifted_outputs_tests(fake, w):
    offsets = shifted.every_offset(w)
    got = routes(fake, [(n, w, first, density) for n, first, density in offsets])
    assert [out for _, out in got] == ["shifted"] * len(offsets) and {route for route, _ in got} == {"scan8", "two"}
    edges = shifted.chunk_edges(w)
    assert routes(fake, [(n, w, first, density) for n, first, density in edges]) == [("two", "shifted")] * len(edges)
    ends = shifted.early_ends(w)
    assert {out for _, out in routes(fake, [(n, w, first, 0.6) for n, first, _ in ends[:4]])} == {"loose"}
    assert routes(fake, [(n, w, first, 0.6) for n, first, _ in ends[4:]]) == [
        ("scan8", "shifted"), ("scan4", "shifted")] + [("two", "shifted")] * 3
