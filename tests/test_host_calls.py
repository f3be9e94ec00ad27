"""What the library asks of the HIP runtime, call by call, written down by a stand-in for the runtime
(fake_hip.cpp) in a child process: which streams work and copies go to, and which events order them.
No GPU needed."""
import os
import re
import subprocess
import sys

import pytest

from paper_1705_01626_amd import build as zvc_build

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
