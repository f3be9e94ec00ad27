"""The calls that the codec's speed is measured by.

A case is one pass through the public entry points of paper_1705_01626_amd.zvc
on buffers that a training or serving program keeps: the dense activation
tensor, the compressed buffer, the workspace.  Sizes and densities are those of
the repository's workloads (the small convolution, the AlexNet-style first
layer, the VGG-16 layers, the layout variants, the density sweep) and, for the
drawn cases, anything between a 64 KB and a 640 MB tensor: any element count,
16- and 32-bit types, any density, tensors of their own and tensors that begin
in the middle of a packed arena.

All outputs are bytes and integers and are compared exactly.
"""
import math

import torch

from paper_1705_01626_amd import zvc

DTYPES = {"fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
PLANE = 55 * 55        # elements of one channel of one image, for the per-channel densities
CLUSTER = 8            # neighbouring elements that share most of their luck (zeros cluster)
LARGEST_BYTES = 640 << 20
OFFLOAD_BYTES = 64 * 512 * 14 * 14 * 4
WINDOWS = (1024, 2048, 4096, 8192, 16384, 32768, 65536)
OPS = ("compress", "decompress", "relu_compress", "bounded", "static", "size", "window_compress",
       "window_decompress", "offload")


def _case(name, op, dtype, n, lo, hi, **more):
    """lo, hi: share of non-zero elements of the sparsest and the densest channel (equal: iid)."""
    case = {"op": op, "dtype": dtype, "n": int(n), "lo": float(lo), "hi": float(hi), "offset": 0, "window": 4096,
            "part": 1.0}
    if name:
        case["name"] = name
    case.update(more)
    return case


def listed():
    return [
        # The smallest call of an offload stream: the class scores of a VGG-16 batch of 64.
        _case("fc_scores_compress_fp32", "compress", "fp32", 64 * 1000, 0.1, 0.1),
        # A small convolution layer's output (6.4 MB), leaving and coming back: latency and launches count.
        _case("conv_small_compress_fp32", "compress", "fp32", 8 * 64 * 56 * 56, 0.4, 0.4),
        _case("conv_small_decompress_fp32", "decompress", "fp32", 8 * 64 * 56 * 56, 0.4, 0.4),
        # An ordinary layer in mixed-precision training (51 MB): pre-activations in, stream of ReLU(x) out ...
        _case("layer_relu_compress_bf16", "relu_compress", "bf16", 128 * 256 * 28 * 28, 0.1, 0.5),
        # ... and the same layer's stream decoded before its backward pass.
        _case("layer_decompress_bf16", "decompress", "bf16", 128 * 256 * 28 * 28, 0.1, 0.5),
        # Activations of a batch of 63 packed back to back in one arena: the tensor begins at an odd
        # element and has an odd number of them.
        _case("arena_decompress_fp16", "decompress", "fp16", 63 * 127 * 57 * 57, 0.2, 0.6, offset=3),
        # The paper's own stream order in 4 KB windows, written for the first layer of an AlexNet-sized
        # network (297 MB) ...
        _case("conv1_window_compress_fp32", "window_compress", "fp32", 256 * 96 * 55 * 55, 0.1, 0.9),
        # ... a deep, sparse layer's whole tensor read back from 4 KB windows (103 MB) ...
        _case("deep_window_decompress_fp32", "window_decompress", "fp32", 64 * 512 * 28 * 28, 0.05, 0.3),
        # ... and a prefetch of half the images of a 16-bit first layer from 64 KB windows.
        _case("conv1_window_part_bf16", "window_decompress", "bf16", 256 * 96 * 55 * 55, 0.1, 0.9, window=65536,
              part=0.5),
        # The largest layers (822 MB, VGG-16's first): half of the elements non-zero on the way out,
        # a fifth on the way back.
        _case("sweep_compress_fp32", "compress", "fp32", 64 * 64 * 224 * 224, 0.5, 0.5),
        _case("sweep_decompress_fp32", "decompress", "fp32", 64 * 64 * 224 * 224, 0.2, 0.2),
        # The whole round trip over the link: compress, copy to pinned host memory, copy back, decompress.
        _case("offload_round_trip_fp32", "offload", "fp32", 64 * 512 * 14 * 14, 0.2, 0.2),
    ]


def draw(rng):
    op = rng.choice(OPS)
    dtype = rng.choice(("fp32", "fp32", "bf16", "fp16"))
    w = 4 if dtype == "fp32" else 2
    top = OFFLOAD_BYTES if op == "offload" else LARGEST_BYTES
    n = int(math.exp(rng.uniform(math.log(65536), math.log(top)))) // w
    if rng.random() < 0.3:
        n = max(1024, n // 1024 * 1024)
    if rng.random() < 0.5:
        lo = hi = round(rng.choice((rng.uniform(0.02, 1.0), rng.uniform(0.02, 0.5), 1.0)), 3)
    else:
        lo = round(rng.uniform(0.02, 0.5), 3)
        hi = round(rng.uniform(lo, 0.95), 3)
    offset = rng.choice((0, 0, 0, 0, 0, 1, 2, 3, 4, 7))
    part = rng.choice((1.0, 1.0, 0.5, 0.125)) if op == "window_decompress" else 1.0
    return _case(None, op, dtype, n, lo, hi, offset=0 if op == "offload" else offset, window=rng.choice(WINDOWS),
                 part=part)


# ------------------------------------------------------------------------------- inputs
def _activations(case, seed):
    """The dense tensor: |N(0,1)| where kept; elsewhere zero or, for the fused ReLU, a negative
    number (one in fifty of them a zero of either sign)."""
    n, lo, hi = case["n"], case["lo"], case["hi"]
    dtype = DTYPES[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)

    def normal(count):
        return torch.randn(count, generator=g, device="cuda", dtype=torch.float32)

    base = torch.zeros(case["offset"] + n, dtype=dtype, device="cuda")
    x = base[case["offset"]:]
    planes = -(-n // PLANE)
    dens = lo + (hi - lo) * torch.rand(planes, generator=g, device="cuda")
    threshold = math.sqrt(2.0) * torch.erfinv((2.0 * dens - 1.0).clamp(-1.0, 1.0))
    step = PLANE * CLUSTER * 2048                       # 50 M elements at a time
    for at in range(0, n, step):
        count = min(step, n - at)
        luck = normal(count)
        if lo != hi:
            luck.mul_(0.6).add_(normal(-(-count // CLUSTER)).repeat_interleave(CLUSTER)[:count], alpha=0.8)
        keep = luck < threshold[at // PLANE:].repeat_interleave(PLANE)[:count] if lo < 1.0 else luck == luck
        del luck
        v = normal(count).abs_().clamp_(min=1e-3)
        if _relu(case):
            zeros = torch.rand(count, generator=g, device="cuda")
            dropped = torch.where(zeros < 0.01, 0.0, torch.where(zeros < 0.02, -0.0, -v))
        else:
            dropped = torch.zeros((), device="cuda")
        x[at:at + count] = torch.where(keep, v, dropped).to(dtype)
    return x


def _relu(case):
    return case["op"] == "relu_compress"


def _kept(case, x):
    return x > 0 if _relu(case) else x != 0


def _stream_bytes(case, x):
    n, w = x.numel(), x.element_size()
    return 4 * (-(-n // 32)) + w * int(torch.count_nonzero(_kept(case, x)).item())


def _bound(case):
    """Capacity for a stream kept in GPU memory: what the densest channel's share would need, and a little."""
    w = 4 if case["dtype"] == "fp32" else 2
    return 4 * (-(-case["n"] // 32)) + w * int(case["n"] * min(1.0, case["hi"] + 0.1))


def _range(case):
    """First window and number of windows of a (partial) window decode, and its elements."""
    w = 4 if case["dtype"] == "fp32" else 2
    per = case["window"] // w
    windows = -(-case["n"] // per)
    count = max(1, int(windows * case["part"]))
    first = (windows - count) // 2
    return first, count, first * per, min(case["n"], (first + count) * per)


def prepare(case, seed):
    op, n = case["op"], case["n"]
    x = _activations(case, seed)
    w = x.element_size()
    s = {"case": case, "ws": zvc.new_workspace(n, w), "d_bytes": torch.zeros(1, dtype=torch.int64, device="cuda")}
    nbytes = _stream_bytes(case, x)
    s["nbytes"] = nbytes
    windowed = op.startswith("window")
    if windowed:
        s["offsets"] = torch.zeros(zvc.zvc_window_count(n, w, case["window"]) + 1, dtype=torch.int64, device="cuda")
    if op == "bounded":
        s["comp"] = torch.zeros(_bound(case), dtype=torch.uint8, device="cuda")
    elif op != "size":
        s["comp"] = zvc.new_compressed_buffer(n, w).zero_()
    if op == "decompress":
        zvc.zvc_compress(x, s["comp"], s["d_bytes"], s["ws"])
        s["out"] = torch.zeros(case["offset"] + n, dtype=x.dtype, device="cuda")[case["offset"]:]
    elif op == "window_decompress":
        zvc.zvc_window_compress(x, s["comp"], s["offsets"], s["d_bytes"], s["ws"], window_bytes=case["window"])
        _, _, lo, hi = _range(case)
        s["out"] = torch.zeros(case["offset"] + hi - lo, dtype=x.dtype, device="cuda")[case["offset"]:]
    else:
        s["x"] = x
    if op == "offload":
        s["out"] = torch.zeros_like(x)
        s["pinned"] = torch.zeros(s["comp"].numel(), dtype=torch.uint8, pin_memory=True)
        s["h_bytes"] = torch.zeros(1, dtype=torch.int64, pin_memory=True)
        s["copy"] = torch.cuda.Stream()
    torch.cuda.synchronize()
    return s


def run(s):
    case, op = s["case"], s["case"]["op"]
    stream = s.get("comp")               # whole buffer: the stream, then bytes that prepare() cleared
    if op == "compress":
        zvc.zvc_compress(s["x"], s["comp"], s["d_bytes"], s["ws"])
        return stream, s["d_bytes"]
    if op == "relu_compress":
        zvc.zvc_relu_compress(s["x"], s["comp"], s["d_bytes"], s["ws"])
        return stream, s["d_bytes"]
    if op == "bounded":
        zvc.zvc_compress_bounded(s["x"], s["comp"], s["d_bytes"], s["ws"])
        return stream, s["d_bytes"]
    if op == "static":
        zvc.zvc_compress_static(s["x"], s["comp"], s["d_bytes"])
        return stream, s["d_bytes"]
    if op == "size":
        zvc.zvc_compressed_size(s["x"], s["d_bytes"], s["ws"])
        return s["d_bytes"]
    if op == "decompress":
        zvc.zvc_decompress(s["comp"], s["nbytes"], s["out"], s["ws"])
        return s["out"]
    if op == "window_compress":
        zvc.zvc_window_compress(s["x"], s["comp"], s["offsets"], s["d_bytes"], s["ws"], window_bytes=case["window"])
        return stream, s["offsets"], s["d_bytes"]
    if op == "window_decompress":
        first, count, _, _ = _range(case)
        zvc.zvc_window_decompress(s["comp"], s["nbytes"], s["offsets"], case["n"], first, count, s["out"],
                                  window_bytes=case["window"])
        return s["out"]
    compute = torch.cuda.current_stream()
    nbytes = zvc.zvc_offload(s["x"], s["comp"], s["pinned"], s["h_bytes"], s["ws"], compute, s["copy"])
    zvc.zvc_prefetch(s["pinned"], nbytes, s["comp"], s["out"], s["ws"], s["copy"], compute)
    return s["pinned"], s["h_bytes"], s["out"]


def work(case):
    n, op = case["n"], case["op"]
    w = 4 if case["dtype"] == "fp32" else 2
    density = 0.5 * (case["lo"] + case["hi"])
    stream = 4 * (-(-n // 32)) + int(w * n * density)
    table = 8 * (-(-n * w // case["window"]) + 1)
    if op == "size":
        total = n * w + 8
    elif op == "window_decompress":
        _, count, lo, hi = _range(case)
        total = (hi - lo) * w + int(stream * (hi - lo) / n) + 8 * (count + 1)
    elif op == "window_compress":
        total = n * w + stream + table
    elif op == "offload":
        total = 2 * (n * w + stream)          # and `stream` bytes over the link, each way
    else:
        total = n * w + stream
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------------------- the same in plain torch
def _masks(keep):
    groups = -(-keep.numel() // 32)
    padded = torch.zeros(groups * 32, dtype=torch.bool, device=keep.device)
    padded[:keep.numel()] = keep
    out = torch.zeros(groups, dtype=torch.int64, device=keep.device)
    rows = padded.view(groups, 32)
    for b in range(32):
        out |= rows[:, b].to(torch.int64) << b
    return out, rows.sum(dim=1)


def _low_bytes(masks):
    return masks.view(torch.int32)[::2].contiguous().view(torch.uint8)      # little-endian low halves


def _padded(case, stream):
    """`stream` as it lies in its buffer."""
    w = 4 if case["dtype"] == "fp32" else 2
    out = torch.zeros(_bound(case) if case["op"] == "bounded" else zvc.zvc_max_compressed_bytes(case["n"], w),
                      dtype=torch.uint8, device="cuda")
    out[:stream.numel()] = stream
    return out


def _windowed(case, x):
    w = x.element_size()
    keep = x != 0
    masks, kept = _masks(keep)
    words_per_mask = 4 // w
    ends = torch.cumsum(kept + words_per_mask, 0)
    begins = ends - kept - words_per_mask                                   # in elements, of every group
    total = int(ends[-1].item())
    word = torch.int32 if w == 4 else torch.int16
    stream = torch.zeros(total, dtype=word, device=x.device)
    halves = _low_bytes(masks).view(word).view(-1, words_per_mask)
    for k in range(words_per_mask):
        stream[begins + k] = halves[:, k]
    index = torch.nonzero(keep).view(-1)
    # a kept element lies behind the masks of the groups up to its own and the kept elements before it
    place = torch.arange(index.numel(), device=x.device) + (index // 32 + 1) * words_per_mask
    stream[place] = x.view(word)[index]
    per_groups = case["window"] // w // 32
    offsets = torch.cat([begins[::per_groups], ends[-1:]]) * w
    return _padded(case, stream.view(torch.uint8)), offsets, torch.tensor([total * w], device=x.device)


def exact(case, seed):
    x = _activations(case, seed)
    op = case["op"]
    if op == "decompress":
        return x
    if op == "window_decompress":
        _, _, lo, hi = _range(case)
        return x[lo:hi]
    if op == "window_compress":
        return _windowed(case, x)
    keep = _kept(case, x)
    size = torch.tensor([_stream_bytes(case, x)], device="cuda")
    if op == "size":
        return size
    masks, _ = _masks(keep)
    stream = _padded(case, torch.cat([_low_bytes(masks), x[keep].contiguous().view(torch.uint8)]))
    if op == "offload":
        return stream, size, x
    return stream, size
