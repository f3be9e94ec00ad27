"""What the compiled kernels may rely on, read from the assembly of the library built here (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_1705_01626_amd import build as zvc_build


def tool(name):
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(zvc_build.HIPCC))), "llvm", "bin", name)
    if not os.path.exists(path):
        pytest.skip("%s was not found beside the HIP compiler" % name)
    return path


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    where = tmp_path_factory.mktemp("device_code")
    fat, code = str(where / "fat"), str(where / "gfx950.co")
    subprocess.run([tool("llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, zvc_build.ensure_built(),
                    str(where / "rest.so")], check=True)
    subprocess.run([tool("clang-offload-bundler"), "--unbundle", "--type=o",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + code], check=True)
    return subprocess.run([tool("llvm-objdump"), "-d", "--no-show-raw-insn", code], check=True, capture_output=True,
                          text=True).stdout


def test_buffer_loads_have_their_whole_offset_in_the_range_check(assembly):
    """The encoder reads past the tensor's end by buffer loads whose descriptor ends with the tensor.  The
    range check covers a load's vector and immediate offset; the scalar offset is no part of it, so it has
    to be zero in every one of them."""
    loads = re.findall(r"buffer_load_\w+ +v[\w\[\]:]+, (?:v\w+|off), s\[[\d:]+\], (\w+)", assembly)
    assert len(loads) == len(re.findall(r"\bbuffer_load_", assembly)) > 100
    assert set(loads) == {"0"}, "%d of %d loads have a scalar offset" % (sum(x != "0" for x in loads), len(loads))


def functions(assembly, name):
    """The bodies of the kernels of that name, by mangled name."""
    parts = re.split(r"^[0-9a-f]+ <(\w+)>:$", assembly, flags=re.M)
    return {k: body for k, body in zip(parts[1::2], parts[2::2]) if re.search(r"\d%sI" % name, k)}


def test_input_that_is_read_once_is_read_with_the_streaming_hint(assembly):
    """Without it the tensor's lines push others out of the caches: slower for a tensor from memory, also
    where a kernel has just written it, and no faster for one that is read again and again."""
    encoders, counters = functions(assembly, "compress_kernel"), functions(assembly, "count_kernel")
    assert len(encoders) > 10 and sum("Lb1E" in k for k in counters) >= 2
    for name, body in encoders.items():
        loads = re.findall(r"^\s*(buffer_load_.*?)(?:\s*//.*)?$", body, flags=re.M)
        # (at an odd half dword the last lane of a load needs a dword of the next one's, once more)
        again = re.search(r"Li2ELi\d+ELi4ELb[01]ELb[01]ELb1E", name) is not None
        assert len(loads) >= 16 and sum(" nt" not in x for x in loads) == again, name
    for name, body in counters.items():
        if "Lb1E" in name:                            # (at least 16-byte aligned)
            loads = re.findall(r"^\s*(global_load_dwordx4 .*?)(?:\s*//.*)?$", body, flags=re.M)
            assert len(loads) >= 8 and all(" nt" in x for x in loads), name


def test_the_scan_word_is_there_before_a_wave_counts_itself_in(assembly):
    """The last tile of a call overwrites the word once it has every tile's count, and a tile's count is out
    once its waves have counted themselves in (the only LDS atomic with a result).  So a wave reads the word
    with an atomic load that the other XCDs' caches do not serve, and has it before that."""
    kernels = {**functions(assembly, "compress_kernel"), **functions(assembly, "decompress_scan_kernel")}
    assert len(kernels) > 20
    for name, body in kernels.items():
        lines = [line.split("//")[0].strip() for line in body.splitlines()]
        loads = [i for i, line in enumerate(lines) if re.match(r"global_load_dwordx2 .* offset:8\b", line)]
        arrivals = [i for i, line in enumerate(lines) if line.startswith("ds_add_rtn_u32 ")]
        assert len(loads) == 1 and len(arrivals) == 1, name
        assert lines[loads[0]].endswith(" sc1"), name
        assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", line) for line in lines[loads[0]:arrivals[0]]), name
