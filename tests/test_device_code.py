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
