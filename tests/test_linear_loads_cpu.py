"""The linear's operand loads carry their whole offset in the lane's register: a buffer's length is checked against
that, while a scalar offset is described as left out of the check and as subtracted from the length, which wraps for
a buffer of length zero.  And the residual update's two ways of writing the stream are two kernels: as a choice at run
time the compiler made both of them plain.  Read from the library's own gfx950 code."""
import glob
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2506_13497_amd", "libddit_hot.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_buffer_load_has_a_scalar_offset(tmp_path):
    os.symlink(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    loads = []
    for code in glob.glob(str(tmp_path / "lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", code], check=True, capture_output=True, text=True).stdout
        loads += re.findall(r"buffer_load_\w+ .*?\], (\S+) offen.* lds", text)
    assert len(loads) > 100, "the linear's loads were not found"
    assert set(loads) == {"0"}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_small_streams_are_written_streaming_and_large_ones_plainly(tmp_path):
    os.symlink(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    stores = {"2": [], "4": []}
    for code in glob.glob(str(tmp_path / "lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", code], check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"<(\S*k_gemm_bf16\S*)>:\n(.*?)(?=\n\n|\Z)", text, re.S):
            epi = re.search(r"k_gemm_bf16I(?:Li\dE){6}Li(\d)E", name).group(1)
            if epi in stores:
                lines = re.findall(r"(?:flat|global)_store_dwordx4 [^\n]*", body)
                stores[epi].append([bool(re.search(r"\bnt\b", l)) for l in lines])
    assert len(stores["2"]) == 10 and len(stores["4"]) == 6
    assert not any(any(k) for k in stores["2"]) and all(any(k) for k in stores["4"])
