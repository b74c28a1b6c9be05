"""The fused product's kernels for up to eight rows read a codeword in one 64-bit LDS access.  Where the compiler knows two and only
two of a codeword's address bits to be zero it takes two of 32 bits instead, and both meet the lanes' bank conflicts."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_26339_amd import build, qamw

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_codewords_are_read_whole(tmp_path):
    qamw.lib()                                                # builds it if nothing is there
    lib = str(tmp_path / "lib.so")
    shutil.copy(build.LIB, lib)
    subprocess.check_call([OBJDUMP, "--offloading", lib], cwd=tmp_path, stdout=subprocess.DEVNULL)
    code = [p for p in tmp_path.iterdir() if p.name.endswith("gfx950") and b"k_qgemv" in p.read_bytes()]
    assert len(code) == 1
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(code[0])], capture_output=True, text=True, check=True).stdout
    kernels = re.split(r"^[0-9a-f]+ <", text, flags=re.M)
    gemv = {k.split(">", 1)[0]: k for k in kernels if "k_qgemv" in k.split(">", 1)[0]}
    assert len(gemv) > 50
    for name, body in gemv.items():
        assert "ds_read_b64" in body, name
        assert "ds_read2_b32" not in body, name
