"""The team kernels' mail leaves in 16-byte buffer stores, whose four data registers
are read over several cycles.  With a scalar offset the compiler keeps no wait states
before their next write (lanes 12..15 of each row then sent what the register held
afterwards), so none may have one; read from the built library's gfx950 code."""
import os
import re
import subprocess

import pytest

from test_kernel_resources import LLVM, MAGIC, TARGET

pytestmark = pytest.mark.skipif(
    not all(os.path.exists(os.path.join(LLVM, t))
            for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")),
    reason="ROCm LLVM tools not available")


def test_16_byte_buffer_stores_have_no_scalar_offset(tmp_path):
    from paper_1905_06850_amd import plcg
    fat = tmp_path / "fat.bin"
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}",
                    plcg.LIB_PATH, os.devnull], check=True, capture_output=True)
    data = fat.read_bytes()
    starts = [m.start() for m in re.finditer(re.escape(MAGIC), data)]
    stores = 0
    for k, s in enumerate(starts):
        e = starts[k + 1] if k + 1 < len(starts) else len(data)
        if b"team_kernel" not in data[s:e]:
            continue
        b, co = tmp_path / f"b{k}.bin", tmp_path / f"co{k}.o"
        b.write_bytes(data[s:e])
        subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o",
                        f"--input={b}", f"--targets={TARGET}", f"--output={co}"],
                       check=True, capture_output=True)
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", str(co)], check=True,
                              capture_output=True, text=True).stdout
        for line in re.findall(r"buffer_store_dwordx[34] .*", text):
            stores += 1
            soffset = line.split("//")[0].split(",")[3].split()[0]
            assert soffset == "0", line
    assert stores > 0
