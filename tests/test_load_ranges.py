"""A buffer resource's range covers a load's vector offset only: packed weight words are read past a filter block's last one (the
half-wave that holds no block), so the place of the K-step has to be in the vector offset (no GPU: the built kernels are looked
over)."""
import glob
import os
import re
import shutil
import subprocess

from paper_1603_05279_amd import xnor
from tests.test_store_hazard import ROCM


def word_loads(lines):
    """(one-word buffer loads of the matrix-core convolutions, those of them whose scalar offset is a register)."""
    kernel, loads, scalar = "", 0, []
    for line in lines:
        label = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if label:
            kernel = label[1]
            continue
        m = re.match(r"buffer_load_dword v\d+, v\d+, s\[\d+:\d+\], (\S+)", line.split("//")[0].strip())
        if m and "conv_mfma_kernel" in kernel:
            loads += 1
            if re.match(r"s\d|m0|vcc|ttmp", m[1]):
                scalar.append((kernel, line.strip()))
    return loads, scalar


def test_the_check_sees_a_scalar_register():
    head, load = "0000 <_ZN4xnor16conv_mfma_kernelE>:", "buffer_load_dword v1, v2, s[4:7], %s offen"
    assert word_loads([head, load % "s9"])[1] and not word_loads([head, load % "0"])[1]


def test_packed_words_are_read_within_the_range_of_their_resource(tmp_path):
    objdump = os.path.join(ROCM, "llvm", "bin", "llvm-objdump")
    shutil.copy(xnor._LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for obj in sorted(glob.glob(str(tmp_path / "*gfx950*"))):
        out = subprocess.Popen([objdump, "-d", obj], stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True)
        loads, scalar = word_loads(out.stdout)
        assert out.wait() == 0
        assert not scalar, (len(scalar), scalar[:3])
        total += loads
    assert total > 0
