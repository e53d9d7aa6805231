"""Vector stores of more than 64 bits keep reading their data registers for two wait states after they issue: a vector
instruction that writes one of them sooner reaches memory in place of the value stored.  The compiler keeps that distance
except behind buffer stores whose scalar offset is a register, so the built kernels are looked over (no GPU)."""
import glob
import os
import re
import shutil
import subprocess

from paper_1603_05279_amd import xnor

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
WAIT_STATES = 2


def registers(operand):
    m = re.match(r"([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", operand.strip())
    if not m:
        return set()
    first, last = (m[2], m[3]) if m[2] else (m[4], m[4])
    return {(m[1], i) for i in range(int(first), int(last) + 1)}


def overwritten_stores(lines):
    """(stores of more than 64 bits, [(kernel, store, instruction that overwrites its data too soon)])."""
    kernel, pending, stores, bad = "", [], 0, []
    for line in lines:
        label = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if label:
            kernel, pending = label[1], []
            continue
        text = line.split("//")[0].strip()
        if not text:
            continue
        op, _, rest = text.partition(" ")
        if pending:
            if op.startswith("v_"):
                written = registers(rest)
                bad += [(kernel, store, text) for data, _, store in pending if data & written]
            gap = int(rest, 0) + 1 if op == "s_nop" else 1
            pending = [(data, left - gap, store) for data, left, store in pending if left > gap]
        if re.match(r"(buffer|global|flat)_store_dwordx[34]", op):
            stores += 1
            operands = re.split(r",(?![^\[]*\])", rest)
            pending.append((registers(operands[0 if op.startswith("buffer") else 1]), WAIT_STATES, text))
    return stores, bad


def test_the_check_sees_an_overwritten_register():
    store = "buffer_store_dwordx4 v[40:43], v0, s[36:39], s81 offen"
    head = "0000 <k>:"
    assert overwritten_stores([head, store, "v_mul_f32_e32 v40, v22, v1"])[1]
    assert overwritten_stores([head, store, "s_add_i32 s0, s1, s2", "v_mul_f32_e32 v43, v22, v1"])[1]
    assert not overwritten_stores([head, store, "s_nop 1", "v_mul_f32_e32 v40, v22, v1"])[1]
    assert not overwritten_stores([head, store, "v_mul_f32_e32 v44, v40, v41", "s_nop 0", "v_mul_f32_e32 v40, v22, v1"])[1]
    assert overwritten_stores([head, "global_store_dwordx4 v0, v[4:7], s[0:1]", "v_mov_b32_e32 v5, 0"])[1]


def test_no_kernel_overwrites_the_data_of_a_wide_store(tmp_path):
    objdump = os.path.join(ROCM, "llvm", "bin", "llvm-objdump")
    shutil.copy(xnor._LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for obj in sorted(glob.glob(str(tmp_path / "*gfx950*"))):
        out = subprocess.Popen([objdump, "-d", obj], stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True)
        stores, bad = overwritten_stores(out.stdout)
        assert out.wait() == 0
        assert not bad, bad[:3]
        total += stores
    assert total > 0                                             # (the packers and the fully connected epilogue have some)
