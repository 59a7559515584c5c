"""The attention kernel's matrix instructions written in asm: the compiler does
not know their wait states, so its own instructions must not touch an
accumulation register within 18 wait states of one that writes it (it might copy
one, were it to allocate them differently), and nothing may be spilled to
memory (the kernel counts its own loads).  Checked on the assembly of the
source as the build compiles it.  Likewise for its loads in asm: a vector
instruction may have written a scalar register that such a load reads (the
reload of a spilled one does) right before the block, and the load has to be
five wait states behind it."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2408_03675_amd import build

WAIT = 18  # wait states after a 32x32x16 MFMA


def _registers(text):
    out = set()
    for a, b in re.findall(r"\ba\[(\w+):(\w+)\]", text):
        out |= set(range(int(a, 0), int(b, 0) + 1))
    for a in re.findall(r"\ba\[(\w+)\]|\ba(\d+)\b", text):
        out.add(int(a[0] or a[1], 0))
    return out


def _violations(asm):
    """Instructions that touch an accumulation register too early.  Each one
    issued counts as one wait state (s_nop n as n + 1), and a block entered by a
    branch is taken to follow the code above it."""
    bad, blocks, in_asm, age = [], 0, False, {}
    for line in asm.splitlines():
        if "ASMSTART" in line or "ASMEND" in line:
            in_asm = "ASMSTART" in line
            continue
        t = line.split(";")[0].strip()
        if re.match(r"_Z\w+:", t):
            age = {}
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        regs = _registers(t)
        if in_asm and t.startswith("v_mfma"):
            blocks += 1
            dst = _registers(t.split(",")[0])
            if any(r in age for r in _registers(",".join(t.split(",")[1:3]))):
                bad.append(t)
            age = {r: n + 1 for r, n in age.items()}
            age.update({r: 0 for r in dst})
            continue
        if any(age.get(r, WAIT) < WAIT for r in regs):
            bad.append(t)
        m = re.match(r"s_nop (\d+)", t)
        step = int(m.group(1)) + 1 if m else 1
        age = {r: n + step for r, n in age.items() if n + step < 64}
        if t.startswith(("s_cbranch", "s_branch")) and any(n < WAIT for n in age.values()):
            bad.append("a branch " + t)
    return bad, blocks


def _load_waits(asm):
    """Wait states inside each asm block ahead of its buffer load."""
    out, waits = [], None
    for line in asm.splitlines():
        if "ASMSTART" in line:
            waits = 0
        elif "ASMEND" in line:
            waits = None
        elif waits is not None:
            t = line.split(";")[0].strip()
            if t.startswith("buffer_load"):
                out.append(waits)
            m = re.match(r"s_nop (\d+)", t)
            waits += int(m.group(1)) + 1 if m else bool(t)
    return out


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("asm") / "attention.s"
    cmd = [build._hipcc()] + build.HIP_FLAGS + build.SOURCE_FLAGS["attention.hip"] + [
        "--cuda-device-only", "-S", "-x", "hip", os.path.join(build.CSRC, "attention.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def test_check_finds_an_early_copy():
    mfma = ";;#ASMSTART\nv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n;;#ASMEND\n"
    assert _violations(mfma + "v_accvgpr_mov_b32 a40, a3\n")[0]
    assert _violations(mfma + "s_nop 15\nv_accvgpr_read_b32 v1, a[0x3]\n")[0]
    assert not _violations(mfma + "s_nop 15\ns_nop 15\nv_accvgpr_read_b32 v1, a3\n")[0]
    assert not _violations(mfma + mfma)[0]


def test_accumulators_are_left_alone(assembly):
    bad, blocks = _violations(assembly)
    assert blocks == 64  # two steps of 32 value products
    assert not bad, bad[:5]
    assert "scratch_" not in assembly


def test_loads_wait_for_their_scalar_registers(assembly):
    waits = _load_waits(assembly)
    assert waits and min(waits) >= 5
