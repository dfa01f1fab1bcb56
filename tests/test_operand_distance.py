"""Distance the compiler keeps behind the fp32 matrix instruction, read from the library as built.

v_mfma_f32_16x16x4_f32 reads the four registers of its C operand one after the other.  Where the destination is another
set of registers, those of C are free for the compiler at once, and it keeps no distance to a vector instruction that
writes them (it does for the bf16 instructions: seven instructions for those of the same length).  Measured: a v_mul_f32
into the third register as the next instruction gave wrong sums, and others from run to run.  The kernels keep vector
instructions out of such places; this test looks whether the code they compiled to does."""
import os
import re
import subprocess

import pytest

from paper_2506_01380_amd import binding as nb

LLVM = "/opt/rocm/llvm/bin"
MIN_DISTANCE = 8


def _registers(text):
    m = re.match(r"v\[(\d+):(\d+)\]$", text)
    if m:
        return list(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)$", text)
    return [int(m[1])] if m else []


def hazards(lines):
    """(function, instruction, writer) of every vector write that comes too early.  Each instruction counts one, s_nop n
    n + 1; what follows a branch in the listing is taken to follow it in time."""
    code, function, found = [], None, []
    for line in lines:
        m = re.match(r"(?:[0-9a-f]+ )?<(.+)>:$", line.strip())
        if m:
            function = m[1]
            continue
        text = line.split("//")[0].strip()
        if text and function:
            code.append((function, text))
    for n, (function, text) in enumerate(code):
        if not text.startswith("v_mfma_f32_16x16x4_f32"):
            continue
        ops = [o.strip() for o in text.split(None, 1)[1].split(",")]
        dst, c = _registers(ops[0]), _registers(ops[3])
        if not c or c == dst:
            continue
        distance = 0
        for other, follower in code[n + 1:n + 1 + MIN_DISTANCE]:
            op, _, rest = follower.partition(" ")
            if distance >= MIN_DISTANCE or other != function:
                break
            if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readfirstlane", "v_nop")):
                if set(_registers(rest.split(",")[0].strip())) & set(c):
                    found.append((function, text, follower))
            distance += 1 + int(rest) if op == "s_nop" else 1
    return found


def test_the_search_finds_an_early_write():
    listing = """<k>:
	v_mfma_f32_16x16x4_f32 v[136:139], v66, v30, v[126:129]
	v_mul_f32_e32 %s, s36, v132
"""
    assert len(hazards((listing % "v128").splitlines())) == 1
    assert not hazards((listing % "v125").splitlines()) and not hazards((listing % "v136").splitlines())
    assert not hazards((listing % "v128").replace("\tv_mul", "\ts_nop 7\n\tv_mul").splitlines())
    assert not hazards((listing % "v128").replace("v[136:139]", "v[126:129]").splitlines())


def test_no_vector_write_close_behind_a_matrix_instruction(tmp_path):
    if not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("no disassembler")
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.check_call([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, nb.LIB_PATH, str(tmp_path / "rest")])
    subprocess.check_call([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                           "--input=" + bundle, "--output=" + code])
    listing = subprocess.check_output([LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", code], text=True)
    assert listing.count("v_mfma_f32_16x16x4_f32") > 1000
    assert not hazards(listing.splitlines())
