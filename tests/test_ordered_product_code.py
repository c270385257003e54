"""The ordered product reads LDS through inline assembly a few steps ahead of the instruction that needs the values, so the
compiler takes a register as written when the read is issued.  In the compiled kernel nothing may touch such a register
before the wait that covers its read, and no branch or label may stand between the two: a value that crosses a branch may be
copied there, and a copy of what has not arrived is a copy of something else."""
import os
import re
import subprocess

import pytest

from paper_2109_15082_amd import build

SPLIT = '#include "mrem_gemm_quad.h"'


def registers(text):
    regs = set()
    for lo, hi, one in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+))\b", text):
        regs |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return regs


def in_flight(lines):
    """(reads, offending lines) of a kernel's body; LDS reads return in order, lgkmcnt counts those still on their way"""
    flying, reads, bad = [], 0, []
    for raw in lines:
        line = raw.split(";")[0].strip()
        wait = re.match(r"s_waitcnt.*lgkmcnt\((\d+)\)", line)
        read = re.match(r"ds_read_u16_d16_hi (v\d+),", line)
        if wait:
            flying = flying[-int(wait[1]):] if int(wait[1]) else []
        elif read:
            bad += [line] if any(f & registers(line) for f in flying) else []
            flying.append(registers(read[1]))
            reads += 1
        elif flying and (re.match(r"s_c?branch|\.LBB", line) or any(f & registers(line) for f in flying)):
            bad.append(line)
    return reads, bad


def test_nothing_touches_a_value_on_its_way(tmp_path):
    source = open(os.path.join(build.CSRC, "mrem_gemm.hip")).read()
    assert source.count(SPLIT) == 1
    probe = tmp_path / "ordered.hip"
    probe.write_text(source.split(SPLIT)[0] + '#include "mrem_gemm_chain.h"\nnamespace mrem {\nvoid ordered(const void* A, const void* B, void* C, int M, '
                     "int N, int K, const Epilogue& e, hipStream_t st) { launch_chain(A, K, B, K, C, N, M, N, K, e, st); }\n}\n")
    out = tmp_path / "ordered.s"
    r = subprocess.run([build.hipcc(), *build.FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(probe), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    asm = out.read_text().split("\n")
    kernels = [i for i, line in enumerate(asm) if re.match(r"\w*gemm_chain_k\w*:", line)]
    assert len(kernels) >= 2
    for k in kernels:
        end = next(i for i in range(k, len(asm)) if asm[i].startswith(".Lfunc_end"))
        reads, bad = in_flight(asm[k + 1:end])
        assert reads > 0 and not bad, (asm[k], bad[:4])


@pytest.mark.parametrize("line", ["v_mov_b32_e32 v9, v3", "ds_read_u16_d16_hi v5, v3", "s_cbranch_scc1 .LBB0_3", ".LBB0_2:"])
def test_the_check_sees(line):
    body = ["ds_read_u16_d16_hi v3, v8 offset:16", "ds_read_u16_d16_hi v4, v8", "s_waitcnt lgkmcnt({})", line]
    reads = 2 + line.startswith("ds_read")
    assert in_flight([b.format(1) for b in body]) == (reads, [] if "v3" in line else [line])
    assert in_flight([b.format(2) for b in body]) == (reads, [line])
    assert in_flight([b.format(0) for b in body]) == (reads, [])
