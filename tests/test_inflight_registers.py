"""LDS reads written as inline asm (csrc/taq_gemm.hip): the compiler takes their results to be there at once, so between such a
read and the wait for it no instruction may touch its destination registers, neither the arithmetic that uses the operands nor
anything the compiler places into registers it believes free. Checked on the generated assembly of every kernel, over all paths.
No GPU: hipcc cross-compiles."""
import os
import re
import subprocess

import pytest

from paper_2603_22943_amd import build as B

REG = re.compile(r"\bv(?:(\d+)\b|\[(\d+):(\d+)\])")
DEVICE_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
                "-fno-honor-nans", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S"]


def registers(text):
    out = set()
    for one, lo, hi in REG.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def kernels(asm):
    """{name: [(line number, instruction or label, written by hand)]} of every kernel in an assembly file."""
    found, name, body, by_hand = {}, None, [], False
    for no, line in enumerate(asm.splitlines(), 1):
        start = re.match(r"(_Z\w+):", line)
        if start:
            name, body = start.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            found[name], name = body, None
        elif name:
            by_hand = (by_hand or "#ASMSTART" in line) and "#ASMEND" not in line
            text = line.split(";")[0].strip()
            if text and (text.endswith(":") or not text.startswith(".")):
                body.append((no, text, by_hand))
    return found


def touched_in_flight(body):
    """Instructions that name a register which a read written by hand may still write, over all paths through the kernel."""
    label = {text[:-1]: i for i, (_, text, _) in enumerate(body) if text.endswith(":")}
    pending = [None] * len(body)  # registers in flight in front of an instruction, over the paths seen so far
    work, bad = [(0, frozenset())], {}
    while work:
        i, regs = work.pop()
        while i < len(body):
            if pending[i] is not None and regs <= pending[i]:
                break
            pending[i] = regs = regs | (pending[i] or frozenset())
            no, text, by_hand = body[i]
            op = text.split()[0]
            if op == "s_waitcnt" and ("lgkmcnt(0)" in text or text.split()[1:] == ["0"]):
                regs = frozenset()
            elif not text.endswith(":") and not op.startswith("s_"):
                if registers(text) & regs:
                    bad[no] = text
                if by_hand and op.startswith("ds_read"):
                    regs = regs | registers(text.split(",")[0])
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op == "s_branch":
                i = label[text.split()[1]]
                continue
            if op.startswith("s_cbranch"):
                work.append((label[text.split()[1]], regs))
            i += 1
    return sorted(bad.items())


PLANTED = """
_Zk:
	v_mov_b32 v9, 0
.LBB0_1:
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	v_add_u32 v8, v0, v1
	;;#ASMSTART
	ds_read_b128 v[0:3], v9 offset:16
	;;#ASMEND
	ds_read_b32 v7, v9
	v_add_u32 v8, v8, v7
	s_cbranch_scc1 .LBB0_1
	{between}
	;;#ASMSTART
	s_waitcnt lgkmcnt(0)
	;;#ASMEND
	v_mov_b32 v2, v9
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("between,found", [("v_mov_b32 v4, v8", 0), ("v_mov_b32 v2, v8", 1), ("global_store_dwordx2 v[4:5], v[2:3], off", 1)])
def test_the_check_sees_a_planted_touch(between, found):
    assert len(touched_in_flight(kernels(PLANTED.format(between=between))["_Zk"])) == found


def test_no_register_of_a_read_in_flight_is_touched(tmp_path):
    out = str(tmp_path / "gemm.s")
    include = os.path.join(os.path.dirname(B.HERE), "include")
    r = subprocess.run([B.hipcc_path()] + DEVICE_FLAGS + ["-I", include, os.path.join(B.CSRC, "taq_gemm.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    bodies = {k: b for k, b in kernels(open(out).read()).items() if any(h and t.startswith("ds_read") for _, t, h in b)}
    assert len(bodies) == 22  # every instantiation of gemm_op_kernel
    bad = {k: touched_in_flight(b)[:4] for k, b in bodies.items() if touched_in_flight(b)}
    assert not bad, "\n".join(f"{k}: {v}" for k, v in bad.items())
