"""Waits that the compiler does not place by itself, checked on the generated assembly of every kernel, over all paths. No GPU:
hipcc cross-compiles.

LDS reads written as inline asm (csrc/taq_gemm_op.h): the compiler takes their results to be there at once, so between such a
read and the wait for it no instruction may touch its destination registers, neither the arithmetic that uses the operands nor
anything the compiler places into registers it believes free.

Loads from global memory straight into LDS that other wavefronts read (csrc/taq_attn.hip, csrc/taq_quant.hip): a wavefront has to
wait for its own ones before the barrier; the barrier alone does not."""
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


ASSEMBLED = {}  # (a source takes up to 40 s)


def assembly(source, tmp_path):
    if source in ASSEMBLED:
        return ASSEMBLED[source]
    out = str(tmp_path / (source + ".s"))
    include = os.path.join(os.path.dirname(B.HERE), "include")
    r = subprocess.run([B.hipcc_path()] + DEVICE_FLAGS + ["-I", include, os.path.join(B.CSRC, source), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    ASSEMBLED[source] = kernels(open(out).read())
    return ASSEMBLED[source]


def test_no_register_of_a_read_in_flight_is_touched(tmp_path):
    bodies = {k: b for k, b in assembly("taq_gemm.hip", tmp_path).items() if any(h and t.startswith("ds_read") for _, t, h in b)}
    assert len(bodies) == 22  # every instantiation of gemm_op_kernel
    bad = {k: touched_in_flight(b)[:4] for k, b in bodies.items() if touched_in_flight(b)}
    assert not bad, "\n".join(f"{k}: {v}" for k, v in bad.items())


def barriers_with_lds_loads_in_flight(body):
    """Barriers that a path reaches with a direct-to-LDS load of its own possibly outstanding. Vector memory operations complete
    in order as far as vmcnt tells: one is done when at most as many are outstanding as were issued after it."""
    label = {text[:-1]: i for i, (_, text, _) in enumerate(body) if text.endswith(":")}
    seen = [()] * len(body)  # () not reached; None: nothing in flight; n: operations issued since the last such load, the fewest
    work, bad = [(0, None)], set()
    while work:
        i, since = work.pop()
        while i < len(body):
            if seen[i] != ():
                both = [x for x in (since, seen[i]) if x is not None]
                since = min(both) if both else None
                if since == seen[i]:
                    break
            seen[i] = since
            no, text, _ = body[i]
            op = text.split()[0]
            count = re.search(r"vmcnt\((\d+)\)", text) if op == "s_waitcnt" else None
            if count and since is not None and int(count.group(1)) <= since:
                since = None
            elif "load_lds" in op:
                since = 0
            elif since is not None and re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", op):
                since += 1
            elif op == "s_barrier" and since is not None:
                bad.add(no)
            if since is not None:
                since = min(since, 64)
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op == "s_branch":
                i = label[text.split()[1]]
                continue
            if op.startswith("s_cbranch"):
                work.append((label[text.split()[1]], since))
            i += 1
    return sorted(bad)


LDS_LOAD = """
_Zk:
	global_load_lds_dwordx4 v[0:1], off
	global_load_dword v4, v[0:1], off
	s_cbranch_scc1 .LBB0_2
	{wait}
.LBB0_2:
	{then}
	s_barrier
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("wait,then,found", [("s_waitcnt vmcnt(0)", "s_nop 0", 1), ("s_nop 0", "s_waitcnt vmcnt(1)", 0),
                                             ("s_nop 0", "s_waitcnt vmcnt(2)", 1), ("s_nop 0", "s_waitcnt vmcnt(0) lgkmcnt(0)", 0)])
def test_the_barrier_check_sees_a_planted_gap(wait, then, found):
    assert len(barriers_with_lds_loads_in_flight(kernels(LDS_LOAD.format(wait=wait, then=then))["_Zk"])) == found


@pytest.mark.parametrize("source,count", [("taq_attn.hip", 90), ("taq_quant.hip", 10)])
def test_lds_loads_have_arrived_at_the_barrier(tmp_path, source, count):
    bodies = {k: b for k, b in assembly(source, tmp_path).items() if any("load_lds" in t for _, t, _ in b)}
    assert len(bodies) == count
    bad = {k: barriers_with_lds_loads_in_flight(b) for k, b in bodies.items() if barriers_with_lds_loads_in_flight(b)}
    assert not bad, bad
    # ... and not by luck of the schedule: the source waits itself between the loads and the barrier
    text = open(os.path.join(B.CSRC, source)).read()
    at = text.index("__builtin_amdgcn_global_load_lds")
    wait = text.find("__builtin_amdgcn_s_waitcnt(0x0F70)", at)
    assert 0 < wait < text.index("__syncthreads()", at), "no explicit wait between the loads and the barrier"
