"""A 16-deep fp16 product that goes on with the sums of a 32-deep one (csrc/taq_device.h, sums_settle) needs wait states in between that
the compiler does not place: on the generated code of every kernel, in program order. No GPU."""
import re

import pytest

from test_waits import assembly, kernels

DEEP, SHALLOW = "v_mfma_f32_16x16x32_f16", "v_mfma_f32_16x16x16_f16"
WAIT = 8


def too_close(body):
    """(line, wait states) of 16-deep products closer than WAIT wait states to the 32-deep product that wrote their sums."""
    written, at, bad = {}, 0, []  # register: (instruction, wait states up to it)
    for no, text, _ in body:
        if text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        at += int(rest) + 1 if op == "s_nop" else 1
        regs = [(int(a), int(b or a)) for a, b in re.findall(r"\bv\[?(\d+)(?::(\d+))?\]?", rest)]
        if op == SHALLOW and len(regs) == 4:
            deep = [at - when - 1 for r in range(regs[3][0], regs[3][1] + 1) for by, when in [written.get(r, ("", 0))] if by == DEEP]
            if deep and min(deep) < WAIT:
                bad.append((no, min(deep)))
        if regs and not op.startswith(("s_", "ds_write", "global_store", "buffer_store")):
            for r in range(regs[0][0], regs[0][1] + 1):
                written[r] = (op, at)
    return bad


def unguarded(body):
    """Lines of 16-deep products without wait states of our own since a 32-deep product that wrote their sums: whatever else stands in
    between is there by the compiler's choice."""
    written, bad = {}, []  # register: (instruction, whether a hand-written s_nop 7 came behind it)
    for no, text, by_hand in body:
        op, _, rest = text.partition(" ")
        regs = [(int(a), int(b or a)) for a, b in re.findall(r"\bv\[?(\d+)(?::(\d+))?\]?", rest)]
        if by_hand and text == "s_nop 7":
            written = {r: (by, True) for r, (by, _) in written.items()}
        if op == SHALLOW and len(regs) == 4:
            if any(written.get(r, ("", True)) == (DEEP, False) for r in range(regs[3][0], regs[3][1] + 1)):
                bad.append(no)
        if regs and not text.endswith(":") and not op.startswith(("s_", "ds_write", "global_store", "buffer_store")):
            for r in range(regs[0][0], regs[0][1] + 1):
                written[r] = (op, False)
    return bad


PLANTED = """
_Zk:
	v_mfma_f32_16x16x32_f16 v[0:3], v[8:11], v[12:15], v[0:3]
	{between}
	v_mfma_f32_16x16x16_f16 v[0:3], v[8:9], v[12:13], v[0:3]
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("between,found", [("s_waitcnt lgkmcnt(0)", 1), ("s_nop 7", 0), ("s_nop 6", 1), ("v_mov_b32_e32 v0, v1\n\tv_mov_b32_e32 v1, v0", 1)])
def test_the_check_sees_a_planted_gap(between, found):
    assert len(too_close(kernels(PLANTED.format(between=between))["_Zk"])) == found


@pytest.mark.parametrize("between,found", [("s_nop 7", 1), (";#ASMSTART\n\ts_nop 7\n\t;#ASMEND", 0), ("\n\t".join(["v_mov_b32_e32 v20, v21"] * 20), 1)])
def test_the_check_sees_what_only_the_compiler_placed(between, found):
    assert len(unguarded(kernels(PLANTED.format(between=between))["_Zk"])) == found


@pytest.mark.parametrize("source", ["taq_heads160.hip", "taq_heads64.hip", "taq_heads80.hip", "taq_heads64x10.hip", "taq_attn.hip", "taq_fused_d40.hip",
                                    "taq_fused_d80.hip", "taq_fused_d64.hip"])
def test_sums_have_settled(source, tmp_path):
    bodies = assembly(source, tmp_path)
    assert any(text.startswith(SHALLOW) for body in bodies.values() for _, text, _ in body)
    bad = {k: too_close(b) for k, b in bodies.items() if too_close(b)}
    assert not bad, bad
    bad = {k: unguarded(b) for k, b in bodies.items() if unguarded(b)}
    assert not bad, bad
