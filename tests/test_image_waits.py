"""The fused block kernels request a head's K~/V~ image in LDS at their very beginning and wait for it once, behind to_q. On every path of
the generated code the pieces have arrived before the LDS reads of the scores (K~ codes, the A operand of a product with Q~; the scales
and the bias, operands of an FMA), which are the image's first readers, and before the first exponential of the softmax, ahead of which
V~ may be read. No GPU: hipcc cross-compiles."""
import re

import pytest

from test_waits import assembly


def exponentials_with_lds_loads_in_flight(body):
    """Exponentials that a path reaches with a direct-to-LDS load possibly outstanding (vector memory operations complete in order as
    far as vmcnt tells: one is done when at most as many are outstanding as were issued after it)."""
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
            elif op.startswith("buffer_load") and text.endswith(" lds"):
                since = 0
            elif since is not None and re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", op):
                since = min(since + 1, 64)
            elif op == "v_exp_f32_e32" and since is not None:
                bad.add(no)
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op == "s_branch":
                i = label[text.split()[1]]
                continue
            if op.startswith("s_cbranch"):
                work.append((label[text.split()[1]], since))
            i += 1
    return sorted(bad)


PLANTED = [(1, "buffer_load_dwordx4 v1, s[0:3], 0 offen lds", False), (2, "buffer_load_dwordx4 v[2:5], v1, s[0:3], 0 offen", False),
           (3, "{}", True), (4, "v_exp_f32_e32 v6, v6", False), (5, "s_endpgm", False)]


@pytest.mark.parametrize("wait,found", [("s_waitcnt vmcnt(0)", 0), ("s_waitcnt vmcnt(1)", 0), ("s_waitcnt vmcnt(2)", 1), ("s_nop 0", 1)])
def test_the_check_sees_a_planted_gap(wait, found):
    assert len(exponentials_with_lds_loads_in_flight([(n, t.format(wait), h) for n, t, h in PLANTED])) == found


@pytest.mark.parametrize("source", ["taq_fused_d40.hip", "taq_fused_d64.hip", "taq_fused_d80.hip"])
def test_the_image_has_arrived(tmp_path, source):
    bodies = {k: b for k, b in assembly(source, tmp_path).items() if "fused_block_kernel" in k}
    assert bodies and all(any(t.startswith("buffer_load") and t.endswith(" lds") for _, t, _ in b) for b in bodies.values())
    bad = {k: exponentials_with_lds_loads_in_flight(b) for k, b in bodies.items() if exponentials_with_lds_loads_in_flight(b)}
    assert not bad, bad


REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def names(operand):
    """Vector registers of an operand, or of several."""
    return [f"{kind}{i}" for kind, one, lo, hi in REG.findall(operand) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)])]


def score_reads(body):
    """(products of the scores, their lines and those of score FMAs with an operand that was read from LDS while a direct-to-LDS load was
    possibly outstanding). A product of the scores is an int8 one whose B operand (Q~) was computed; that of to_q and to_out (token codes)
    is read from LDS. State: vector memory operations since the last LDS load, the fewest; registers that hold what an LDS read gave;
    those of them that were read too early; over all paths."""
    label = {text[:-1]: i for i, (_, text, _) in enumerate(body) if text.endswith(":")}
    seen = [None] * len(body)
    work, scores, bad = [(0, None, frozenset(), frozenset())], set(), set()
    while work:
        i, since, read, early = work.pop()
        while i < len(body):
            if seen[i] is not None:
                s0, r0, e0 = seen[i]
                both = [x for x in (since, s0) if x is not None]
                since, read, early = (min(both) if both else None), read | r0, early | e0
                if (since, read, early) == seen[i]:
                    break
            seen[i] = (since, read, early)
            no, text, _ = body[i]
            op, *rest = text.split(None, 1)
            args = [a.strip() for a in rest[0].split(",")] if rest else []
            count = re.search(r"vmcnt\((\d+)\)", text) if op == "s_waitcnt" else None
            if count and since is not None and int(count.group(1)) <= since:
                since = None
            elif op.startswith("buffer_load") and text.endswith(" lds"):
                since = 0
            elif since is not None and re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", op):
                since = min(since + 1, 64)
            if op == "v_mfma_i32_16x16x64_i8" and not read & set(names(args[2])):
                scores.add(no)
                if early & set(names(args[1])):
                    bad.add(no)
            if re.match(r"v_(pk_)?fma", op) and early & set(names(",".join(args[1:]))):
                bad.add(no)
            if args and not op.startswith("s_") and not text.endswith(" lds") and not re.match(r"(ds_write|(global|buffer|flat|scratch)_store)", op):
                into = names(args[0])
                if op.startswith("ds_read"):
                    read, early = read | set(into), early | set(into) if since is not None else early - set(into)
                elif op in ("v_mov_b32_e32", "v_accvgpr_write_b32", "v_accvgpr_read_b32", "v_accvgpr_mov_b32"):
                    source = names(args[1])
                    read = read | set(into) if source and source[0] in read else read - set(into)
                    early = early | set(into) if source and source[0] in early else early - set(into)
                else:
                    read, early = read - set(into), early - set(into)
            if op in ("s_endpgm", "s_setpc_b64"):
                break
            if op == "s_branch":
                i = label[text.split()[1]]
                continue
            if op.startswith("s_cbranch"):
                work.append((label[text.split()[1]], since, read, early))
            i += 1
    return scores, sorted(bad)


SCORES = """buffer_load_dwordx4 v1, s[0:3], 0 offen lds
ds_read_b128 v[20:23], v2
v_mfma_i32_16x16x64_i8 v[30:33], v[60:63], v[20:23], 0
v_cvt_f32_i32_e32 v40, v30
{}
ds_read_b128 v[24:27], v3
{}
ds_read_b32 v50, v3 offset:64
{}
v_mfma_i32_16x16x64_i8 v[34:37], v[24:27], v[40:43], 0
v_fma_f32 v38, v34, v50, v51
s_endpgm"""


@pytest.mark.parametrize("where,found", [(0, 0), (1, 1), (2, 2)])
def test_the_check_sees_an_early_read(where, found):
    text = SCORES.format(*("s_waitcnt vmcnt(0)" if k == where else "s_nop 0" for k in range(3)))
    scores, bad = score_reads([(n, t, False) for n, t in enumerate(text.split("\n"), 1)])
    assert len(scores) == 1 and len(bad) == found


@pytest.mark.parametrize("source", ["taq_fused_d40.hip", "taq_fused_d64.hip", "taq_fused_d80.hip"])
def test_the_scores_read_an_image_that_has_arrived(tmp_path, source):
    for name, body in assembly(source, tmp_path).items():
        if "fused_block_kernel" in name:
            scores, bad = score_reads(body)
            products = sum(t.startswith("v_mfma_i32_16x16x64_i8") for _, t, _ in body)
            assert len(scores) >= 5 and products >= 2 * len(scores), (name, len(scores), products)
            assert not bad, (name, bad[:4])
