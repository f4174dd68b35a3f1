"""The fused block kernels request a head's K~/V~ image in LDS at their very beginning and wait for it once, behind to_q: on every path
of the generated code the pieces have arrived before the first exponential of the softmax (the scores, which read the K~ part, stand
between that wait and the exponentials). No GPU: hipcc cross-compiles."""
import re

import pytest

from tests.test_waits import assembly


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
