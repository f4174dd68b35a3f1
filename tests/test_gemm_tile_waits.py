"""As tests/test_waits.py for the sources that instantiate gemm_op_kernel besides taq_gemm.hip: no register of a read in flight is
touched (the compiler takes the reads written by hand to be there at once)."""
import pytest

from test_waits import assembly, touched_in_flight


@pytest.mark.parametrize("source,kernels", [("taq_gemm_rows.hip", 22), ("taq_gemm_out.hip", 6)])
def test_no_register_of_a_read_in_flight_is_touched(source, kernels, tmp_path):
    bodies = {k: b for k, b in assembly(source, tmp_path).items() if any(h and t.startswith("ds_read") for _, t, h in b)}
    assert len(bodies) == kernels
    bad = {k: touched_in_flight(b)[:4] for k, b in bodies.items() if touched_in_flight(b)}
    assert not bad, "\n".join(f"{k}: {v}" for k, v in bad.items())
