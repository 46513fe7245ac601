"""A tuning table's choice for a pass launched by itself is kept, also where
the untuned default is a tile sweep (k >= 5): the amplitudes are those of the
chosen kernel bit for bit, and equal the oracle's to 1e-5."""
import json

import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12, 20, 22])
@pytest.mark.parametrize("k,code,variant", [(5, 1, "reg"), (5, 2, "lds"), (6, 2, "lds")])
def test_table_decides_a_single_pass(tmp_path, n, k, code, variant):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n + k))
    qs = tuple(range(n - k, n))  # no target below bit 6: class (precision, k, 0, 0)
    assert qs[0] >= 6
    gate = C.Gate(qs, C.haar_unitary(k, rng))
    psi = C.random_state_c64(n, n)
    p = tmp_path / "t.json"
    p.write_text(json.dumps({"format": "libsv-tune-1",
                             "entries": [[0, k, 0, sum(1 <= q < 7 for q in qs), code, 10, 1.0]]}))
    sv.sv_tune_load(str(p))
    st = sv.State(n)
    try:
        out = []
        for v in (variant, "auto"):
            st.write(0, psi)
            st.apply_circuit([gate], fusion="none", variant=v)
            out.append(st.read())
        st.write(0, psi)
        st.apply_gate(qs, gate.matrix)
        out.append(st.read())
    finally:
        st.free()
    ref = oracle.apply_circuit(n, [gate], psi=psi.astype(np.complex128))
    assert np.max(np.abs(out[0] - ref)) <= 1e-5
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
