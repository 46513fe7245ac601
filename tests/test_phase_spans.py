"""Phase passes where the span a thread walks changes: a whole state in one
span (20 qubits), the smallest split (21), and spans of a sixteenth of the
state (24, 25), every pair of qubits interacting.  Bar: max |delta| <= 1e-6
from the uniform superposition (amplitudes 2^(-n/2) <= 1e-3, angles rounded
once to FP32)."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [20, 21, 24, 25])
def test_phase_spans_every_pair(n):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    phases = [C.Gate((a, b), C.CP(float(rng.uniform(-3, 3)))) for a in range(n) for b in range(a)]
    phases += [C.Gate((q,), C.RZ(float(rng.uniform(-3, 3)))) for q in range(n)]
    st = sv.State(n)
    try:
        st.apply_circuit([C.Gate((q,), C.H) for q in range(n)], max_k=4)
        before = st.read().astype(np.complex128)
        st.apply_circuit(phases, max_k=2, fusion="phase")
        got = st.read()
    finally:
        st.free()
    idx = np.concatenate([rng.integers(0, 1 << n, 4096), np.arange(4096), np.arange((1 << n) - 4096, 1 << n)])
    ref = before[idx] * oracle.diagonal_factors(phases, idx)
    assert np.max(np.abs(got[idx] - ref)) <= 1e-6
