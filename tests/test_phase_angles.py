"""Phase passes relative to the amplitude they rotate, where the span a thread
walks changes and on a state of one span.  Bar 1e-6: one FP32 rounding of the
folded angle (2^-26 turns, 9e-8 rad), sine and cosine within 2 ulp (1.7e-7
together) and three roundings of the rotation (1.8e-7), doubled."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 10, 20, 21, 22, 24, 25, 26])
def test_phase_angles(n):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    phases = [C.Gate((a, b), C.CP(float(rng.uniform(-3, 3)))) for a in range(n) for b in range(a)]
    phases += [C.Gate((q,), C.RZ(float(rng.uniform(-3, 3)))) for q in range(n)]
    st = sv.State(n)
    try:
        st.apply_circuit([C.Gate((q,), C.H) for q in range(n)], max_k=4)
        before = st.read().astype(np.complex128)
        assert st.apply_circuit(phases, max_k=2, fusion="phase", stats=True)["passes"] == 1
        got = st.read()
    finally:
        st.free()
    idx = np.concatenate([rng.integers(0, 1 << n, 4096), np.arange(min(4096, 1 << n)),
                          np.arange(max(0, (1 << n) - 4096), 1 << n)])
    ref = before[idx] * oracle.diagonal_factors(phases, idx)
    assert np.max(np.abs(got[idx] - ref) / np.abs(ref)) <= 1e-6
