"""Pauli sums of many flip masks: more sweeps than one launch's arguments
hold, more than one call's scratch, every class of terms per sweep, and the
states where a sweep has one workgroup.  Bar: 1e-12 (FP64 sums of exact
products), as for single sweeps."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,flips", [(1, 2), (2, 4), (3, 8), (9, 300), (10, 520), (16, 40), (21, 12)])
def test_pauli_many_sweeps(n, flips):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    f = rng.permutation(1 << n)[:flips]
    x = np.concatenate([np.full(int(c), v, dtype=np.uint64) for v, c in zip(f, rng.integers(1, 10, f.size))])
    x = x[rng.permutation(x.size)]
    z = rng.integers(0, 1 << n, size=x.size, dtype=np.uint64)
    psi = C.random_state_c64(n, 5 + n)
    st = sv.State(n)
    try:
        st.write(0, psi)
        got = st.expect_pauli(x, z)
    finally:
        st.free()
    pick = rng.permutation(x.size)[:200 if n < 16 else 20]
    ref = np.array([oracle.pauli_expectation(psi.astype(np.complex128), n, int(x[i]), int(z[i])).real for i in pick])
    assert np.max(np.abs(got[pick] - ref)) < 1e-12
