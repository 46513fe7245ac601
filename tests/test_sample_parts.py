"""Sampling where its chunks and parts change: one chunk smaller than a lane's
eight amplitudes, one part, two and eight parts, and several chunks, on states
with long runs of zeros and with the weight at either end."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 9, 10, 12, 13, 15, 18])
@pytest.mark.parametrize("shape", ["dense", "sparse", "first", "last"])
def test_sample_parts(n, shape):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    psi = C.random_state_c64(n, 70 + n)
    if shape == "sparse":
        psi[rng.random(1 << n) < 0.99] = 0
        psi[int(rng.integers(1 << n))] = 0.5
    elif shape in ("first", "last"):
        psi[:] = 0
        psi[0 if shape == "first" else -1] = 1
    st = sv.State(n)
    try:
        st.write(0, psi)
        u = np.concatenate([C.uniforms(500, n), [0.0, np.nextafter(1.0, 0.0)]])
        got = st.sample(u)
    finally:
        st.free()
    ref = oracle.sample_indices(psi.astype(np.complex128), u)
    assert np.array_equal(got, ref)
