"""A Pauli term's value is its own: the same term on the same state rounds the
same alone, among terms with its flip mask, among many other masks, and past
the number of masks one launch sequence takes."""
import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 12, 17, 20, 23, 25])
def test_term_alone_and_in_company(n):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    flips = rng.integers(0, 1 << n, size=min(1 << n, 300), dtype=np.uint64)
    x = np.repeat(flips, rng.integers(1, 4, flips.size))
    z = rng.integers(0, 1 << n, size=x.size, dtype=np.uint64)
    st = sv.State(n)
    try:
        st.write(0, C.random_state_c64(n, n))
        every = st.expect_pauli(x, z)
        few = st.expect_pauli(x[:24], z[:24])
        assert np.array_equal(every[:24], few)
        for i in [0, 1, x.size // 2, x.size - 2, x.size - 1]:
            assert st.expect_pauli(x[i:i + 1], z[i:i + 1])[0] == every[i]
    finally:
        st.free()
