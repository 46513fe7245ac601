"""Passes that fit one tile go out as one launch, in every precision, and as
one launch inside a graph; a forced variant and a timed call launch each pass
by itself."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


def pair(n, k, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    qs = [int(q) for q in rng.permutation(n)]
    return [C.Gate(tuple(qs[:k]), C.haar_unitary(k, rng)), C.Gate(tuple(qs[1:k + 1]), C.haar_unitary(k, rng))]


@pytest.mark.parametrize("precision", ["fp32_valu", "fp32_mfma", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("n", [12, 13, 21])
def test_two_passes_one_launch(n, k, precision):
    from paper_2602_09604_amd import sv
    if n > 12 and k == 6:
        pytest.skip("two such matrices fit a workgroup's LDS only beside a small tile")
    gates = pair(n, k, 100 * n + k)
    psi = C.random_state_c64(n, k)
    ref = oracle.apply_circuit(n, gates, psi=psi.astype(np.complex128))
    st = sv.State(n)
    try:
        for kw, launches in ((dict(), 1), (dict(use_graph=True), 1), (dict(timing=True), 2), (dict(variant="reg"), 2)):
            st.write(0, psi)
            s = st.apply_circuit(gates, fusion="none", precision=precision, stats=True, **kw)
            assert (s["passes"], s["launches"]) == (2, launches), kw
            assert np.max(np.abs(st.read() - ref)) <= (1e-4 if precision == "bf16x3" else 1e-5), kw
    finally:
        st.free()
