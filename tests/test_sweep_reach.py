"""How far an infinite or NaN amplitude reaches in a tile sweep: a pass mixes
the 2^k amplitudes of a group and no others, so after several passes only the
amplitudes that share groups with the bad one may be spoiled.  The others keep
their value to FP32 rounding (1e-5, as for finite states; 1e-4 in BF16X3)."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("n,precision", [(9, "fp32_valu"), (12, "fp32_valu"), (14, "fp32_valu"), (21, "fp32_valu"),
                                         (12, "bf16x3"), (22, "bf16x3")])
def test_bad_amplitude_stays_in_its_groups(n, precision, k, bad):
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(10 * n + k))
    sets = [tuple(int(q) for q in rng.permutation(6)[:k]) for _ in range(3)]
    gates = [C.Gate(qs, C.haar_unitary(k, rng)) for qs in sets]
    psi = C.random_state_c64(n, n + k)
    at = int(rng.integers(1 << n))
    psi[at] = bad
    st = sv.State(n)
    try:
        st.write(0, psi)
        s = st.apply_circuit(gates, fusion="none", precision=precision, stats=True)
        got = st.read()
    finally:
        st.free()
    assert s["launches"] < len(gates)
    spoiled = {at}
    for qs in sets:
        for q in qs:
            spoiled |= {i ^ (1 << q) for i in spoiled}
    keep = np.setdiff1d(np.arange(1 << n), sorted(spoiled))
    clean = psi.copy()
    clean[at] = 0
    ref = oracle.apply_circuit(n, gates, psi=clean.astype(np.complex128))
    assert np.all(np.isfinite(got[keep])), np.flatnonzero(~np.isfinite(got[keep])).size
    assert np.max(np.abs(got[keep] - ref[keep])) <= (1e-4 if precision == "bf16x3" else 1e-5)
