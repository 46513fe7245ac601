"""Tile sweeps (several passes in one trip through memory) against the CPU
complex128 oracle, at the sizes where the tile changes: the smallest (one unit
of a k = 4 pass), a whole state in one tile, the first states of several
tiles, and a streamed state.

Bar: max |delta amplitude| <= 1e-5 and infidelity <= 1e-6 (complex64 state,
FP32 arithmetic, a few hundred passes), as for the single passes; BF16 splits
carry 16 bits, so on the smallest states, whose amplitudes are large, their
amplitudes are held to 2^-16 times the root of the pass count."""
import numpy as np
import pytest

import circuits as C
import oracle

pytestmark = pytest.mark.gpu

MAX_ABS, INFID = 1e-5, 1e-6


def mixed_circuit(n, gates, max_k, seed):
    """Gates of every size, in random order of qubits, diagonal ones and
    controlled ones (passes of their own that a sweep may not pass by) among
    them."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = [C.Gate((q,), C.H) for q in range(n)]
    for i in range(gates):
        k = int(rng.integers(1, min(max_k, n) + 1))
        qs = tuple(int(v) for v in rng.permutation(n)[:k + 1])
        if i % 11 == 5 and n > k + 1:
            out.append(C.Gate(qs[:k], C.haar_unitary(k, rng), qs[k:]))
        elif i % 7 == 3 and n >= 2:
            out.append(C.Gate(tuple(int(v) for v in rng.permutation(n)[:2]), C.CP(float(rng.uniform(0, 6)))))
        else:
            out.append(C.Gate(qs[:k], C.haar_unitary(k, rng)))
    return out


@pytest.mark.parametrize("n", [7, 8, 9, 10, 11, 12, 13, 14, 17, 20, 21, 22, 26])
@pytest.mark.parametrize("fusion,max_k,precision", [("none", 1, "fp32_valu"), ("greedy", 4, "fp32_valu"),
                                                    ("greedy", 5, "fp32_mfma"), ("phase", 3, "fp16x3"),
                                                    ("greedy", 4, "bf16x3"), ("greedy", 6, "fp16x3")])
def test_sweeps_against_oracle(n, fusion, max_k, precision):
    from paper_2602_09604_amd import sv
    gates = mixed_circuit(n, 24 if n == 26 else 90, 6 if fusion == "none" else 3, 100 + n)
    st = sv.State(n)
    try:
        s = st.apply_circuit(gates, max_k=max_k, fusion=fusion, precision=precision, stats=True)
        got = st.read()
        norm = st.norm()
    finally:
        st.free()
    r = oracle.compare(got, oracle.apply_circuit(n, gates))
    print(n, fusion, max_k, precision, "passes", s["passes"], "launches", s["launches"], r, flush=True)
    assert s["launches"] <= s["passes"]
    if n >= 8 and fusion == "none":
        assert s["launches"] < s["passes"]
    bar = max(MAX_ABS, 2.0 ** -16 * s["passes"] ** 0.5) if precision == "bf16x3" else MAX_ABS
    assert r["max_abs"] <= bar and r["infidelity"] <= INFID, r
    assert abs(norm - 1.0) <= (1e-4 if precision == "bf16x3" else 1e-5)


@pytest.mark.parametrize("n", [12, 22])
def test_sweep_graph_and_launches_agree(n):
    """A kept graph of sweeps, relaunched, gives the plain launches' state bit
    for bit."""
    from paper_2602_09604_amd import sv
    gates = C.grid_circuit(2, n // 2, 8, seed=3)
    arr = sv.GateArray(gates)
    st = sv.State(n)
    try:
        st.apply_circuit(arr, max_k=4)
        ref = st.read()
        for rep in range(3):
            st.set_basis(0)
            s = st.apply_circuit(arr, max_k=4, use_graph=True, stats=True)
            assert s["graph_relaunched"] == (1 if rep else 0)
            assert np.array_equal(st.read(), ref)
            assert abs(st.norm() - 1.0) <= 1e-5
    finally:
        st.free()
