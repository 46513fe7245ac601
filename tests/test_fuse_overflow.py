"""Fused matrices where the product overflows double precision: zero entries of
a gate times an infinite entry of the block are NaN, as in the full product, and
nothing is left out before that (finite gates, non-unitary)."""
import os

import numpy as np
import pytest

import circuits as C
from paper_2602_09604_amd import sv

needs_lib = pytest.mark.skipif(not os.path.exists(sv.LIB_PATH), reason="libsv.so not built")
X = np.array([[0, 1], [1, 0]], dtype=np.complex128)


def full_product(mats):
    """Row by row in the order of the gates, every product formed."""
    d = mats[0].shape[0]
    m = np.eye(d, dtype=np.complex128)
    re, im = m.real.copy(), m.imag.copy()
    with np.errstate(all="ignore"):
        for g in mats:
            nr, ni = np.zeros((d, d)), np.zeros((d, d))
            for r in range(d):
                for c in range(d):
                    a, b = g[r, c].real, g[r, c].imag
                    nr[r] += a * re[c] - b * im[c]
                    ni[r] += a * im[c] + b * re[c]
            re, im = nr, ni
    return re, im


@needs_lib
@pytest.mark.parametrize("scale", [1.0, 1e70, 1e120, 1e200, 1e307])
@pytest.mark.parametrize("seed", range(4))
def test_block_of_large_entries(scale, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    mats = []
    for i in range(9):
        kind = int(rng.integers(0, 3))
        m = X.copy() if kind == 0 else np.diag(rng.standard_normal(2) + 0j) if kind == 1 else rng.standard_normal((2, 2)) + 0j
        mats.append(m * (scale if rng.random() < 0.5 else 1.0))
    fused, _ = sv.sv_fuse([C.Gate((0,), m) for m in mats], 1, sv.make_opts(max_k=1))
    assert len(fused) == 1
    re, im = full_product(mats)
    got = fused[0].matrix
    assert np.array_equal(np.isnan(got.real), np.isnan(re)) and np.array_equal(np.isnan(got.imag), np.isnan(im))
    ok = np.isfinite(re)
    assert np.allclose(got.real[ok], re[ok], rtol=1e-13, atol=0)


@needs_lib
@pytest.mark.parametrize("entries", [(1e200, 1.0), (1e160, 1e-160), (1e100, 1.0)])
def test_one_row_overflows(entries):
    mats = [np.diag(np.array(entries) + 0j)] * 2 + [X, np.diag([1.0, 2.0]) + 0j]
    fused, _ = sv.sv_fuse([C.Gate((0,), m) for m in mats], 1, sv.make_opts(max_k=1))
    re, im = full_product(mats)
    assert np.array_equal(fused[0].matrix.real, re, equal_nan=True)
    assert np.array_equal(fused[0].matrix.imag, im, equal_nan=True)


@needs_lib
def test_long_block_stays_exact():
    """Thousands of gates in one block: the bound on its entries is renewed."""
    rng = np.random.Generator(np.random.PCG64(7))
    gates = [C.Gate((int(rng.integers(3)),), C.haar_unitary(1, rng)) for _ in range(3000)]
    fused, _ = sv.sv_fuse(gates, 3, sv.make_opts(max_k=3))
    m = np.eye(8, dtype=np.complex128)
    for g in gates:
        full = np.eye(1)
        for q in (2, 1, 0):
            full = np.kron(full, g.matrix if q == g.qubits[0] else np.eye(2))
        m = full @ m
    assert len(fused) == 1 and np.max(np.abs(fused[0].matrix - m)) < 1e-12
