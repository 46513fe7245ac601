"""Batched circuits below the sizes of tests/test_batch.py: states no tile
takes (n < 8, and 8 or 9 qubits with gates too wide for the tile), the
smallest tiles, one-tile states with one and several sweeps, and all of them in
one batch.  Bar: 1e-5 and infidelity 1e-6, as for single circuits."""
import json

import numpy as np
import pytest

import circuits as C
import oracle
from test_sweep import mixed_circuit

pytestmark = pytest.mark.gpu


def run(ns, circs, **opts):
    from paper_2602_09604_amd import sv
    states = [sv.State(n) for n in ns]
    try:
        stats = sv.sv_batch_run([s.h for s in states], circs, sv.make_opts(**opts))
        return [s.read() for s in states], stats
    finally:
        for s in states:
            s.free()


def check(ns, circs, out):
    for n, c, got in zip(ns, circs, out):
        r = oracle.compare(got, oracle.apply_circuit(n, c))
        assert r["max_abs"] <= 1e-5 and r["infidelity"] <= 1e-6, (n, r)


def uncontrolled(n, gates, max_k, seed):
    return [g for g in mixed_circuit(n, gates, max_k, seed) if not g.controls]


@pytest.mark.parametrize("opts", [dict(fusion="none"), dict(max_k=4), dict(max_k=6), dict(max_k=5, fusion="block")])
@pytest.mark.parametrize("n", list(range(1, 14)))
def test_one_size(n, opts):
    ns = [n] * 3
    circs = [uncontrolled(n, 60, 6 if opts.get("fusion") == "none" else 3, 7 * n + i) for i in range(3)]
    out, stats = run(ns, circs, **opts)
    check(ns, circs, out)
    assert stats["launches"] <= stats["passes"]
    if n < 8:
        assert stats["launches"] == 1


@pytest.mark.parametrize("narrow,wide", [(4, 5), (3, 6)])
def test_every_path_in_one_batch(narrow, wide):
    ns, circs = [], []
    for n in (3, 7, 8, 8, 9, 9, 10, 12, 13, 16):
        k = wide if len(ns) % 2 else narrow
        ns.append(n)
        circs.append(uncontrolled(n, 40, min(k, n), 50 + len(ns)))
    ns.append(11)
    circs.append([])
    out, stats = run(ns, circs, fusion="none")
    check(ns, circs, out)
    assert stats["gates_in"] == sum(len(c) for c in circs)
