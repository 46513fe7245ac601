"""Distinct handles on distinct threads whose sweeps take different amounts of
LDS in one kernel: every call succeeds and gives what the thread alone gives."""
import threading

import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


def test_threads_with_different_lds():
    import torch
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(3))
    work = []
    # 160 KiB (two 64 KiB matrices beside the tile) and 80 KiB (three of 16)
    for n, gates in ((18, [C.Gate((0, 1, 2, 3, 4, 5), C.haar_unitary(6, rng)),
                           C.Gate((2, 3, 4, 5, 6, 7), C.haar_unitary(6, rng))]),
                     (22, [C.Gate(tuple(range(i, i + 5)), C.haar_unitary(5, rng)) for i in range(3)])):
        for _ in range(2):
            work.append((n, sv.GateArray(gates)))
    reps, errors = 150, []

    def run(n, arr):
        s = torch.cuda.Stream()
        st = sv.State(n, stream=s)
        try:
            for _ in range(reps):
                st.apply_circuit(arr, fusion="none", precision="fp16x3")
            return st.read()
        finally:
            st.free()

    alone = [run(n, a) for n, a in work]
    got = [None] * len(work)

    def body(i):
        try:
            got[i] = run(*work[i])
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=body, args=(i,)) for i in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a, b in zip(alone, got):
        assert np.array_equal(a, b)
