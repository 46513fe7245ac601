"""What a batch needs beside its states is given back: a large one leaves at
most 64 MiB of staging with its first handle."""
import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


def test_staging_is_given_back():
    import torch
    from paper_2602_09604_amd import sv
    n = 10
    m = C.haar_unitary(6, np.random.Generator(np.random.PCG64(2)))
    gates = [C.Gate((1, 2, 3, 5, 7, 9), m)] * 3000  # 96 MiB of matrices
    st = sv.State(n)
    try:
        sv.sv_batch_run([st.h], [gates[:4]], sv.make_opts(fusion="none"))
        free = torch.cuda.mem_get_info()[0]
        for _ in range(2):
            st.set_basis(0)
            stats = sv.sv_batch_run([st.h], [gates], sv.make_opts(fusion="none"))
            assert stats["passes"] == len(gates)
            assert free - torch.cuda.mem_get_info()[0] <= 64 << 20
            assert abs(st.norm() - 1.0) < 1e-4
        st.apply_circuit(gates[:8], fusion="none")  # the handle's ring still works
        assert abs(st.norm() - 1.0) < 1e-4
    finally:
        st.free()
