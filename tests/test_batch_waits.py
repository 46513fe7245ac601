"""sv_batch_run returns once the work queued on every handle's stream has
finished, also when the circuits turn out to hold nothing to launch."""
import pytest

import circuits as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("circuit", [[], [C.Gate((0,), C.H)]])
def test_batch_returns_after_queued_work(circuit):
    import numpy as np
    import torch
    from paper_2602_09604_amd import sv
    m = C.haar_unitary(5, np.random.Generator(np.random.PCG64(1)))
    big, small = sv.State(28, stream=torch.cuda.Stream()), sv.State(9, stream=torch.cuda.Stream())
    try:
        big.norm()
        for _ in range(100):  # about 80 ms of work
            big.apply_gate((20, 21, 22, 23, 24), m)
        done = torch.cuda.Event()
        done.record(big.stream)
        assert not done.query()
        sv.sv_batch_run([small.h, big.h], [circuit, []])
        assert done.query()
    finally:
        small.free()
        big.free()
