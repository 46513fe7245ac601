"""A batch whose gradient partials do not fit on the device is refused (919 GB
for 2^31 - 64 samples), and the network goes on as if it had not been asked."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def make(samples):
    import torch
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(samples))
    x = torch.tensor(rng.standard_normal((samples, sv.SV_COST_FEATURES)).astype(np.float32), device="cuda")
    y = torch.tensor(rng.standard_normal(samples).astype(np.float32), device="cuda")
    return sv, x, y


def too_large(sv, m, x, y):
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    loss = ctypes.c_float()
    rc = sv.lib().sv_mlp_train(ctypes.c_void_p(m.h), p(x), p(y), 2 ** 31 - 64, 1, ctypes.c_float(1e-3),
                               ctypes.byref(loss))
    assert rc == sv.SV_EDEVICE


def test_smaller_batch_after_a_failed_one():
    sv, x, y = make(200)
    a, b = sv.Mlp(seed=1), sv.Mlp(seed=1)
    try:
        for m in (a, b):
            m.train(x, y, epochs=2, lr=3e-3)
        g0 = b.loss_grad(x, y)
        too_large(sv, a, x, y)
        g1 = a.loss_grad(x, y)
        assert g0[0] == g1[0] and np.array_equal(g0[1], g1[1])
    finally:
        a.free()
        b.free()


def test_a_failed_call_counts_no_step():
    """Adam's bias corrections go by the number of updates made."""
    sv, x, y = make(100)
    a, b = sv.Mlp(seed=2), sv.Mlp(seed=2)
    try:
        too_large(sv, a, x, y)
        for m in (a, b):
            m.train(x, y, epochs=3, lr=3e-3)
        assert np.array_equal(a.get_params(), b.get_params())
    finally:
        a.free()
        b.free()
