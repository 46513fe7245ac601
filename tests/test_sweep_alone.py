"""Single wide passes take the kernel that is the fastest for their targets and
state: the amplitudes are those of the forced kernel bit for bit, or, where a
tile sweep is the choice, of neither of them, and within rounding of both."""
import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu

CASES = [  # n, targets, precision, the kernel AUTO is to take (None: a tile sweep)
    (22, (3, 7, 9, 14, 20, 21), "fp32_mfma", None),
    (24, (3, 7, 9, 14, 20, 21), "fp32_mfma", "mfma"),
    (24, (0, 1, 2, 4, 17, 19), "fp32_mfma", "mfma"),
    (21, (0, 2, 9, 14, 20), "fp32_mfma", "mfma"),
    (26, (4, 9, 14, 20, 25), "fp32_mfma", "mfma"),
    (26, (0, 3, 14, 20, 25), "fp32_mfma", None),
    (20, (3, 7, 9, 14, 19), "fp32_mfma", None),
    (28, (0, 18, 20, 25, 26), "fp32_valu", "reg"),
    (28, (0, 3, 20, 25, 26), "fp32_valu", None),
    (27, (0, 18, 20, 25, 26), "fp32_valu", None),
    (28, (1, 18, 20, 25, 26), "fp32_valu", None),
    (22, (4, 18, 19, 20, 21), "fp32_valu", None),
]


@pytest.mark.parametrize("n,targets,precision,kernel", CASES)
def test_single_pass_kernel(n, targets, precision, kernel):
    import torch
    from paper_2602_09604_amd import sv
    rng = np.random.Generator(np.random.PCG64(n))
    gate = C.Gate(targets, C.haar_unitary(len(targets), rng))
    start = torch.randn(1 << n, dtype=torch.complex64, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    start /= torch.linalg.vector_norm(start)
    st = sv.State(n)
    out = {}
    try:
        for variant in ("auto", "reg", "mfma"):
            st.buf.copy_(start)
            st.apply_circuit([gate], fusion="none", precision=precision, variant=variant)
            out[variant] = st.buf.clone()
        st.buf.copy_(start)
        st.apply_circuit([gate], fusion="none", precision=precision, use_graph=True)
        graph = st.buf.clone()
    finally:
        st.free()
    # below 24 qubits a kept graph of a 6-qubit matrix-core pass takes its own kernel
    want = "mfma" if precision == "fp32_mfma" and len(targets) == 6 and n > 20 else "auto"
    assert torch.equal(torch.view_as_real(graph), torch.view_as_real(out[want]))
    scale = float(out["reg"].abs().max())
    assert float((out["auto"] - out["reg"]).abs().max()) <= 2e-6 * scale * (1 << len(targets)) ** 0.5
    for variant in ("reg", "mfma"):
        same = torch.equal(torch.view_as_real(out["auto"]), torch.view_as_real(out[variant]))
        if variant == kernel or (kernel == "reg" and precision == "fp32_valu"):
            assert same  # at FP32_VALU a forced matrix-core pass is the register kernel
        else:
            assert not same
