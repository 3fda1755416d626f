"""GPU checks of the expectation values of two-byte states: integer sums over
raw codes (block sizes of 2^6 amplitudes and more, states of 24 qubits and
more) and, around them, the sums over decoded amplitudes.

Reference: the pair sums in FP64 of the decoded amplitudes, which are the
codes times an FP32 factor rounded to FP32 (relative 2^-24).  Every sum is
bounded by the squared norm (about 1), twice that rounding enters a product,
and the value is half the sum, so they agree to 2^-24 times the squared norm;
FP64 summation adds less than 2^-30."""
import numpy as np
import pytest

from paper_1912_03243_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def J():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1912_03243_amd import juqcs
    return juqcs


def reference(phi, n):
    """[(1 - <sigma>)/2] of qubit q from pair sums, on the GPU in FP64."""
    import torch
    a = torch.from_numpy(phi).cuda()
    out = np.empty((n, 3))
    for q in range(n):
        v = a.view(-1, 2, 1 << q)
        p = torch.sum(torch.conj(v[:, 0]) * v[:, 1])
        z = torch.sum(torch.abs(v[:, 0]) ** 2) - torch.sum(torch.abs(v[:, 1]) ** 2)
        out[q] = [0.5 * (1 - 2 * p.real.item()), 0.5 * (1 - 2 * p.imag.item()), 0.5 * (1 - z.item())]
    return out


@pytest.mark.parametrize("n, block", [(23, 8), (24, 5), (24, 6), (24, 8), (24, 12), (25, 7), (26, 8)])
def test_expectations_of_codes(J, n, block):
    print("CASE expect enc2", n, block, flush=True)
    rng = np.random.default_rng(100 * n + block)
    circ = W.concat(*[W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(n)],
                    *[W.gate(W.OP_CZ, q, q + 1) for q in range(n - 1)],
                    *[W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(0, n, 2)])
    with J.State(n, "enc2", block_bits=block) as s:
        s.init(0)
        s.run(circ)
        got = np.asarray(s.expectations()).reshape(n, 3)
        phi = s.state_vector()
    want = reference(np.asarray(phi, dtype=np.complex128), n)
    norm2 = float(np.vdot(phi, phi).real)
    assert np.max(np.abs(got - want)) < 2.0 ** -24 * norm2 + 2.0 ** -30
