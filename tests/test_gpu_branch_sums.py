"""GPU checks of the sums over branches: sums of many bitstrings read
interleaved copies of the part states, sums of few read the states where they
lie; eight, four or single branches run side by side.  All add the same FP64
products in the same order, so every way gives the same bits."""
import numpy as np
import pytest

from oracle import statevector as sv
from paper_1912_03243_amd import workloads as W

pytestmark = pytest.mark.gpu

MANY = 1 << 16    # bitstrings from which sums read interleaved states


@pytest.fixture(scope="module")
def J():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1912_03243_amd import juqcs
    return juqcs


def circuit(sizes, crossings, seed):
    """Parts of the given sizes, Haar layers with a CZ ladder in each part, and
    crossings (part, part) at random qubits between the layers."""
    rng = np.random.default_rng(seed)
    side = np.repeat(np.arange(len(sizes)), sizes).astype(np.uint8)
    first = np.concatenate([[0], np.cumsum(sizes)])
    recs = []
    for i in range(len(crossings) + 1):
        recs += [W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(len(side))]
        for p, n in enumerate(sizes):
            recs += [W.gate(W.OP_CZ, int(first[p]) + k, int(first[p]) + k + 1) for k in range(i % 2, n - 1, 2)]
        if i < len(crossings):
            a, b = crossings[i]
            recs.append(W.gate(W.OP_CZ, int(first[a] + rng.integers(sizes[a])),
                               int(first[b] + rng.integers(sizes[b]))))
    return len(side), side, W.concat(*recs)


CASES = [
    ((6, 6), [(0, 1)], (0, 1)),                              # two branches
    ((8, 8), [(0, 1)] * 3, (0, 4, 1)),                       # 16 states: from LDS
    ((9, 8), [(0, 1)] * 6, (0, 32, 2)),                      # 128 states: where they lie
    ((5, 6, 7), [(0, 1), (1, 2), (0, 1), (1, 2)], (0, 8, 1)),
    ((4, 3, 5, 4), [(0, 1), (2, 3), (1, 2), (0, 3), (0, 1)], (0, 8)),
    ((5, 5, 6), [(0, 1)] * 3, (0,)),                         # a part without crossings
]


@pytest.mark.parametrize("sizes, crossings, groups", CASES)
def test_sums_of_many_and_few_agree(J, sizes, crossings, groups):
    n, side, circ = circuit(list(sizes), list(crossings), 7 * sum(sizes) + len(crossings))
    full = sv.run_circuit(n, circ)
    z = np.random.default_rng(n).integers(0, 1 << n, MANY + 3, dtype=np.uint64)
    few = J.juqcs_branch_amplitudes(n, circ, side, z[:1000])
    assert np.max(np.abs(few - full[z[:1000].astype(np.int64)])) / np.abs(full).max() < 1e-5
    for group in groups:
        print("CASE branch sums", sizes, len(crossings), group, flush=True)
        many = J.juqcs_branch_amplitudes(n, circ, side, z, group_size=group)
        assert np.array_equal(many[:1000], few)
        tail = J.juqcs_branch_amplitudes(n, circ, side, z[-5000:], group_size=group)
        assert np.array_equal(many[-5000:], tail)


def test_sums_in_a_workspace_without_room_for_interleaved_states(J):
    import torch
    n, side, circ = circuit([9, 8], [(0, 1)] * 6, 5)
    z = np.random.default_rng(1).integers(0, 1 << n, MANY, dtype=np.uint64)
    least, most = J.juqcs_branch_bytes(n, circ, side, 1, MANY, 0, True)
    want = J.juqcs_branch_amplitudes(n, circ, side, z)
    for size in (least, most - 1, most):
        work = torch.empty(size, dtype=torch.uint8, device="cuda")
        assert np.array_equal(J.juqcs_branch_amplitudes(n, circ, side, z, work=work), want)
