"""GPU checks of the sums over branches: sums of many bitstrings read
interleaved copies of the part states, sums of few read the states where they
lie; eight, four or single branches run side by side.  All add the same FP64
products in the same order, so every way gives the same bits."""
import numpy as np
import pytest

from oracle import decomposition as odec
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


def parts_of(nloc, parts, per, rounds, seed):
    """Equal parts, per random gates each between the crossings."""
    rng = np.random.default_rng(seed)
    recs = []
    for r in range(rounds):
        for p in range(parts):
            for _ in range(per):
                a, b = (int(x) + p * nloc for x in rng.choice(nloc, 2, replace=False))
                recs.append([W.gate(W.OP_U, a, u=W.haar_u2(rng)), W.gate(W.OP_H, a), W.gate(W.OP_CNOT, a, b),
                             W.gate(W.OP_CZ, a, b), W.gate(W.OP_CP, a, b, theta=1.1)][int(rng.integers(5))])
        if r + 1 < rounds:
            a, b = (int(x) for x in rng.choice(parts, 2, replace=False))
            recs.append(W.gate(W.OP_CZ, a * nloc + int(rng.integers(nloc)), b * nloc + int(rng.integers(nloc))))
    return nloc * parts, np.repeat(np.arange(parts), nloc).astype(np.uint8), W.concat(*recs)


# Workspaces (64 bitstrings from the host) of these circuits with fused passes,
# per group size; the register-resident passes' work lists are larger.
FUSED_BYTES = [((11, 2, 40, 7, 1), {1: 45312, 4: 160512, 0: 2481664}),
               ((11, 3, 78, 4, 2), {1: 82176, 4: 174080, 0: 288768}),
               ((12, 3, 30, 4, 3), {1: 115968, 4: 284160, 0: 487424})]


@pytest.mark.parametrize("args, sizes", FUSED_BYTES)
def test_workspaces_of_the_fused_passes(J, args, sizes):
    # a workspace that one of the two kinds of passes has room in is enough, and
    # every group size gives the same bits where both kinds have for one branch
    import torch
    print("CASE fused workspaces", args, flush=True)
    n, side, circ = parts_of(*args)
    z = np.random.default_rng(1).integers(0, 1 << n, 64, dtype=np.uint64)
    want = odec.branch_amplitudes(n, circ, side, z)
    ref = J.juqcs_branch_amplitudes(n, circ, side, z)
    least = J.juqcs_branch_bytes(n, circ, side, 1, 64, 1)[0]
    assert sizes[1] < least
    for group, size in sizes.items():
        work = torch.empty(size, dtype=torch.uint8, device="cuda")
        got = J.juqcs_branch_amplitudes(n, circ, side, z, group_size=group, work=work)
        assert np.max(np.abs(got - want)) < 1e-5 * np.abs(want).max()
        if size >= least:
            assert np.array_equal(got, ref)
    with pytest.raises(J.JuqcsError) as e:
        J.juqcs_branch_amplitudes(n, circ, side, z, group_size=1, work=work[:sizes[1] // 512 * 256])
    assert e.value.status == J.ERR_SIZE


def test_noalloc_bits_do_not_depend_on_the_group_size(J):
    # bitstrings until the largest group's register-resident passes no longer fit
    # the static scratch, where the fused ones do
    import torch
    n, side, circ = parts_of(11, 3, 78, 4, 2)
    need = lambda count: J.juqcs_branch_bytes(n, circ, side, 1, count, 0, False)
    lo, hi = 1 << 10, 1 << 22
    least, whole = need(lo)  # the largest group takes this much more than one branch
    full = lambda count: need(count)[0] + whole - least
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if full(mid) <= J.NOALLOC_SCRATCH_BYTES else (lo, mid)
    count = hi + 64
    print("CASE noalloc groups", count, flush=True)
    z = torch.from_numpy(np.random.default_rng(2).integers(0, 1 << n, (count, 1), dtype=np.int64)).cuda()
    out = []
    for group in (0, 8, 1):
        got = torch.empty(2 * count, dtype=torch.float64, device="cuda")
        J.juqcs_branch_amplitudes_noalloc(n, circ, side, z, got, group_size=group)
        out.append(got.cpu().numpy())
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("group", [0, 1, 4, 16])
@pytest.mark.parametrize("args", [(11, 2, 12, 7, 11), (12, 3, 30, 5, 12), (13, 2, 8, 9, 13)])
def test_reported_workspaces_hold_the_group(J, args, group):
    # the sizes come from the gates' shapes, without a plan for every setting of
    # the crossings
    import torch
    print("CASE reported workspaces", args, group, flush=True)
    n, side, circ = parts_of(*args)
    z = np.random.default_rng(3).integers(0, 1 << n, 200, dtype=np.uint64)
    least, size = J.juqcs_branch_bytes(n, circ, side, 1, len(z), group)
    for want, work in ((group, size), (1, least)):
        got = J.juqcs_branch_amplitudes(n, circ, side, z, group_size=want,
                                        work=torch.empty(work, dtype=torch.uint8, device="cuda"))
        st = J.juqcs_branch_last_stats()
        assert st["group_bits"] == (0 if want == 0 else max(0, st["crossings"] - int(np.log2(want))))
    ref = odec.branch_amplitudes(n, circ, side, z)
    assert np.max(np.abs(got - ref)) < 1e-5 * np.abs(ref).max()
