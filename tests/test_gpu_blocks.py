"""GPU checks of the register-resident tile programs.

Circuits over every gate kind, at the tile sizes the kernels are built for
and at the edges of the state sizes that use them (one tile, two tiles, many),
against the FP64 oracle.  Gates that are not unitary, singular ones and ones
of very different size take the dense form of a program; diagonal ones, bit
flips and controls on every kind of tile bit take the others.

Tolerance: a gate is at most 8 roundings per amplitude component, each of
relative size eps / 2 (eps = 2^-52, 2^-23), and coefficients rounded to eps / 2,
so the 2-norm error of a gate stays below 8 eps times the product of the
gates' largest singular values; it grows at most linearly in the gates.
"""
import numpy as np
import pytest

from _programs import SIGNED, signed_rotations
from oracle import decomposition as odec
from oracle import statevector as sv
from paper_1912_03243_amd import workloads as W

pytestmark = pytest.mark.gpu

EPS = {"c128": 2.0 ** -52, "c64": 2.0 ** -23}


@pytest.fixture(scope="module")
def J():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1912_03243_amd import juqcs
    return juqcs


def random_gate(rng, n, general):
    """One gate of any kind; general: dense matrices that are not unitary too."""
    kind = int(rng.integers(0, 13 if general else 10))
    a, b = (int(x) for x in rng.choice(n, 2, replace=False))
    if kind in W.TWO_QUBIT_OPS:
        return W.gate(kind, a, b, theta=float(rng.uniform(0, 2 * np.pi)) if kind == W.OP_CP else 0.0)
    if kind == W.OP_U:
        return W.gate(W.OP_U, a, u=W.haar_u2(rng))
    if kind == 10:    # not unitary
        return W.gate(W.OP_U, a, u=W.haar_u2(rng) @ np.diag(rng.uniform(0.7, 1.3, 2)) @ W.haar_u2(rng))
    if kind == 11:    # triangular, one entry zero
        return W.gate(W.OP_U, a, u=np.array([[1.0, rng.uniform(-0.5, 0.5)], [0.0, 1.0j]]))
    if kind == 12:    # a diagonal of different sizes
        return W.gate(W.OP_U, a, u=np.diag([rng.uniform(0.6, 1.2), np.exp(1j * rng.uniform(0, 6)) * 0.9]))
    return W.gate(kind, a)


def circuit(n, count, seed, general):
    rng = np.random.default_rng([seed, n, count])
    return W.concat(*[random_gate(rng, n, general) for _ in range(count)])


def growth(circ):
    p = 1.0
    for g in circ:
        if int(g["op"]) == W.OP_U:
            m = g["u"].reshape(2, 2, 2)
            p *= max(1.0, float(np.linalg.norm(m[..., 0] + 1j * m[..., 1], 2)))
    return p


def check(J, n, dtype, circ, **opts):
    want = sv.run_circuit(n, circ)
    with J.State(n, dtype) as s:
        s.init(0)
        half = len(circ) // 2
        s.run(circ[:half], **opts)          # the second run starts from a permuted layout
        s.run(circ[half:], **opts)
        got = s.state_vector()
    err = float(np.linalg.norm(got - want))
    bound = 8.0 * EPS[dtype] * len(circ) * growth(circ)
    print(f"blocks {n} {dtype} {opts}: |err| = {err:.2e}, bound {bound:.2e}", flush=True)
    assert err <= bound


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n, tile_bits", [(11, 0), (12, 0), (13, 0), (14, 0), (14, 11), (15, 12), (18, 0), (19, 13)])
@pytest.mark.parametrize("general", [False, True])
def test_programs_against_the_oracle(J, n, tile_bits, dtype, general):
    print("CASE blocks", n, tile_bits, dtype, general, flush=True)
    check(J, n, dtype, circuit(n, 150, 31, general), mode="tile", tile_bits=tile_bits,
          low_bits=min(5, tile_bits - 2) if tile_bits else 0)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_programs_without_relabeling(J, dtype):
    print("CASE blocks-fixed-layout", dtype, flush=True)
    check(J, 17, dtype, circuit(17, 150, 32, True), mode="tile", relabel=-1)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("pass_gates", [1, 7])
def test_short_programs(J, dtype, pass_gates):
    # programs of one gate and of a few: every gate kind alone in its pass
    print("CASE blocks-short", dtype, pass_gates, flush=True)
    check(J, 14, dtype, circuit(14, 60, 33, True), mode="tile", pass_gates=pass_gates)


def test_scalars_stay_in_range(J):
    # 40 layers on one tile: the rotations' scalar factors would overflow FP32
    # if they were left to the end
    n = 13
    print("CASE blocks-deep", n, flush=True)
    check(J, n, "c64", W.layered_brick(n, 40, seed=34), mode="tile")


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_exact_gates_stay_exact(J, dtype):
    # permutations, signs and +-i phases of a basis state: no rounding at all
    n = 15
    rng = np.random.default_rng(35)
    print("CASE blocks-exact", dtype, flush=True)
    ops = [W.OP_X, W.OP_Y, W.OP_Z, W.OP_S, W.OP_CNOT, W.OP_CZ]
    recs = []
    for _ in range(200):
        op = int(rng.choice(ops))
        a, b = (int(x) for x in rng.choice(n, 2, replace=False))
        recs.append(W.gate(op, a, b if op in (W.OP_CNOT, W.OP_CZ) else -1))
    circ = W.concat(*recs)
    with J.State(n, dtype) as s:
        s.init(5)
        s.run(circ)
        got = s.state_vector()
    want = sv.run_circuit(n, circ, psi=sv.init_state(n, 5))
    assert np.array_equal(got, want)


def sized_circuits(sizes, gates, seed):
    rng = np.random.default_rng(seed)
    out = [(n, W.concat(*[random_gate(rng, n, False) for _ in range(gates)])) for n in sizes]
    return out + [(n, W.empty_circuit(0)) for n in sizes[-2:]]


@pytest.mark.parametrize("relabel", [-1, 0])
@pytest.mark.parametrize("sizes", [[10, 11, 12, 13], [14, 11, 15, 13, 16, 12], [13, 13, 13], [17, 10]])
def test_batch_tile_sizes(J, sizes, relabel):
    # one tile and many, every tile size in one list, beside circuits too
    # small for them and circuits without gates; run again over garbage
    print("CASE batch", sizes, relabel, flush=True)
    gates = 60
    circuits = sized_circuits(sizes, gates, 5 + len(sizes))
    b = J.Batch(circuits, relabel=relabel)
    for again in range(2):
        b.run()
        b.wait()
        for i, (n, circ) in enumerate(circuits):
            want = sv.run_circuit(n, circ)
            assert np.linalg.norm(b.state_vector(i) - want) < 8 * (len(circ) + 1) * EPS["c64"]
            assert (b.fusion()[i] == 1) == (n >= 11)
        b.states.fill_(7)
    b.close()


@pytest.mark.parametrize("group", [0, 4])
@pytest.mark.parametrize("nloc, per_run", [(10, 2), (11, 2), (13, 3), (14, 1)])
def test_branch_tile_sizes(J, nloc, per_run, group):
    # two parts around the smallest and the largest tile (10 keeps the fused
    # passes), runs of one to three crossings, every group size's tree;
    # against the oracle's branch sum with the bound of the other branch tests
    print("CASE branch", nloc, per_run, group, flush=True)
    rng = np.random.default_rng(100 * nloc + per_run)
    n, side = 2 * nloc, np.repeat([0, 1], nloc).astype(np.uint8)
    recs = [W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(n)]
    for run in range(3):
        for h in (0, nloc):
            for _ in range(20):
                g = random_gate(rng, nloc, False).copy()
                g["q0"] += h
                g["q1"] = np.where(g["q1"] >= 0, g["q1"] + h, g["q1"])
                recs.append(g)
        if run < 2:
            for _ in range(per_run):
                recs.append(W.gate(W.OP_CZ, int(rng.integers(nloc)), nloc + int(rng.integers(nloc))))
    circ = W.concat(*recs)
    z = rng.integers(0, 1 << n, 64, dtype=np.uint64)
    got = J.juqcs_branch_amplitudes(n, circ, side, z, group_size=group)
    want = odec.branch_amplitudes(n, circ, side, z)
    assert np.max(np.abs(got - want)) / np.abs(want).max() < 1e-5


@pytest.mark.parametrize("dtype, n, count, qubits, theta", SIGNED)
def test_scalars_of_signed_rotations(J, dtype, n, count, qubits, theta):
    # rotations that all carry signs or phases: their scalars would leave FP32's
    # (and FP64's) range over a pass
    print("CASE blocks-signed", dtype, n, count, qubits, theta, flush=True)
    circ = signed_rotations(count, qubits, n, theta)
    want = sv.run_circuit(n, circ)
    bound = 8.0 * EPS[dtype] * len(circ)
    with J.State(n, dtype) as s:
        s.init(0)
        s.run(circ, mode="tile")
        assert np.linalg.norm(s.state_vector() - want) <= bound
    if dtype == "c64":
        b = J.Batch([(n, circ)])
        b.run()
        b.wait()
        assert b.fusion()[0] == 1
        assert np.linalg.norm(b.state_vector(0) - want) <= bound
        b.close()


@pytest.mark.parametrize("dtype", ["c128", "c64", "enc2"])
@pytest.mark.parametrize("n", [10, 12, 14])
def test_no_gates_no_pass(J, n, dtype):
    print("CASE blocks-empty", n, dtype, flush=True)
    with J.State(n, dtype) as s:
        s.init(3)
        for opts in (dict(), dict(mode="tile"), dict(mode="tile", relabel=-1)):
            assert s.run(W.empty_circuit(0), **opts).passes == 0
        got = s.state_vector()
    assert got[3] == 1 and np.count_nonzero(got) == 1


@pytest.mark.parametrize("dtype, power", [("c128", 1010), ("c64", 115), ("enc2", 115)])
def test_scaled_states_stay_in_range(J, dtype, power):
    # a pass of 300 rotations would enlarge amplitudes of 2^power / 91 by up to 2^24
    # before its scalars come in: such states take the fused passes, and a power
    # of two changes none of their roundings
    print("CASE blocks-scaled", dtype, power, flush=True)
    n = 13
    first = W.layered_brick(n, 2, seed=37)
    circ = W.layered_brick(n, 24, seed=38)

    def run(p, fuse_k):
        with J.State(n, dtype) as s:
            s.init(0)
            s.run(first, mode="tile", fuse_k=3)
            s.scale(2.0 ** (p // 2))
            s.scale(2.0 ** (p - p // 2))
            s.run(circ, mode="tile", fuse_k=fuse_k)
            return s.state_vector() * 2.0 ** -(p // 2) * 2.0 ** -(p - p // 2)
    got = run(power, 0)
    assert np.isfinite(got).all() and np.array_equal(got, run(0, 3))
