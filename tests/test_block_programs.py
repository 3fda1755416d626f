"""Register-resident tile programs on the host: the planner's output run by an
interpreter of the kernels (threads, LDS slots, layers), without a GPU."""
import time

import numpy as np
import pytest

import _programs
from _programs import SIGNED, signed_rotations
from oracle import statevector as sv
from paper_1912_03243_amd import workloads as W
from test_gpu_blocks import EPS, circuit, growth


@pytest.fixture(scope="module")
def P(tmp_path_factory):
    return _programs.Programs(str(tmp_path_factory.mktemp("programs")))


def cnots_and_rotations(n, count, seed):
    rng = np.random.default_rng([seed, n])
    recs = []
    for _ in range(count):
        a, b = (int(x) for x in rng.choice(n, 2, replace=False))
        recs.append(W.gate(W.OP_CNOT, a, b) if rng.random() < 0.6 else W.gate(W.OP_U, a, u=W.haar_u2(rng)))
    return W.concat(*recs)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("tile", [11, 12, 13])
def test_waves_share_slots_only_across_barriers(P, tile, dtype):
    # CNOTs done by the exchanges move the slots of a wave's amplitudes, within a
    # tile and from its last exchange to the next tile's first
    for seed in range(60):
        n = tile + seed % 3
        circ = cnots_and_rotations(n, 100, seed) if seed % 2 else circuit(n, 100, seed, True)
        got, rep = P.run(n, circ, dtype, tile=tile, low=5, relabel=-(seed & 1))
        assert rep.races == 0 and rep.misplaced == 0, (seed, rep.races, rep.misplaced)
        err = float(np.linalg.norm(got - sv.run_circuit(n, circ)))
        assert err <= 8.0 * EPS[dtype] * len(circ) * growth(circ), seed


# a pass whose relabel swap takes a bit of the scale block for a gathered one
SWAPPED_BLOCK = W.concat(W.gate(W.OP_H, 1), W.gate(W.OP_CNOT, 14, 5), W.gate(W.OP_H, 11),
                         W.gate(W.OP_CNOT, 15, 12), W.gate(W.OP_CNOT, 6, 7), W.gate(W.OP_CNOT, 0, 10),
                         W.gate(W.OP_CNOT, 2, 9), W.gate(W.OP_H, 1))


@pytest.mark.parametrize("pass_gates", [1, 2, 3, 4])
@pytest.mark.parametrize("block", [3, 4, 5, 6, 9])
def test_scale_blocks_stay_in_neighbouring_lanes(P, block, pass_gates):
    # the kernel takes a block's maximum over the lowest block - 3 lane bits
    for seed in range(-1, 10):
        n = 16 if seed < 0 else 14 + seed % 3
        circ = SWAPPED_BLOCK if seed < 0 else circuit(n, 12, seed, False)
        got, rep = P.run(n, circ, "enc2", low=max(3, block), pass_gates=pass_gates, block=block)
        assert rep.blocks == 0 and rep.races == 0 and rep.misplaced == 0, seed
        assert np.linalg.norm(got - sv.run_circuit(n, circ)) <= 8.0 * EPS["c64"] * len(circ)


@pytest.mark.parametrize("dtype, n, count, qubits, theta", SIGNED)
def test_scalars_of_signed_rotations(P, dtype, n, count, qubits, theta):
    # [[1, -t], [t, 1]] enlarges the state by sqrt(1 + t^2): the scalars cannot
    # wait for a rotation without signs and phases
    circ = signed_rotations(count, qubits, n, theta)
    got, rep = P.run(n, circ, dtype)
    want = sv.run_circuit(n, circ)
    assert np.linalg.norm(got - want) <= 8.0 * EPS[dtype] * len(circ)
    assert 2.0 ** -50 <= rep.least and rep.most <= 2.0 ** 30


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_matrices_far_from_unitary(P, dtype):
    # diagonals and rotations of very different sizes: planned so that the
    # coefficients hold them, or left to the fused passes
    left = 0
    for seed in range(60):
        rng = np.random.default_rng([seed, 77])
        n, recs = 13, []
        most = 10.0 ** [2, 12, 25][seed % 3]
        for _ in range(40):
            a, b = (int(x) for x in rng.choice(n, 2, replace=False))
            size = float(most ** rng.uniform(-1, 1))
            m = [np.diag([1.0, size * np.exp(1j * rng.uniform(0, 6))]), W.haar_u2(rng) @ np.diag([1.0, size]),
                 np.diag([size, 1.0]) @ W.haar_u2(rng), size * W.haar_u2(rng)][int(rng.integers(4))]
            recs.append(W.gate(W.OP_U, a, u=m) if rng.random() < 0.3 else
                        W.gate(W.OP_X, a) if rng.random() < 0.3 else W.gate(W.OP_CNOT, a, b))
        circ = W.concat(*recs)
        psi = sv.run_circuit(n, W.concat(*[W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(n)]))
        if dtype == "c64":
            psi = psi.astype(np.complex64).astype(np.complex128)
        got, rep = P.run(n, circ, dtype, psi=psi)
        if got is None:
            left += 1
            continue
        want = sv.run_circuit(n, circ, psi=psi.copy())
        limit = np.finfo(np.float32 if dtype == "c64" else np.float64)
        if np.abs(want).max() > limit.max / 2 ** 10 or np.linalg.norm(want) < limit.tiny * 2 ** 40:
            continue  # outside what the amplitudes can hold
        assert np.linalg.norm(got - want) <= 8.0 * EPS[dtype] * len(circ) * growth(circ), seed
    assert left < 60


def exact_state(n, circ):
    """The circuit's product in extended precision, from the gates' FP64 entries."""
    v = np.zeros(1 << n, np.clongdouble)
    v[0] = 1
    for g in circ:
        a, b = int(g["q0"]), int(g["q1"])
        if int(g["op"]) == W.OP_CZ:
            idx = np.arange(1 << n)
            v[((idx >> a) & (idx >> b) & 1) == 1] *= -1
            continue
        assert int(g["op"]) == W.OP_U
        u = g["u"].reshape(2, 2, 2).astype(np.longdouble)
        u = u[..., 0] + 1j * u[..., 1]
        w = v.reshape(-1, 2, 1 << a)
        w[:] = np.stack([u[0, 0] * w[:, 0] + u[0, 1] * w[:, 1], u[1, 0] * w[:, 0] + u[1, 1] * w[:, 1]], axis=1)
    return v


# A rounding's error has a standard deviation of about 0.41 2^-p of the value (p
# = 53, 24).  A rotation rounds the set half three times and the other half
# once, after its partner's, and its two or three coefficients once each, the
# phase's shared by both halves: less than six roundings, independent of each
# other.
ROUNDING = {"c128": 0.41 * 2.0 ** -53, "c64": 0.41 * 2.0 ** -24}


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n, layers", [(12, 20), (13, 40)])
def test_a_rotation_is_a_few_roundings(P, n, layers, dtype):
    errs = []
    for seed in range(4):
        circ = W.layered_brick(n, layers, seed=seed)
        got, _ = P.run(n, circ, dtype)
        errs.append(float(np.linalg.norm((got - exact_state(n, circ)).astype(complex))))
    assert np.sqrt(np.mean(np.square(errs))) <= ROUNDING[dtype] * np.sqrt(6 * n * layers)


@pytest.mark.parametrize("n, layers", [(12, 20), (13, 40)])
def test_rounded_phases_keep_the_norm(P, n, layers):
    # A phase rounded to FP32 changes the norm squared of the half that it acts on
    # by one rounding times that half's weight, and the pass's scalar takes back
    # what that is on average: what is left is in proportion to how far the
    # weight is from 1/2.  Squared and summed over a qubit's layers that is the
    # first rotation's 1 (on |0>) and less than 1 for the rest, while the qubits
    # become entangled.  The few dense ops that carry the scalars round once more.
    drift, left = [], 0
    for seed in range(8):
        circ = W.layered_brick(n, layers, seed=seed)
        got, rep = P.run(n, circ, "c64")
        exact = np.sum(np.abs(exact_state(n, circ)) ** 2)
        drift.append(float(np.sum(np.abs(got.astype(np.clongdouble)) ** 2) / exact - 1))
        left = max(left, 2 * n + rep.misc)
    assert np.sqrt(np.mean(np.square(drift))) <= ROUNDING["c64"] * np.sqrt(left)


@pytest.mark.parametrize("idle", [0, 8])
def test_planning_time_is_in_proportion_to_the_gates(P, idle):
    # one tile, all gates in one pass of many stages; idle: qubits that only the
    # last gate acts on.  Eight times the gates: eight times the time, 64 times if
    # every stage went through all of them
    n = 13

    def plan(count):
        circ = W.concat(W.random_mixed(n - idle, count, 5), W.gate(W.OP_CNOT, 0, n - 1))
        best = 1e9
        for _ in range(3):
            t = time.perf_counter()
            _, rep = P.run(n, circ, "c64", plan_only=True)
            best = min(best, time.perf_counter() - t)
        assert rep.passes == 1
        return best
    few, many = plan(5000), plan(40000)
    assert many < 24 * few, (few, many)


def test_first_rotations_find_a_basis_state(P):
    # the set half of a qubit in |0> is empty: a rounded phase there changes
    # nothing, and nothing has to be made up for
    n, known, unknown = 13, [], []
    start = np.zeros(1 << n)
    start[0] = 1
    for seed in range(12):
        circ = W.layered_brick(n, 1, seed=seed)
        exact = np.sum(np.abs(exact_state(n, circ)) ** 2)
        for psi, drift in ((None, known), (start, unknown)):
            got, _ = P.run(n, circ, "c64", psi=psi)
            drift.append(float(np.sum(np.abs(got.astype(np.clongdouble)) ** 2) / exact - 1))
    rms = lambda x: np.sqrt(np.mean(np.square(x)))
    assert rms(known) < rms(unknown)
