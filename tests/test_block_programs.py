"""Register-resident tile programs on the host: the planner's output run by an
interpreter of the kernels (threads, LDS slots, layers), without a GPU."""
import numpy as np
import pytest

import _programs
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
