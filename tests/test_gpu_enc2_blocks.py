"""GPU checks of the register-resident passes on two-byte states: against the
same passes with explicitly fused gates (which decode tiles into LDS), for the
scale block sizes that they take and their neighbours, and states of one tile
and more.

Both apply a pass's gates to the same decoded amplitudes in FP32 and encode
the results.  A gate is at most 8 roundings of at most 2^-24 of the block's
largest component, and a code step is 1/127 of it, so G gates change a code
(by one) with a probability of at most 8 G 127 2^-24.  With a block's largest
component at most 6 times the root mean square, a pass adds at most 6/127
times the root of that probability to the relative 2-norm of the difference,
independently of the passes before it.
"""
import numpy as np
import pytest

from oracle import enc2 as oenc2
from paper_1912_03243_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def J():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1912_03243_amd import juqcs
    return juqcs


def general(n, seed):
    rng = np.random.default_rng(seed)
    recs = [W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(n)]
    for _ in range(3 * n):
        a, b = (int(x) for x in rng.choice(n, 2, replace=False))
        recs.append([W.gate(W.OP_CNOT, a, b), W.gate(W.OP_CZ, a, b), W.gate(W.OP_X, a),
                     W.gate(W.OP_U, a, u=W.haar_u2(rng)), W.gate(W.OP_S, a),
                     W.gate(W.OP_CP, a, b, theta=float(rng.uniform(0, 6)))][int(rng.integers(6))])
    return W.concat(*recs)


def state(J, n, block, circ, **kw):
    with J.State(n, "enc2", block_bits=block) as s:
        s.init(0)
        o = s.run(circ, **kw)
        codes, scales = s.raw_codes()
        psi = oenc2.decode(np.array(codes), np.array(scales), block) * s.global_factor()
        return psi, s.layout(), o.passes


@pytest.mark.parametrize("block", [3, 5, 8, 9, 10])
@pytest.mark.parametrize("n, relabel", [(13, -1), (14, 0), (16, -1), (18, 0)])
def test_codes_of_one_circuit(J, n, block, relabel):
    print("CASE enc2 blocks", n, block, relabel, flush=True)
    circ = general(n, 31 * n + block)
    got, layout, passes = state(J, n, block, circ, mode="tile", relabel=relabel)
    want, layout3, passes3 = state(J, n, block, circ, mode="tile", relabel=relabel, fuse_k=3)
    assert layout == layout3 and passes == passes3
    flip = 8 * len(circ) * 127 * 2.0 ** -24
    bound = np.sqrt(passes * flip) * 6 / 127
    assert np.linalg.norm(got - want) < bound * np.linalg.norm(want)


@pytest.mark.parametrize("flips", range(8))
def test_flips_within_a_group_of_codes(J, flips):
    # X on qubits 0-2 (the order of the eight codes of a group) and on others,
    # exact: the codes are permuted and nothing else
    print("CASE enc2 flips", flips, flush=True)
    n, block = 15, 8
    rng = np.random.default_rng(7)
    first = W.concat(*[W.gate(W.OP_U, q, u=W.haar_u2(rng)) for q in range(n)])
    x = [q for q in range(3) if (flips >> q) & 1] + [9, 14]
    circ = W.concat(*[W.gate(W.OP_X, q) for q in x])
    with J.State(n, "enc2", block_bits=block) as s:
        s.init(0)
        s.run(first, mode="tile", relabel=-1)
        codes, scales = (np.array(v) for v in s.raw_codes())
        s.run(circ, mode="tile", relabel=-1)
        codes2, scales2 = (np.array(v) for v in s.raw_codes())
    mask = sum(1 << q for q in x)
    before = oenc2.decode(codes, scales, block)
    want = before[np.arange(1 << n) ^ mask]
    assert np.array_equal(oenc2.decode(codes2, scales2, block), want)


@pytest.mark.parametrize("pass_gates", [1, 3])
@pytest.mark.parametrize("block", [4, 5])
def test_codes_with_short_chunks(J, block, pass_gates):
    # chunks of one scale block and passes of few gates: relabel swaps reach the
    # block's own bits
    print("CASE enc2 short chunks", block, pass_gates, flush=True)
    H, C = W.OP_H, W.OP_CNOT
    swapped = W.concat(W.gate(H, 1), W.gate(C, 14, 5), W.gate(H, 11), W.gate(C, 15, 12), W.gate(C, 6, 7),
                       W.gate(C, 0, 10), W.gate(C, 2, 9), W.gate(H, 1))
    opts = dict(mode="tile", low_bits=block, pass_gates=pass_gates)
    for circ in (swapped, W.concat(*[W.gate(H, q) for q in range(0, 16, 3)], swapped), general(16, 40 + block)):
        got, layout, passes = state(J, 16, block, circ, **opts)
        want, layout3, passes3 = state(J, 16, block, circ, fuse_k=3, **opts)
        assert layout == layout3 and passes == passes3
        flip = 8 * len(circ) * 127 * 2.0 ** -24
        bound = np.sqrt(passes * flip) * 6 / 127
        assert np.linalg.norm(got - want) < bound * np.linalg.norm(want)


@pytest.mark.parametrize("relabel", [-1, 0])
def test_scales_up_to_the_largest(J, relabel):
    # 2^14 amplitudes of 2^-7 times a factor that brings the scales next to FP32's
    # largest number: X gates move the codes and nothing else
    print("CASE enc2 largest scales", relabel, flush=True)
    n, block = 14, 8
    with J.State(n, "enc2", block_bits=block) as s:
        s.init(5)
        s.run(W.hadamard_all(n))
        s.scale(2.0 ** 7)
        s.scale(3.395e38)
        codes, scales = (np.array(v) for v in s.raw_codes())
        s.run(W.concat(W.gate(W.OP_X, 1), W.gate(W.OP_X, 9), W.gate(W.OP_X, 13)), mode="tile", relabel=relabel)
        got = s.state_vector()
    assert scales.max() > np.float32(127 / 128) * np.finfo(np.float32).max
    want = oenc2.decode(codes, scales, block)[np.arange(1 << n) ^ (1 << 1 | 1 << 9 | 1 << 13)]
    assert np.isfinite(want).all() and np.array_equal(got, want)
