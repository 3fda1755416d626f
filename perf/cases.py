"""Performance cases of the state-vector engine: the work its users have it do.

A case names a program ("kind"), its sizes and its amplitude type:

  circuit  a state is initialised, a circuit is run in the planner's default
           mode, and amplitudes of M bitstrings are read (all of them on small
           states), optionally with the norm and the expectation values of all
           qubits: the simulator's ordinary use (Sections 3 and 4 of
           arXiv:1912.03243);
  fused    the same with dense k-qubit blocks (mode "fused");
  gates    a program that drives the state gate by gate: single-qubit,
           controlled, two-qubit and fused-block calls on qubits all over the
           register;
  codec    two-byte encoding and decoding of an amplitude array (saving and
           loading states);
  batch    many independent small circuits in one launch;
  branch   amplitudes of a circuit too wide for a state vector by the
           entangling-gate decomposition (Section 4).

Amplitudes of C64 and two-byte states are computed in 32 bits and returned as
32-bit numbers; those of a two-byte state after gates that do not keep its
codes exact have about three digits and are returned as bfloat16.
"""
import math

import numpy as np
import torch

from paper_1912_03243_amd import juqcs
from paper_1912_03243_amd import workloads as W

DEV = "cuda"
AMP_BYTES = {"c128": 16, "c64": 8, "enc2": 2}
WHOLE = 22      # states of up to this many qubits are read whole
MANY = 1 << 20  # bitstrings read from larger ones (Section 4 extracts 2^20)


def listed():
    return [
        # a first small experiment: every call's fixed cost
        dict(name="mixed12_c128", kind="circuit", circuit="mixed", n=12, size=80, dtype="c128", read=1 << 12),
        # a circuit of named and random gates on a state that fits the caches
        dict(name="mixed20_c128", kind="circuit", circuit="mixed", n=20, size=200, dtype="c128", read=1 << 20),
        # the headline: 20 brick layers on a 16 GiB double-precision state
        dict(name="brick30_c128", kind="circuit", circuit="brick", n=30, size=20, dtype="c128", read=4096),
        # the same circuit family in single precision, odd qubit count
        dict(name="brick31_c64", kind="circuit", circuit="brick", n=31, size=16, dtype="c64", read=1000003),
        # the Section 3 benchmark (GHZ and all expectation values) on two-byte amplitudes
        dict(name="ghz33_enc2", kind="circuit", circuit="ghz", n=33, size=0, dtype="enc2", read=65537),
        # random layers on two-byte amplitudes
        dict(name="brick29_enc2", kind="circuit", circuit="brick", n=29, size=1, dtype="enc2", read=MANY),
        # quantum Fourier transform of a basis state: controlled phases of every range
        dict(name="qft27_c128", kind="circuit", circuit="qft", n=27, size=0, dtype="c128", read=MANY),
        # a program that applies its gates one call at a time
        dict(name="gates27_c128", kind="gates", n=27, size=24, dtype="c128", read=MANY),
        # dense blocks on the matrix cores
        dict(name="fused28_c64", kind="fused", circuit="brick", n=28, size=6, dtype="c64", read=MANY),
        # variational sweep: many small independent circuits at once
        dict(name="batch301", kind="batch", size=301, nmin=12, nmax=21, dmin=10, dmax=40, read=64),
        # Section 4: 42 qubits in two halves, 8 decomposed CZs, 2^20 coefficients
        dict(name="grid42", kind="branch", circuit="grid", n=42, size=8, parts=2, read=MANY),
        # Section 4: GHZ on 128 qubits in eight parts
        dict(name="ghz128", kind="branch", circuit="ghz", n=128, size=7, parts=8, read=(1 << 24) + 5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "circuit", "fused", "gates", "codec", "batch", "branch", "branch"])
    if kind in ("circuit", "fused"):
        dtype = rng.choice(["c128", "c64"] if kind == "fused" else ["c128", "c128", "c64", "c64", "enc2"])
        circuit = "brick" if kind == "fused" else rng.choice(["mixed", "brick", "brick", "qft", "ghz"])
        lo, hi = {"c128": (12, 29), "c64": (12, 30), "enc2": (16, 31)}[dtype]
        if kind == "fused":
            lo, hi = 16, 27
        n = rng.randint(lo, hi)
        size = {"mixed": _log_int(rng, 40, 400), "brick": rng.randint(4, 20), "qft": 0, "ghz": 0}[circuit]
        if dtype == "enc2" and circuit != "ghz":
            circuit, size = "brick", 1
        read = 1 << n if n <= WHOLE else _log_int(rng, 1000, MANY)
        return dict(kind=kind, circuit=circuit, n=n, size=size, dtype=dtype, read=read)
    if kind == "gates":
        n = rng.randint(14, 28)
        return dict(kind="gates", n=n, size=rng.randint(8, 40), dtype=rng.choice(["c128", "c64"]), read=1 << n if n <= WHOLE else MANY)
    if kind == "codec":
        return dict(kind="codec", n=rng.randint(16, 29), block=rng.randint(5, 10), dtype=rng.choice(["c128", "c64"]))
    if kind == "batch":
        nmin = rng.randint(8, 14)
        return dict(kind="batch", size=_log_int(rng, 3, 400), nmin=nmin, nmax=nmin + rng.randint(0, 7), dmin=5, dmax=rng.randint(10, 40),
                    read=rng.choice([1, 64, 500]))
    if rng.random() < 0.6:
        rows, cols = rng.choice([(4, 6), (5, 6), (6, 6), (5, 8), (7, 6)])
        return dict(kind="branch", circuit="grid", n=rows * cols, size=rng.randint(3, 8), parts=2, read=_log_int(rng, 1000, MANY))
    parts = rng.randint(2, 8)
    return dict(kind="branch", circuit="ghz", n=parts * rng.randint(10, 16), size=parts - 1, parts=parts, read=_log_int(rng, 1000, 1 << 24))


# ---- inputs ----------------------------------------------------------------
GRID_ROWS = {24: 4, 30: 5, 36: 6, 40: 5, 42: 7}


def _rng(seed):
    return np.random.default_rng([1912, seed])


def _circuit(case, seed):
    """(gate records, basis index the state starts from)."""
    n = case["n"]
    if case["circuit"] == "mixed":
        return W.random_mixed(n, case["size"], seed=seed), 0
    if case["circuit"] == "brick":
        return W.layered_brick(n, case["size"], seed=seed), 0
    return (W.qft(n) if case["circuit"] == "qft" else W.ghz(n)), int(_rng(seed).integers(0, 1 << n))


def _ghz_pair(n, x):
    """The two basis states that the GHZ chain turns basis state x into, and
    the sign of the second: H on qubit 0, then y_i = y_(i-1) xor x_i."""
    s = [0, 1]
    for q in range(1, n):
        for b in (0, 1):
            s[b] |= (((s[b] >> (q - 1)) ^ (x >> q)) & 1) << q
    return s[0], s[1], -1.0 if x & 1 else 1.0


def _bitstrings(case, seed, start):
    n, m = case["n"], case["read"]
    if m == 1 << n:
        return torch.arange(m, dtype=torch.int64, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(seed + 7)
    z = torch.randint(0, 1 << n, (m,), generator=g, dtype=torch.int64, device=DEV)
    if case["circuit"] == "ghz":  # the two amplitudes that are not zero are among those asked for
        z[:: max(1, m // 500)] = _ghz_pair(n, start)[0]
        z[1:: max(2, m // 400)] = _ghz_pair(n, start)[1]
    return z


def _drive(case, seed):
    """The calls of a gate-by-gate program: (name, qubits, matrix)."""
    rng, n = _rng(seed), case["n"]
    calls = []
    for k in range(case["size"]):
        what = ["1q", "1q", "cu", "2q", "diag", "fused"][k % 6]
        width = {"1q": 1, "diag": 1, "cu": 2, "2q": 2, "fused": 2 + k % 4}[what]
        # low, middle and high qubits alike
        qs = [int(q) for q in rng.choice(n, size=width, replace=False)]
        if what == "diag":
            m = np.diag(np.exp(1j * rng.uniform(0, 2 * np.pi, 2)))
        else:
            dim = 2 if what == "cu" else 1 << width
            z = rng.standard_normal((dim, dim)) + 1j * rng.standard_normal((dim, dim))
            m, r = np.linalg.qr(z)
            m = m * (np.diag(r) / np.abs(np.diag(r)))
        calls.append((what, qs, m))
    return calls


def _batch_circuits(case, seed):
    out = []
    for i in range(case["size"]):
        rng = _rng((seed << 12) + i)
        n = int(rng.integers(case["nmin"], case["nmax"] + 1))
        out.append((n, W.layered_random_pairs(n, int(rng.integers(case["dmin"], case["dmax"] + 1)), rng)))
    return out


def _branch(case, seed):
    """(gates, part of each qubit, x): x the basis state before a GHZ chain."""
    n = case["n"]
    if case["circuit"] == "grid":
        rows = GRID_ROWS[n]
        gates, side = W.grid_circuit(rows, n // rows, 12, seed=seed, max_cross=case["size"])
        return gates, side, 0
    bits = _rng(seed).integers(0, 2, n)
    x = sum(int(b) << q for q, b in enumerate(bits))
    return W.concat(W.prepare_basis(n, x), W.ghz(n)), W.block_parts(n, case["parts"]), x


def _branch_bitstrings(case, seed, x):
    n, m = case["n"], case["read"]
    words = (n + 63) // 64
    g = torch.Generator(device=DEV).manual_seed(seed + 9)
    z = torch.empty((m, words), dtype=torch.int64, device=DEV)
    for w in range(words):
        bits = min(64, n - 64 * w)
        if bits == 64:
            z[:, w] = torch.randint(-(1 << 63), (1 << 63) - 1, (m,), generator=g, dtype=torch.int64, device=DEV)
        else:
            z[:, w] = torch.randint(0, 1 << bits, (m,), generator=g, dtype=torch.int64, device=DEV)
    if case["circuit"] == "ghz":
        pair = torch.from_numpy(W.ints_to_words(_ghz_pair(n, x)[:2], n).view(np.int64)).to(DEV)
        z[:: max(1, m // 500)] = pair[0]
        z[1:: max(2, m // 400)] = pair[1]
    return z


# ---- what a user's program holds, and one pass -------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("circuit", "fused"):
        s["gates"], s["start"] = _circuit(case, seed)
        s["state"] = juqcs.State(case["n"], case["dtype"], device=DEV)
        s["z"] = _bitstrings(case, seed, s["start"])
        s["out"] = torch.empty(2 * case["read"], dtype=torch.float64, device=DEV)
    elif kind == "gates":
        s["calls"] = _drive(case, seed)
        s["state"] = juqcs.State(case["n"], case["dtype"], device=DEV)
        s["z"] = _bitstrings(dict(case, circuit=""), seed, 0)
        s["out"] = torch.empty(2 * case["read"], dtype=torch.float64, device=DEV)
    elif kind == "codec":
        count = 1 << case["n"]
        g = torch.Generator(device=DEV).manual_seed(seed)
        t = torch.float64 if case["dtype"] == "c128" else torch.float32
        s["src"] = torch.randn(2 * count, generator=g, dtype=t, device=DEV) * 2.0 ** (-case["n"] / 2)
        s["dst"] = torch.empty_like(s["src"])
        s["codes"] = torch.empty(2 * count, dtype=torch.int8, device=DEV)
        s["scales"] = torch.empty(count >> case["block"], dtype=torch.float32, device=DEV)
    elif kind == "batch":
        circuits = _batch_circuits(case, seed)
        s["batch"] = juqcs.Batch(circuits, device=DEV)
        rng = _rng(seed)
        z = np.stack([rng.integers(0, 1 << n, case["read"]) for n, _ in circuits])
        s["z"] = torch.from_numpy(z.astype(np.int64)).to(DEV)
        s["out"] = torch.empty(2 * z.size, dtype=torch.float64, device=DEV)
        s["norms"] = torch.empty(len(circuits), dtype=torch.float64, device=DEV)
    else:
        s["gates"], s["side"], x = _branch(case, seed)
        s["z"] = _branch_bitstrings(case, seed, x)
        s["out"] = torch.empty(2 * case["read"], dtype=torch.float64, device=DEV)
        s["work"] = juqcs.branch_workspace(case["n"], s["gates"], s["side"], s["z"].shape[1], case["read"], 0, False, DEV)
    return s


def _digits(case, x):
    """Amplitudes in the precision that they were computed in."""
    if case.get("dtype") == "c128":
        return x
    if case.get("dtype") == "enc2" and case["circuit"] != "ghz":
        return x.to(torch.bfloat16)
    return x.to(torch.float32)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("circuit", "fused"):
        st = s["state"]
        st.init(s["start"])
        if kind == "fused":
            st.run(s["gates"], mode="fused", fuse_k=5)
        else:
            st.run(s["gates"])
        st.amplitudes_device(s["z"], s["out"])
        r = {"amplitudes": _digits(case, s["out"])}
        if case["circuit"] == "ghz":
            r["expectations"] = st.expectations().astype(np.float64 if case["dtype"] == "c128" else np.float32)
        elif case["dtype"] != "enc2":
            r["norm"] = np.asarray([st.norm()]).astype(np.float64 if case["dtype"] == "c128" else np.float32)
        return r
    if kind == "gates":
        st = s["state"]
        st.init(0)
        for what, qs, m in s["calls"]:
            if what == "cu":
                st.apply_controlled(qs[0], qs[1], m)
            elif what == "2q":
                st.apply_2q(qs[0], qs[1], m)
            elif what == "fused":
                st.apply_fused(qs, m)
            else:
                st.apply_1q(qs[0], m)
        st.amplitudes_device(s["z"], s["out"])
        return {"amplitudes": _digits(case, s["out"])}
    if kind == "codec":
        dt = juqcs.DTYPES[case["dtype"]]
        count = s["codes"].numel() // 2
        juqcs.juqcs_encode2(s["src"], dt, count, case["block"], s["codes"], s["scales"])
        juqcs.juqcs_decode2(s["codes"], s["scales"], count, case["block"], s["dst"], dt)
        return {"codes": s["codes"], "scales": s["scales"], "decoded": s["dst"]}
    if kind == "batch":
        b = s["batch"]
        b.run()
        b.amplitudes_device(s["z"], case["read"], s["out"])
        b.norms_device(s["norms"])
        return {"amplitudes": s["out"].to(torch.float32), "norms": s["norms"].to(torch.float32)}
    juqcs.juqcs_branch_amplitudes_device(case["n"], s["gates"], s["side"], s["z"], s["out"], work=s["work"])
    return {"amplitudes": s["out"].to(torch.float32)}


# ---- the least a pass has to move and compute --------------------------------
#: Flops per amplitude of a gate: a dense 2x2 is a rotation and a phase (4 fused
#: multiply-adds per amplitude), a controlled phase multiplies a quarter of the
#: amplitudes, a sign flip and a permutation compute nothing.
DENSE1, PHASE2 = 8.0, 1.5


def _circuit_flops(gates):
    op = gates["op"]
    dense = np.isin(op, [W.OP_H, W.OP_U]).sum()
    return DENSE1 * float(dense) + PHASE2 * float((op == W.OP_CP).sum())


def work(case):
    kind = case["kind"]
    if kind in ("circuit", "fused", "gates"):
        amps = 2.0 ** case["n"]
        state = amps * AMP_BYTES[case["dtype"]]
        read = 24.0 * case["read"]
        if kind == "gates":  # each call is a pass of its own over the state
            flops = sum({"1q": 14.0, "diag": 3.0, "cu": 7.0}.get(w, 8.0 * m.shape[0]) for w, _, m in _drive(case, 0)) * amps
            part = sum({"diag": 1.0, "cu": 1.0}.get(w, 2.0) for w, _, m in _drive(case, 0))
            return {"bytes": state * (1 + part) + read, "flops": flops}
        # the state is written once and read for the norm or the expectation values
        return {"bytes": 2 * state + read, "flops": _circuit_flops(_circuit(case, 0)[0]) * amps}
    if kind == "codec":
        count = 2.0 ** case["n"]
        amp = AMP_BYTES[case["dtype"]]
        return {"bytes": count * (2 * amp + 4 + 8 / 2.0 ** case["block"]), "flops": 20.0 * count}
    if kind == "batch":
        circuits = _batch_circuits(case, 0)
        return {"bytes": sum(16.0 * 2.0 ** n for n, _ in circuits) + 24.0 * case["read"] * len(circuits),
                "flops": sum(_circuit_flops(g) * 2.0 ** n for n, g in circuits)}
    # part states: each part's gates run once at the least; the sum over the
    # branches multiplies one amplitude of every part per branch and bitstring
    gates, side, _ = _branch(case, 0)
    part = sum(2.0 ** int((side == p).sum()) for p in range(case["parts"]))
    words = (case["n"] + 63) // 64
    return {"bytes": 8.0 * part + (8.0 * words + 16.0) * case["read"],
            "flops": 8.0 * (case["parts"] - 1 if case["circuit"] == "ghz" else 2.0 ** case["size"]) * case["read"]
            + _circuit_flops(gates) / case["n"] * part}


# ---- 64-bit values ------------------------------------------------------------
#: Amplitude updates (gates times amplitudes) that take about 10 seconds in plain torch.
EXACT_UPDATES = 4.0e11
_H = np.array([[1, 1], [1, -1]]) / math.sqrt(2.0)
_ONE = {W.OP_H: _H, W.OP_X: np.array([[0, 1], [1, 0]]), W.OP_Y: np.array([[0, -1j], [1j, 0]]), W.OP_Z: np.diag([1, -1]),
        W.OP_S: np.diag([1, 1j]), W.OP_T: np.diag([1, np.exp(0.25j * np.pi)])}


def _matrix(g):
    if int(g["op"]) == W.OP_U:
        u = g["u"].reshape(2, 2, 2)
        return u[..., 0] + 1j * u[..., 1]
    return _ONE[int(g["op"])]


def _bit(psi, n, q, b):
    """The amplitudes with qubit q equal to b, as a view (last axis: the state)."""
    return psi.view(psi.shape[0], 1 << (n - 1 - q), 2, 1 << q)[:, :, b]


def _pair(psi, n, q0, b0, q1, b1):
    lo, hi = min(q0, q1), max(q0, q1)
    v = psi.view(psi.shape[0], 1 << (n - 1 - hi), 2, 1 << (hi - 1 - lo), 2, 1 << lo)
    return v[:, :, b1 if hi == q1 else b0, :, b1 if lo == q1 else b0]


def _apply1(psi, n, q, m):
    m = np.asarray(m, dtype=np.complex128)
    a, b = _bit(psi, n, q, 0), _bit(psi, n, q, 1)
    if m[0, 1] == 0 and m[1, 0] == 0:
        if m[0, 0] != 1:
            a.mul_(complex(m[0, 0]))
        b.mul_(complex(m[1, 1]))
        return
    x = complex(m[0, 0]) * a + complex(m[0, 1]) * b
    b.copy_(complex(m[1, 0]) * a + complex(m[1, 1]) * b)
    a.copy_(x)


def _apply_rows(psi, n, qs, m):
    """A dense matrix on qubits qs (row index sum_j b_(qs[j]) 2^j)."""
    k = len(qs)
    v = psi.view(psi.shape[0], *([2] * n))
    axes = [1 + n - 1 - q for q in reversed(qs)]
    rest = [i for i in range(n + 1) if i not in axes]
    p = v.permute(*axes, *rest).reshape(1 << k, -1)
    out = torch.from_numpy(np.ascontiguousarray(m, dtype=np.complex128)).to(psi.device) @ p
    inverse = np.argsort(axes + rest).tolist()
    shape = [2] * k + [v.shape[i] for i in rest]
    psi.copy_(out.view(shape).permute(*inverse).reshape(psi.shape))


def _simulate(psi, n, gates, where=None):
    """Runs gate records on psi (branches, 2^n); where: local number of each qubit."""
    for g in gates:
        op, q0, q1 = int(g["op"]), int(g["q0"]), int(g["q1"])
        q0 = q0 if where is None else where[q0]
        if q1 < 0:
            _apply1(psi, n, q0, _matrix(g))
            continue
        q1 = q1 if where is None else where[q1]
        if op == W.OP_CNOT:
            a, b = _pair(psi, n, q0, 1, q1, 0), _pair(psi, n, q0, 1, q1, 1)
            t = a.clone()
            a.copy_(b)
            b.copy_(t)
        else:
            _pair(psi, n, q0, 1, q1, 1).mul_(-1.0 if op == W.OP_CZ else complex(np.exp(1j * g["theta"])))


def _basis(n, x, dtype=torch.complex128):
    psi = torch.zeros((1, 1 << n), dtype=dtype, device=DEV)
    psi[0, x] = 1.0
    return psi


def _ri(a):
    return torch.view_as_real(a.contiguous()).reshape(-1)


def _ghz_amplitudes(hit0, hit1, sign):
    r = math.sqrt(0.5)
    re = hit0.to(torch.float64) * r + hit1.to(torch.float64) * (r * sign)
    return torch.stack([re, torch.zeros_like(re)], dim=-1).reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("circuit", "fused", "gates"):
        return _exact_state(case, seed)
    if kind == "codec":
        count = 1 << case["n"]
        g = torch.Generator(device=DEV).manual_seed(seed)
        t = torch.float64 if case["dtype"] == "c128" else torch.float32
        src = torch.randn(2 * count, generator=g, dtype=t, device=DEV) * 2.0 ** (-case["n"] / 2)
        return {"codes": None, "scales": src.view(-1, 2 << case["block"]).abs().amax(dim=1).double(), "decoded": None}
    if kind == "batch":
        circuits = _batch_circuits(case, seed)
        if sum(len(g) * (2.0 ** n + 3e5) for n, g in circuits) > EXACT_UPDATES:
            return None
        rng = _rng(seed)
        amps = []
        for n, g in circuits:
            psi = _basis(n, 0)
            _simulate(psi, n, g)
            amps.append((psi, n))
        z = [rng.integers(0, 1 << n, case["read"]) for n, _ in circuits]
        got = [_ri(psi[0][torch.from_numpy(x.astype(np.int64)).to(DEV)]) for (psi, n), x in zip(amps, z)]
        return {"amplitudes": torch.cat(got), "norms": torch.ones(len(circuits), dtype=torch.float64)}
    return _exact_branch(case, seed)


def _exact_state(case, seed):
    n = case["n"]
    if case["kind"] == "gates":
        if case["size"] * 2.0 ** n * 4 > EXACT_UPDATES:
            return None
        psi = _basis(n, 0)
        for what, qs, m in _drive(case, seed):
            if what in ("1q", "diag"):
                _apply1(psi, n, qs[0], m)
            else:
                if what == "cu":
                    full = np.eye(4, dtype=np.complex128)
                    full[1::2, 1::2] = m  # row b_c + 2 b_t
                    m = full
                _apply_rows(psi, n, qs, m)
        return {"amplitudes": _ri(psi[0][_bitstrings(dict(case, circuit=""), seed, 0)])}
    gates, start = _circuit(case, seed)
    z = _bitstrings(case, seed, start)
    if case["circuit"] == "ghz":
        s0, s1, sign = _ghz_pair(n, start)
        # <Q> = (1 - <sigma>) / 2, and every <sigma> of a GHZ state is 0
        return {"amplitudes": _ghz_amplitudes(z == s0, z == s1, sign), "expectations": np.full((n, 3), 0.5)}
    if case["circuit"] == "qft":
        # 2^(-n/2) exp(2 pi i x y / 2^n), the product reduced modulo 2^n in whole numbers
        lo = z & ((1 << 15) - 1)
        hi = z >> 15
        p = (start * lo + (((start * hi) & ((1 << n) - 1)) << 15)) & ((1 << n) - 1)
        a = p.to(torch.float64) * (2.0 * math.pi / (1 << n))
        return {"amplitudes": torch.stack([a.cos(), a.sin()], dim=-1).reshape(-1) * 2.0 ** (-n / 2), "norm": np.ones(1)}
    if len(gates) * (2.0 ** n + 1e6) > EXACT_UPDATES:
        return None
    psi = _basis(n, start)
    _simulate(psi, n, gates)
    r = {"amplitudes": _ri(psi[0][z])}
    if case["dtype"] != "enc2":
        r["norm"] = np.ones(1)
    return r


def _exact_branch(case, seed):
    n = case["n"]
    gates, side, x = _branch(case, seed)
    z = _branch_bitstrings(case, seed, x)
    if case["circuit"] == "ghz":
        pair = torch.from_numpy(W.ints_to_words(_ghz_pair(n, x)[:2], n).view(np.int64)).to(DEV)
        sign = _ghz_pair(n, x)[2]
        return {"amplitudes": _ghz_amplitudes((z == pair[0]).all(dim=1), (z == pair[1]).all(dim=1), sign)}
    # a crossing CZ is |0><0| I + |1><1| Z: projections of its first qubit in
    # one half, I or Z on its second in the other, summed over the projections
    half = n // 2
    crossing = [i for i, g in enumerate(gates) if g["q1"] >= 0 and side[g["q0"]] != side[g["q1"]]]
    m = len(crossing)
    if len(gates) / 2 * 2.0 ** (half + m + 1) > EXACT_UPDATES:
        return None
    states = []
    for p in (0, 1):
        where = {int(q): i for i, q in enumerate(np.flatnonzero(side == p))}
        psi = _basis(half, 0)
        last = 0
        for i in [*crossing, len(gates)]:
            mine = gates[last:i]
            _simulate(psi, half, mine[side[mine["q0"]] == p], where)
            if i < len(gates):
                a, b = int(gates["q0"][i]), int(gates["q1"][i])
                psi = psi.repeat_interleave(2, dim=0)
                q = where[a if side[a] == p else b]
                if side[a] == p:
                    even, odd = psi[0::2].clone(), psi[1::2].clone()
                    _bit(even, half, q, 1).zero_()
                    _bit(odd, half, q, 0).zero_()
                    psi[0::2], psi[1::2] = even, odd
                else:
                    odd = psi[1::2].clone()
                    _bit(odd, half, q, 1).mul_(-1.0)
                    psi[1::2] = odd
            last = i + 1
        states.append(psi)
    w = z[:, 0]
    z0, z1 = w & ((1 << half) - 1), w >> half
    out = torch.zeros(z.shape[0], dtype=torch.complex128, device=DEV)
    for b in range(1 << m):
        out += states[0][b][z0] * states[1][b][z1]
    return {"amplitudes": _ri(out)}
