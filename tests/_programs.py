"""Register-resident tile programs planned and run on the host: the planner's
sources and tests/programs/interpreter.cpp, built with the host compiler."""
import ctypes as ct
import os
import subprocess

import numpy as np

from paper_1912_03243_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_03243_amd", "csrc")


class Report(ct.Structure):
    _fields_ = [("passes", ct.c_int64), ("races", ct.c_int64), ("misplaced", ct.c_int64),
                ("blocks", ct.c_int64), ("least", ct.c_double), ("most", ct.c_double),
                ("layers", ct.c_int64), ("misc", ct.c_int64), ("stages", ct.c_int64)]


class Programs:
    def __init__(self, folder):
        srcs = [os.path.join(ROOT, "tests", "programs", "interpreter.cpp"),
                os.path.join(CSRC, "block.cpp"), os.path.join(CSRC, "planner.cpp")]
        flags = ["-O2", "-std=c++17", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                 "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
        objs = [os.path.join(folder, os.path.basename(s) + ".o") for s in srcs]
        jobs = [subprocess.Popen(["g++", *flags, "-c", s, "-o", o]) for s, o in zip(srcs, objs)]
        assert [j.wait() for j in jobs] == [0] * len(jobs)
        lib = os.path.join(folder, "programs.so")
        subprocess.run(["g++", "-shared", "-pthread", *objs, "-o", lib], check=True)
        self.lib = ct.CDLL(lib)

    def run(self, n, circ, dtype="c128", low=None, tile=None, pass_gates=0, relabel=0, block=0, psi=None,
            plan_only=False):
        """(state, report) of the circuit run from psi (default |0...0>); the
        state is None where the planner leaves the circuit to the fused passes."""
        tile = min(n, 13) if tile is None else tile
        low = min(tile, {"c128": 5, "c64": 7, "enc2": max(block, 7)}[dtype]) if low is None else low
        v = np.zeros(1 << n, np.complex128)
        if psi is None:
            v[0] = 1
        else:
            v[:] = psi
        g = np.ascontiguousarray(circ)
        rep = Report()
        rc = self.lib.run_program(ct.c_int(n), ct.c_void_p(g.ctypes.data), ct.c_int64(g.size),
                                  ct.c_int(dtype == "c128"), ct.c_int(low), ct.c_int(tile),
                                  ct.c_int(pass_gates), ct.c_int(relabel), ct.c_int(block),
                                  ct.byref(ct.c_uint64(0)) if psi is None else None,
                                  ct.c_void_p(None if plan_only else v.ctypes.data), ct.byref(rep))
        assert rc in (0, 1), rc
        return (v if rc == 0 else None), rep


def signed_rotations(count, qubits, n, theta=None):
    """Rotations that all carry a sign or a phase of a qubit that does not rotate any more."""
    recs = [W.gate(W.OP_H, q) for q in range(4, n)]
    for i in range(count):
        for q in range(qubits):
            other = 4 + (i + q) % (n - 4)
            recs.append(W.gate(W.OP_H, q))
            recs.append(W.gate(W.OP_CZ, q, other) if theta is None else W.gate(W.OP_CP, q, other, theta=theta))
    return W.concat(*recs)


# (dtype, qubits, repetitions, qubits that rotate, angle of the controlled phases or None: CZ)
SIGNED = [("c64", 13, 300, 1, None), ("c64", 13, 300, 1, 0.3), ("c64", 14, 300, 2, None), ("c64", 13, 100, 4, 0.3),
          ("c128", 12, 2300, 1, None), ("c128", 13, 1200, 1, 0.3)]
