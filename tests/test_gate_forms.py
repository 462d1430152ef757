"""One-qubit runs are applied as scaled 2x2 forms (unit entries cost no
multiplication), with a factor left pending over gates it commutes with and a
scalar applied once per part.  Every form, on every register bit, in front
of every kind of two-qubit gate and at the end of a part, against the oracle:
on the descriptors on the CPU, on both part kernels on the GPU.

Tolerances: a run of 40 gates rounds each amplitude a few hundred times;
1e-12 (complex128) and 2e-5 (complex64) are the bars of the parity tests.
"""

import math
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from oracle import statevector as sv  # noqa: E402
from paper_2205_06973_amd import hisv  # noqa: E402
from replay import replay_plan  # noqa: E402

TOL = {"c64": 2e-5, "c128": 1e-12}
PI = math.pi
RUNS = {
    "h": [("h", ())],
    "real": [("ry", (0.7,))],
    "real_large": [("ry", (2.9,))],           # |cos| < 1/8: unit entries off the diagonal
    "imaginary": [("rx", (1.1,))],
    "imaginary_large": [("rx", (3.0,))],
    "dense": [("u3", (0.9, 0.3, 1.2))],
    "dense_large": [("u3", (2.4, 0.4, 5.1))],
    "dense_anti": [("u3", (PI - 1e-3, 0.4, 5.1))],
    "diagonal": [("rz", (0.8,)), ("t", ())],
    "flip": [("rz", (0.8,)), ("x", ())],
    "y": [("y", ())],
    "undone": [("h", ()), ("h", ())],         # the identity up to rounding
    "long": [("rz", (0.3,)), ("h", ()), ("rz", (1.7,)), ("h", ()), ("s", ())],
}
PAIRS = ["cx", "xc", "cz", "cp", "swap", None]


def _run(gates, name, q):
    gates.extend((g, q, -1, p) for g, p in RUNS[name])


def circuit(name, pair, n):
    """The run on every qubit (so on every register bit), `pair` on
    neighbours, and the run again, over a state with no zero amplitude."""
    gates = [("u3", q, -1, (0.4 + 0.1 * q, 0.2 * q, 1.0 - 0.3 * q)) for q in range(n)]
    for shift in (0, 1):
        for q in range(n):
            _run(gates, name, q)
        for q in range(shift, n - 1, 2):
            if pair == "xc":
                gates.append(("cx", q + 1, q, ()))
            elif pair:
                gates.append((pair, q, q + 1, (0.6,) if pair == "cp" else ()))
    for q in range(n):
        _run(gates, name, q)
    return gates


@pytest.mark.parametrize("name", list(RUNS))
def test_forms_replay(name):
    n = 11
    for pair in PAIRS:
        gates = circuit(name, pair, n)
        psi0 = sv.basis_state(n, 5)
        want = sv.simulate(n, gates, psi0)
        for dtype, mode in (("c64", "part_lds"), ("c128", "part_spec")):
            plan = hisv.Plan.partition(hisv.Circuit(n, gates), 5, "greedy", 0, 4)
            got, _ = replay_plan(plan, n, psi0, dtype, mode)
            np.testing.assert_allclose(got, want, atol=1e-12, rtol=0, err_msg=f"{pair} {dtype} {mode}")


def test_growth_stays_bounded():
    """Scaled forms enlarge the amplitudes on the way by at most 2^10 times
    one op's factor of 8; 300 Hadamards would reach 2^150 unbounded."""
    n = 6
    gates = [g for i in range(50) for q in range(n)
             for g in (("h", q, -1, ()), ("cz", q, (q + 1 + i % 4) % n, ()))]
    plan = hisv.Plan.partition(hisv.Circuit(n, gates), n, "nat", 0, 1)
    assert plan.num_parts == 1
    for mode in ("part_lds", "part_spec"):
        ops = plan.part_descriptors(0, "c64", mode)[2]
        grow = 0.0
        for op in ops:
            if int(op[0]) in (0, 1):
                c = op[3:11]
                m = (c[0::2] + 1j * c[1::2] if int(op[0]) == 0 else c[:4]).reshape(2, 2)
                grow += math.log2(np.linalg.norm(m, 2))
            elif int(op[0]) == 2:  # a diagonal or a dense 4 x 4 may carry the scalar
                grow += math.log2(abs(complex(op[3], op[4])))
            elif int(op[0]) == 9:
                grow += math.log2(np.linalg.norm((op[3:35:2] + 1j * op[4:35:2]).reshape(4, 4), 2))
            assert -14.0 < grow < 14.0
        assert abs(grow) < 1e-9


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("name", list(RUNS))
def test_forms_gpu(name, dtype):
    torch = pytest.importorskip("torch")
    n = 11
    buf = torch.empty(1 << n, dtype={"c64": torch.complex64, "c128": torch.complex128}[dtype], device="cuda")
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    # one kernel build a run: the pairs one after the other
    gates = [g for pair in PAIRS for g in circuit(name, pair, n)]
    want = sv.simulate(n, gates, sv.basis_state(n, 5))
    for mode, fuse2 in (("part_lds", 1), ("part_lds", 0), ("part_spec", 1)):
        print(f"[case] {name} {dtype} {mode} fuse2={fuse2}", flush=True)
        hisv.hs_tune("fuse2", fuse2)
        try:
            plan = hisv.Plan.partition(hisv.Circuit(n, gates), 5, "greedy", 0, 4)
            st.set_basis(5)
            st.simulate(plan, mode)
            got = st.amplitudes()
        finally:
            hisv.hs_tune("fuse2", 1)
        np.testing.assert_allclose(got, want, atol=TOL[dtype], rtol=0, err_msg=mode)
    st.close()
