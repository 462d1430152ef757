"""The specialized kernels of hs_simulate's sweeps, run on the host like the
part kernels of test_spec_cpu.py: controls, phases and sign changes whose
qubits lie on lane, wave or register bits or outside the tile, factors held
per lane, split re-layouts, and tiles narrower than a wavefront."""

import os
import re
import shutil
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import test_spec_cpu as host  # noqa: E402
from oracle import statevector as sv  # noqa: E402
from paper_2205_06973_amd import hisv  # noqa: E402
from paper_2205_06973_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


class Sweeps:
    """A plan's sweeps where the host runner expects a plan's parts."""

    def __init__(self, plan, dtype):
        self.src = [plan.sweep_source(i, dtype) for i in range(plan.num_sweeps(dtype, "part_spec"))]
        self.num_parts = len(self.src)

    def part_source(self, i, dtype):
        return self.src[i]

    def part_descriptors(self, i, dtype, mode):
        m = len(re.findall(r"b = \(\(b >> ", self.src[i]))
        block = int(re.search(r"__launch_bounds__\((\d+)\)", self.src[i]).group(1))
        return [m, 0, (block // 64).bit_length() - 1], None, None


def run(n, gates, dtype, k, tmp_path, seed=3):
    plan = hisv.Plan.partition(hisv.Circuit(n, gates), k, "greedy", 0, 4)
    sweeps = Sweeps(plan, dtype)
    assert sweeps.num_parts < plan.num_parts
    psi0 = host.random_state(n, seed)
    got = host.run_on_host(sweeps, n, dtype, psi0, tmp_path)
    np.testing.assert_allclose(got, sv.simulate(n, gates, psi0), atol=host.TOL[dtype], rtol=0)
    return "\n".join(sweeps.src)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_every_kind(dtype, tmp_path):
    gates = wl.random_circuit(14, 180, sv.ONE_QUBIT + sv.TWO_QUBIT, seed=71)
    hisv.hs_tune(f"spec_rb_{dtype}", 3)  # small tiles then have wave bits
    try:
        src = run(14, gates, dtype, 5, tmp_path)
    finally:
        hisv.hs_tune(f"spec_rb_{dtype}", {"c64": 5, "c128": 4}[dtype])
    # conditions on lane, wave and outer bits, and the lanes' factor, all occur
    for x in ("on = ((lane", "if (((wave", "if (((tb", "fr *="):
        assert x in src, x


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_controls_and_phases(dtype, tmp_path):
    """Few gates need registers: nearly every control and phase is a condition."""
    n = 14
    rng = np.random.default_rng(5)
    gates = []
    for layer in range(6):
        for q in rng.permutation(n)[:4]:
            gates.append(("h", int(q), -1, ()))
        for _ in range(14):
            a, b = (int(v) for v in rng.choice(n, 2, replace=False))
            name = ("cz", "cp", "cx", "cx")[int(rng.integers(4))]
            gates.append((name, a, b, (0.3 + 0.1 * layer,) if name == "cp" else ()))
        gates.append(("rz", int(rng.integers(n)), -1, (0.7,)))
        gates.append(("t", int(rng.integers(n)), -1, ()))
    run(n, gates, dtype, 4, tmp_path)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_qft(dtype, tmp_path):
    run(13, wl.qft_circuit(13), dtype, 4, tmp_path)


@pytest.mark.parametrize("n", [3, 5, 8])
def test_small_states(n, tmp_path):
    gates = wl.random_circuit(n, 60, ("h", "rz", "u3", "cx", "cz", "cp", "swap"), seed=n)
    run(n, gates, "c64", 2, tmp_path)


def test_split_relayouts(tmp_path):
    hisv.hs_tune("spec_lds_limit_kib", 16)
    hisv.hs_tune("spec_rb_c128", 5)  # tiles of 11 qubits, 32 KiB
    try:
        src = run(15, wl.random_circuit(15, 140, sv.ONE_QUBIT + sv.TWO_QUBIT, seed=72), "c128", 4, tmp_path)
    finally:
        hisv.hs_tune("spec_lds_limit_kib", 64)
        hisv.hs_tune("spec_rb_c128", 4)
    assert "sr0" in src


def test_only_diagonals(tmp_path):
    """Sweeps whose gates need no register at all."""
    n = 12
    gates = [(("cz", "cp")[i % 2], i % n, (i * 5 + 1) % n, (0.2 * i,) if i % 2 else ())
             for i in range(60) if i % n != (i * 5 + 1) % n] + [("s", q, -1, ()) for q in range(n)]
    run(n, gates, "c64", 3, tmp_path)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_gate_wider_than_a_stage_is_refused(dtype):
    """With one register bit a two-qubit gate fits no stage: the parts refuse
    it, and no sweep takes it (CX and CZ, whose conditions would need fewer)."""
    n = 14
    gates = [(("cx", "cz")[i % 2], i % n, (i * 5 + 1) % n, ()) for i in range(40) if i % n != (i * 5 + 1) % n]
    plan = hisv.Plan.partition(hisv.Circuit(n, gates), 5, "dfs")
    default = {"c64": 5, "c128": 4}[dtype]
    hisv.hs_tune(f"spec_rb_{dtype}", 1)
    try:
        assert plan.num_sweeps(dtype, "part_spec") == plan.num_parts
        for source in (plan.part_source, plan.sweep_source):
            with pytest.raises(hisv.HisvError, match="HS_E_UNSUPPORTED"):
                source(0, dtype)
    finally:
        hisv.hs_tune(f"spec_rb_{dtype}", default)
