"""Gate sweeps and readouts on the shapes their vector forms split at: qubit 0
and the lowest qubits, states of one to a few vectors, a complex64 state that
is not 16-byte aligned, and reads around the staging chunk."""

import numpy as np
import pytest

from oracle import statevector as sv
from paper_2205_06973_amd import hisv
from paper_2205_06973_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TDT = {"c64": torch.complex64, "c128": torch.complex128}
TOL = {"c64": 2e-5, "c128": 1e-12}  # the bars of the parity tests


def state(n, dtype, offset):
    """A state `offset` amplitudes into its allocation, filled from a seed."""
    g = torch.Generator().manual_seed(n + offset)
    host = torch.randn(1 << n, dtype=torch.complex128, generator=g) / 2 ** (n / 2)
    buf = torch.empty((1 << n) + offset, dtype=TDT[dtype], device="cuda")[offset:]
    buf.copy_(host)
    return buf, buf.cpu().numpy().astype(np.complex128)


@pytest.mark.parametrize("dtype,offset", [("c64", 0), ("c64", 1), ("c128", 0)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 9])
def test_gate_sweeps(n, dtype, offset):
    buf, psi0 = state(n, dtype, offset)
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    gates = []
    for q in range(n):
        gates += [("h", q, -1, ()), ("rz", q, -1, (0.4 + q,)), ("t", q, -1, ()), ("x", q, -1, ()),
                  ("z", q, -1, ()), ("u3", q, -1, (0.3, 1.1, 0.2 * q)), ("y", q, -1, ())]
        for r in range(n):
            if r != q:
                gates += [("cx", q, r, ()), ("cz", q, r, ()), ("cp", q, r, (0.7,)), ("swap", q, r, ())]
    print(f"[case] n={n} {dtype} offset={offset} {len(gates)} gates", flush=True)
    st.simulate_gate_per_pass(hisv.Circuit(n, gates))
    np.testing.assert_allclose(st.amplitudes(), sv.simulate(n, gates, psi0), atol=TOL[dtype], rtol=0)
    st.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_reads_around_the_chunk(dtype):
    n = 19
    buf, psi = state(n, dtype, 0)
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    chunk = 1 << 16  # amplitudes in one staging buffer
    for count in (1, chunk - 1, chunk, chunk + 1, 3 * chunk + 5):
        for first in (0, 7, (1 << n) - count):
            print(f"[case] {dtype} first={first} count={count}", flush=True)
            assert np.array_equal(st.amplitudes(first, count), psi[first:first + count])
            got = st.probabilities(first, 2 * count if first == 0 else count)
            want = psi[first:first + got.size]
            # a fused multiply-add against two roundings: one unit in the last place
            np.testing.assert_allclose(got, want.real ** 2 + want.imag ** 2, rtol=4e-16, atol=0)
    rng = np.random.default_rng(3)
    for count in (1, (1 << 15) - 1, 1 << 15, (1 << 15) + 1, 100_000):
        idx = rng.integers(0, 1 << n, size=count, dtype=np.uint64)
        assert np.array_equal(st.amplitudes_at(idx), psi[idx.astype(np.int64)])
    exact = float(np.sum(psi.real ** 2 + psi.imag ** 2))
    assert abs(st.norm() - exact) <= 1e-12 * exact and st.norm() == st.norm_noalloc()
    st.close()
