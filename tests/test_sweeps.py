"""hs_simulate cuts a plan's gates into sweeps that fill a kernel tile: the
result against the oracle and against the plan's own parts, at the edges of
the tile widths, and the calls that stay as they were."""

import numpy as np
import pytest

from oracle import statevector as sv
from paper_2205_06973_amd import hisv
from paper_2205_06973_amd import workloads as wl

KINDS = ("h", "u3", "rz", "rx", "cx", "cz", "cp", "swap", "ccx", "cswap")
TOL = {"c64": 2e-5, "c128": 1e-12}  # the bars of the parity tests, at most 10^4 gates


def make(n, gates, k, strategy="closure"):
    return hisv.Plan.partition(hisv.Circuit(n, gates), k, strategy, 0, 8)


def test_sweeps_are_counted():
    n, gates = wl.layered28(0, n=24, layers=12)
    plan = make(n, gates, 6)
    for dtype in ("c64", "c128"):
        for mode in ("part_lds", "part_spec"):
            assert 1 <= plan.num_sweeps(dtype, mode) <= 0.9 * plan.num_parts
        assert plan.sweep_source(plan.num_sweeps(dtype) - 1, dtype).startswith("#ifndef")
        with pytest.raises(hisv.HisvError):
            plan.sweep_source(plan.num_sweeps(dtype), dtype)
    assert plan.num_sweeps("c64", "part_fused") <= plan.num_parts
    assert plan.num_sweeps("c64", "gate_per_pass") == len(gates)


def test_one_part_is_kept():
    n, gates = 9, wl.random_circuit(9, 40, ("h", "cx"), 1)
    plan = make(n, gates, 9)
    assert plan.num_parts == 1 and plan.num_sweeps("c64", "part_lds") == 1


def test_a_part_without_a_tile_is_still_refused():
    n = 16
    gates = [("h", q, -1, ()) for q in range(n)] + [("cx", q, q + 1, ()) for q in range(n - 1)]
    plan = hisv.Plan.from_assignment(hisv.Circuit(n, gates), 16, [0] * 16 + [1] * (len(gates) - 16))
    assert plan.num_parts == 2
    with pytest.raises(hisv.HisvError) as e:
        plan.part_layout(0)
    assert e.value.code == "HS_E_UNSUPPORTED"
    assert plan.num_sweeps("c64", "part_lds") == 2  # no regrouping: hs_simulate reports the part


@pytest.mark.gpu
@pytest.mark.parametrize("n", [3, 6, 10, 11, 13, 14, 17])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_sweeps_gpu(n, dtype):
    torch = pytest.importorskip("torch")
    gates = wl.random_circuit(n, 150, KINDS, 10 + n)
    x = wl.random_basis_index(n, n)
    want = sv.simulate(n, gates, sv.basis_state(n, x))
    buf = torch.empty(1 << n, dtype={"c64": torch.complex64, "c128": torch.complex128}[dtype], device="cuda")
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    k = min(n, 4)
    plan = make(n, gates, k)
    for mode in ("part_lds", "auto", "part_spec", "auto"):  # AUTO before and after the kernels are built
        print(f"[case] n={n} {dtype} {mode}", flush=True)
        st.set_basis(x)
        st.simulate(plan, mode)
        np.testing.assert_allclose(st.amplitudes(), want, atol=TOL[dtype], rtol=0, err_msg=mode)
    assert plan.specialized(dtype)
    for mode in ("part_lds", "part_spec"):
        st.set_basis(x)
        for i in range(plan.num_parts):
            st.simulate_part(plan, i, mode)
        np.testing.assert_allclose(st.amplitudes(), want, atol=TOL[dtype], rtol=0, err_msg=f"parts {mode}")
    st.close()


def test_dense_pieces_are_counted():
    n, gates = 16, wl.dressed_pairs_circuit(16, 200, 1, span=5, dwell=16)
    plan = make(n, gates, 5)
    for dtype in ("c64", "c128"):
        assert plan.num_sweeps(dtype, "part_fused") <= 0.9 * plan.num_parts
    # a part without a fused form: nothing is cut anew, hs_simulate reports it
    wide = make(n, wl.layered_circuit(n, 3, 1), 8)
    assert wide.num_sweeps("c64", "part_fused") == wide.num_parts


@pytest.mark.gpu
@pytest.mark.parametrize("n", [8, 9, 10, 11, 12, 15])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_dense_pieces_gpu(n, dtype):
    """Every width of the fused kernels from the smallest state they take
    (fewer tiles than the waves of one workgroup, one chunk, several chunks),
    part by part and cut anew."""
    torch = pytest.importorskip("torch")
    buf = torch.empty(1 << n, dtype={"c64": torch.complex64, "c128": torch.complex128}[dtype], device="cuda")
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    for w in range(4, min(7, n - 4) + 1):
        for seed, gates in ((1, wl.dressed_pairs_circuit(n, 60, w, span=4, dwell=9)),
                            (2, wl.random_circuit(n, 80, ("h", "u3", "rz", "cx", "cp", "swap"), w))):
            x = wl.random_basis_index(n, seed)
            want = sv.simulate(n, gates, sv.basis_state(n, x))
            plan = make(n, gates, w)
            print(f"[case] n={n} {dtype} w={w} seed={seed} {plan.num_parts} parts", flush=True)
            st.set_basis(x)
            st.simulate(plan, "part_fused")
            np.testing.assert_allclose(st.amplitudes(), want, atol=TOL[dtype], rtol=0, err_msg=f"pieces w={w}")
            st.set_basis(x)
            for i in range(plan.num_parts):
                st.simulate_part(plan, i, "part_fused")
            np.testing.assert_allclose(st.amplitudes(), want, atol=TOL[dtype], rtol=0, err_msg=f"parts w={w}")
    st.close()


@pytest.mark.gpu
def test_a_part_without_a_tile_is_refused_gpu():
    torch = pytest.importorskip("torch")
    n = 16
    gates = [("h", q, -1, ()) for q in range(n)] + [("cx", q, q + 1, ()) for q in range(n - 1)]
    plan = hisv.Plan.from_assignment(hisv.Circuit(n, gates), 16, [0] * 16 + [1] * (len(gates) - 16))
    buf = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
    st = hisv.State.wrap_tensor(buf, torch.cuda.current_stream())
    st.set_basis(0)
    for mode in ("part_lds", "part_spec", "auto", "part_fused"):
        with pytest.raises(hisv.HisvError) as e:
            st.simulate(plan, mode)
        assert e.value.code == "HS_E_UNSUPPORTED"
    st.close()
