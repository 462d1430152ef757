"""The work that programs built on this library have it do, as timed cases.

A case is one pass of one of four paths:

* ``circuit``  set the state to a basis state and run a partitioned circuit
  on it (``State.set_basis`` + ``State.simulate``), the library's main call;
* ``gates``    the same circuit without a partition, one sweep per gate
  (``State.simulate_gate_per_pass``);
* ``readout``  what follows a simulation: the norm, the probabilities of a
  range of basis states and the amplitudes at sampled indices;
* ``serve``    a burst of small and middle-sized circuits through the
  continuous-batching server: submit, wait, read every state, release.

The circuits are the generators of ``workloads.py`` at the sizes of bench.py
and of the tests, between 8 and 32 qubits.  A case's ``circuit`` number seeds
its circuit, which a program keeps (with its plan and its kernels) while the
input state changes; the seed given to ``prepare`` draws the input.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2205_06973_amd import hisv
from paper_2205_06973_amd import workloads as wl

_TORCH = {"c64": torch.complex64, "c128": torch.complex128}
_BYTES = {"c64": 8, "c128": 16}


def listed():
    return [
        # A small circuit run once from Python and read back: 12 qubits, 200
        # gates, k = 4 (the circuit of the smoke run and of the parity tests),
        # on the interpreter.  Launches and latency.
        dict(name="random12_c128_interp", path="circuit", family="random12", n=12, gates=200, k=4,
             strategy="dfs", trials=16, dtype="c128", mode="part_lds", circuit=0),
        # A 20-qubit variational-style circuit evaluated over and over, with
        # specialized kernels: the state fits the caches.
        dict(name="layered20_c64_auto", path="circuit", family="layered", n=20, layers=30, k=6,
             strategy="closure", trials=16, dtype="c64", mode="auto", specialize=True, circuit=1),
        # A circuit that is run once: no kernels are built for it and the
        # interpreter runs it, with the partitioner's defaults.
        dict(name="layered25_c128_interp", path="circuit", family="layered", n=25, layers=24, k=7,
             strategy="closure", trials=1, dtype="c128", mode="part_lds", circuit=2),
        # 28 qubits, 40 layers, k = 6: the layered circuit of the benchmark.
        dict(name="layered28_c64_spec", path="circuit", family="layered", n=28, layers=40, k=6,
             strategy="closure", trials=16, dtype="c64", mode="part_spec", specialize=True, circuit=0),
        # The benchmark's random circuit in single precision (8 GiB state).
        dict(name="random30_c64_spec", path="circuit", family="random34", n=30, gates=1000, k=7,
             strategy="closure", trials=16, dtype="c64", mode="part_spec", specialize=True, circuit=0),
        # The same distribution in the headline's precision, the largest state
        # here (32 GiB), on an odd number of qubits.
        dict(name="random31_c128_spec", path="circuit", family="random34", n=31, gates=1000, k=7,
             strategy="closure", trials=16, dtype="c128", mode="part_spec", specialize=True, circuit=1),
        # The 32-qubit QFT of a random basis state under the multi-level
        # partition: few parts on the widest tiles.
        dict(name="qft32_c64_multilevel", path="circuit", family="qft", n=32, k=0, strategy="closure",
             trials=16, dtype="c64", mode="part_spec", specialize=True, circuit=0),
        # Deep dense parts, which AUTO sends to the matrix cores.
        dict(name="dressed28_c64_auto", path="circuit", family="dressed", n=28, gates=600, k=5,
             strategy="closure", trials=16, dtype="c64", mode="auto", circuit=0),
        dict(name="dressed29_c128_auto", path="circuit", family="dressed", n=29, gates=400, k=5,
             strategy="closure", trials=16, dtype="c128", mode="auto", circuit=1),
        # A short circuit without a plan: one sweep per gate.
        dict(name="gates25_c64", path="gates", family="random34", n=25, gates=60, dtype="c64", circuit=3),
        # Readout of a 27-qubit state: norm, a range of probabilities, shots.
        dict(name="readout27_c64", path="readout", n=27, dtype="c64", count=(1 << 20) + 77, shots=4096),
        # Sixteen requests at once through the server, 10 to 19 qubits.
        dict(name="serve16", path="serve", requests=16, n_lo=10, n_hi=19, layers_lo=20, layers_hi=60, circuit=0),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["circuit"] * 7 + ["gates", "readout", "serve"])
    dtype = rng.choice(["c64", "c128"])
    circuit = rng.randrange(1 << 20)
    if path == "gates":
        return dict(path=path, family=rng.choice(["random34", "layered"]), n=rng.randint(9, 27),
                    gates=rng.randint(20, 90), layers=1 + rng.randrange(3), dtype=dtype, circuit=circuit)
    if path == "readout":
        n = rng.randint(12, 29)
        return dict(path=path, n=n, dtype=dtype, count=min(log_int(100, 1 << 21), (1 << n) - 1),
                    shots=log_int(10, 100_000), circuit=circuit)
    if path == "serve":
        hi = rng.randint(12, 20)
        return dict(path=path, requests=rng.randint(3, 20), n_lo=10, n_hi=hi, layers_lo=20,
                    layers_hi=rng.randint(30, 70), circuit=circuit)
    kind = rng.choice(["interp", "spec", "spec", "multilevel", "dressed"])
    case = dict(path=path, dtype=dtype, circuit=circuit, strategy="closure", trials=16)
    if kind == "dressed":
        case.update(family="dressed", n=rng.randint(14, 29), gates=rng.randint(100, 600), k=rng.choice([4, 5, 6]),
                    mode=rng.choice(["auto", "auto", "part_fused"]))
        return case
    if kind == "interp":
        case.update(family=rng.choice(["random12", "random34", "layered", "adder"]), n=rng.randint(8, 26),
                    gates=log_int(60, 600), layers=log_int(4, 40), k=rng.randint(4, 7), mode="part_lds",
                    strategy=rng.choice(["dfs", "greedy", "closure", "dagp"]))
    else:
        case.update(family=rng.choice(["random34", "layered", "qft", "adder"]), n=rng.randint(14, 30),
                    gates=log_int(100, 600), layers=log_int(4, 24),
                    k=0 if kind == "multilevel" else rng.randint(5, 7),
                    mode=rng.choice(["part_spec", "auto"]), specialize=True)
    if case["family"] == "adder":
        case["n"] -= case["n"] % 2  # 2 * bits + 2
    return case


def _gates(case, n):
    f, c = case["family"], case["circuit"]
    if f == "random12":
        return wl.random_circuit(n, case["gates"], wl.RANDOM12_KINDS, c)
    if f == "random34":
        return wl.random_circuit(n, case["gates"], wl.RANDOM34_KINDS, c)
    if f == "layered":
        return wl.layered_circuit(n, case["layers"], c)
    if f == "qft":
        return wl.qft_circuit(n)
    if f == "adder":
        return wl.adder_circuit((n - 2) // 2)[1]
    return wl.dressed_pairs_circuit(n, case["gates"], c, span=5, dwell=16)


def _requests(case, seed):
    """Sizes and precisions from the case, the circuits themselves from the seed."""
    reqs = wl.serving_stream(case["requests"], 40.0, case["circuit"], (case["n_lo"], case["n_hi"]),
                             (case["layers_lo"], case["layers_hi"]))
    return [(r.n, r.dtype, wl.layered_circuit(r.n, r.layers, seed * 1009 + i)) for i, r in enumerate(reqs)]


def _random_state(case, seed):
    """A dense normalised state, as after a circuit."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    N = 1 << case["n"]
    x = torch.randn(N, dtype=_TORCH[case["dtype"]], device="cuda", generator=g)
    return x.mul_(1.0 / math.sqrt(N))


def _readout_where(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    first = int(rng.integers(0, (1 << case["n"]) - case["count"] + 1))
    return first, rng.integers(0, 1 << case["n"], size=case["shots"], dtype=np.uint64)


def prepare(case, seed):
    path = case["path"]
    if path == "serve":
        return dict(case=case, server=hisv.Server(0, 4), requests=_requests(case, seed))
    stream = torch.cuda.current_stream()
    if path == "readout":
        first, idx = _readout_where(case, seed)
        buf = _random_state(case, seed)
        return dict(case=case, buf=buf, state=hisv.State.wrap_tensor(buf, stream), first=first, idx=idx)
    n, dtype = case["n"], case["dtype"]
    gates = _gates(case, n)
    circ = hisv.Circuit(n, gates)
    buf = torch.empty(1 << n, dtype=_TORCH[dtype], device="cuda")
    s = dict(case=case, circuit=circ, buf=buf, state=hisv.State.wrap_tensor(buf, stream),
             x=wl.random_basis_index(n, seed))
    if path == "circuit":
        if case["k"]:
            s["plan"] = hisv.Plan.partition(circ, case["k"], case["strategy"], 0, case["trials"])
        else:
            s["plan"] = hisv.Plan.partition_multilevel(circ, None, 6, case["strategy"], 0, case["trials"], dtype)
        if case.get("specialize"):
            s["plan"].specialize(dtype)
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "serve":
        srv = s["server"]
        k = {"c64": hisv.hs_max_part_qubits("c64"), "c128": hisv.hs_max_part_qubits("c128")}
        whole = {"c64": 14, "c128": 13}
        tickets = [srv.submit(n, gates, dtype, 0, n if n <= whole[dtype] else k[dtype], "closure")
                   for n, dtype, gates in s["requests"]]
        out = []
        for t, (n, _, _) in zip(tickets, s["requests"]):
            srv.wait(t)
            out.append(srv.amplitudes(t, 0, 1 << n))
            srv.release(t)
        return out
    st = s["state"]
    if path == "readout":
        return {"norm": st.norm(), "probs": st.probabilities(s["first"], case["count"]),
                "amps": st.amplitudes_at(s["idx"])}
    st.set_basis(s["x"])
    if path == "gates":
        st.simulate_gate_per_pass(s["circuit"])
    else:
        st.simulate(s["plan"], case["mode"])
    return st.amplitudes() if case["n"] <= 12 else s["buf"]


# Real operations per amplitude of one gate: dense 2x2 14, rotations about one
# axis 6, real 2x2 4, a phase on half of the amplitudes 3, on a quarter 1.5.
_FLOPS = {"h": 4, "x": 0, "rx": 6, "ry": 6, "rz": 6, "p": 3, "u3": 14, "cx": 0, "cz": 0.5, "cp": 1.5,
          "swap": 0, "ccx": 0}


def _flops(n, gates):
    return sum(_FLOPS[g[0]] for g in gates) * float(1 << n)


def work(case):
    path = case["path"]
    if path == "serve":
        total = {"bytes": 0.0, "flops": 0.0}
        for n, dtype, gates in _requests(case, 0):
            total["bytes"] += 2.0 * (1 << n) * _BYTES[dtype] + 16.0 * (1 << n)  # the state, and its copy read out
            total["flops"] += _flops(n, gates)
        return total
    N = float(1 << case["n"])
    size = N * _BYTES[case["dtype"]]
    if path == "readout":
        return {"bytes": size + 8.0 * case["count"] + 24.0 * case["shots"], "flops": 4.0 * N}
    return {"bytes": 2.0 * size, "flops": _flops(case["n"], _gates(case, case["n"]))}


# --- the same results in 64 bits, in plain torch ------------------------------

def _sub(psi, n, bits):
    """The view of psi with qubit q fixed to bits[q] for every q in bits."""
    shape, index, top = [], [], n
    for q in sorted(bits, reverse=True):
        shape += [1 << (top - 1 - q), 2]
        index += [slice(None), bits[q]]
        top = q
    return psi.view(*shape, 1 << top)[tuple(index)]


def _swap(a, b):
    t = a.clone()
    a.copy_(b)
    b.copy_(t)


def _apply(psi, n, q, u):
    a, b = _sub(psi, n, {q: 0}), _sub(psi, n, {q: 1})
    u = [[complex(v) for v in row] for row in u]
    if u[0][1] == 0 and u[1][0] == 0:
        a.mul_(u[0][0])
        b.mul_(u[1][1])
        return
    t = a.clone()
    a.mul_(u[0][0]).add_(b, alpha=u[0][1])
    b.mul_(u[1][1]).add_(t, alpha=u[1][0])


def _matrix(name, p):
    if name == "h":
        return np.array([[1, 1], [1, -1]]) / math.sqrt(2.0)
    if name == "x":
        return np.array([[0, 1], [1, 0]])
    c, s = (math.cos(p[0] / 2), math.sin(p[0] / 2)) if p else (1.0, 0.0)
    if name == "rx":
        return np.array([[c, -1j * s], [-1j * s, c]])
    if name == "rz":
        return np.array([[complex(c, -s), 0], [0, complex(c, s)]])
    e = lambda v: complex(math.cos(v), math.sin(v))  # noqa: E731
    return np.array([[c, -e(p[2]) * s], [e(p[1]) * s, e(p[1] + p[2]) * c]])  # u3


def _simulate(n, gates, x):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[x] = 1.0
    pending = {}  # runs of one-qubit gates on a qubit, multiplied together

    def flush(qubits):
        for q in qubits:
            if q in pending:
                _apply(psi, n, q, pending.pop(q))

    for name, q0, q1, p, *more in gates:
        if q1 < 0:
            pending[q0] = _matrix(name, p) @ pending.get(q0, np.eye(2))
            continue
        flush([q0, q1, *more])
        if name == "cx":
            _swap(_sub(psi, n, {q0: 1, q1: 0}), _sub(psi, n, {q0: 1, q1: 1}))
        elif name == "swap":
            _swap(_sub(psi, n, {q0: 0, q1: 1}), _sub(psi, n, {q0: 1, q1: 0}))
        elif name == "ccx":
            _swap(_sub(psi, n, {q0: 1, q1: 1, more[0]: 0}), _sub(psi, n, {q0: 1, q1: 1, more[0]: 1}))
        else:
            _sub(psi, n, {q0: 1, q1: 1}).mul_(-1.0 if name == "cz" else complex(math.cos(p[0]), math.sin(p[0])))
    flush(list(pending))
    return psi


def _qft_of_basis(n, x):
    """The QFT circuit maps |x> to 2^(-n/2) sum_j exp(2 pi i x j / 2^n) |j>."""
    N = 1 << n
    out = torch.empty(N, dtype=torch.complex128, device="cuda")
    step = 1 << min(n, 26)
    for lo in range(0, N, step):
        j = torch.arange(lo, lo + step, dtype=torch.int64, device="cuda")
        angle = ((j * x) & (N - 1)).to(torch.float64).mul_(2.0 * math.pi / N)  # wraps mod 2^64: N divides it
        out[lo:lo + step] = torch.polar(torch.full_like(angle, 2.0 ** (-n / 2)), angle)
    return out


def exact(case, seed):
    path = case["path"]
    if path == "readout":
        first, idx = _readout_where(case, seed)
        x = _random_state(case, seed).to(torch.complex128)
        p = torch.view_as_real(x).square().sum(1)
        return {"norm": float(p.sum()), "probs": p[first:first + case["count"]],
                "amps": x[torch.from_numpy(idx.astype(np.int64)).cuda()]}
    if path == "serve":
        return [_simulate(n, gates, 0) for n, _, gates in _requests(case, seed)]
    n = case["n"]
    x = wl.random_basis_index(n, seed)
    if case["family"] == "qft":
        return _qft_of_basis(n, x)
    gates = _gates(case, n)
    if len(gates) * float(1 << n) > 1000 * 2.0 ** 30:  # about 20 s
        return None
    return _simulate(n, gates, x)
