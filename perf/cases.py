"""Performance cases of the state-vector engine: what its users run, through the
public entry points, from a 12-qubit state (launch latency) to a 16 GiB one.

Kinds of case
  gates    one brick layer of U3 and CX gates applied gate by gate (apply_gate)
  circuit  a fused gate list, one device pass per fused gate or diagonal run
  blocked  a fused gate list, several fused gates per device pass
  expval   a Pauli-sum expectation value of a state
  adjoint  energy and gradient of one parametrised circuit
  vqa      energies and gradients of many parameter sets of one circuit
  tfim     energies and gradients of Trotter circuits of different sizes
"""
import math

import numpy as np
import torch

import paper_2503_19894_amd as cast
from circuits import (PauliTerm, ala, dense_haar_layers, hea_vqa, hes, iqp, qft, qvc, rqc_u3_cx, tfim_trotter,
                      vqa_hamiltonian)

DEV = "cuda"
DTYPES = {"c64": torch.complex64, "c128": torch.complex128}
MODES = {"steps": cast.BATCH_STEPS, "graph": cast.BATCH_STEPS_GRAPH, "persistent": cast.BATCH_PERSISTENT_GRAPH}


def listed():
    return [
        # an interactive program that applies its gates one at a time
        {"name": "gates_n12_c128", "kind": "gates", "n": 12, "dtype": "c128"},
        # a random circuit on a small state: launches and latency
        {"name": "rqc_n12_c64", "kind": "circuit", "family": "rqc", "size": 10, "n": 12, "dtype": "c64", "k_max": 5},
        # the same circuit family at an ordinary odd size (cache resident)
        {"name": "rqc_n21_c128", "kind": "circuit", "family": "rqc", "size": 10, "n": 21, "dtype": "c128", "k_max": 5},
        # the headline workload: a fused QFT on 16 GiB of state
        {"name": "qft_n30_c128", "kind": "circuit", "family": "qft", "size": 0, "n": 30, "dtype": "c128", "k_max": 5},
        # dense 5- and 6-qubit unitaries (matrix cores)
        {"name": "dense_n28_c128", "kind": "circuit", "family": "dense", "size": 2, "n": 28, "dtype": "c128",
         "k_max": 6},
        # cache-blocked execution with the planner's usual choices of k_max
        {"name": "qft_n27_c64_blocked", "kind": "blocked", "family": "qft", "size": 0, "n": 27, "dtype": "c64",
         "k_max": 4},
        {"name": "hes_n28_c128_blocked", "kind": "blocked", "family": "hes", "size": 5, "n": 28, "dtype": "c128",
         "k_max": 3},
        # the energy of a variational state, small and large
        {"name": "expval_n15_c64", "kind": "expval", "n": 15, "dtype": "c64", "ham": "vqa"},
        {"name": "expval_n26_c128", "kind": "expval", "n": 26, "dtype": "c128", "ham": "vqa"},
        # one optimiser step of one variational circuit
        {"name": "adjoint_n17_c128", "kind": "adjoint", "n": 17, "dtype": "c128", "layers": 4},
        # many parameter sets of the 20-qubit, 8-layer ansatz at once
        {"name": "vqa_n20_c128", "kind": "vqa", "n": 20, "dtype": "c128", "layers": 8, "sets": 64, "mode": "graph"},
        # field gradients of Trotter circuits on rings of different sizes
        {"name": "tfim_n19_c64", "kind": "tfim", "n": 19, "dtype": "c64", "steps": 20, "mode": "persistent"},
    ]


def draw(rng):
    """One more case of the same ranges: qubit counts uniform (the work doubles
    with each), families, options and types as listed."""
    kind = rng.choice(("gates", "circuit", "circuit", "circuit", "blocked", "blocked", "expval", "adjoint", "vqa",
                       "tfim"))
    c = {"kind": kind, "dtype": rng.choice(("c64", "c128"))}
    if kind == "gates":
        c["n"] = rng.randint(8, 22)
    elif kind == "circuit":
        c["family"] = rng.choice(("qft", "rqc", "iqp", "ala", "qvc", "dense"))
        c["n"] = rng.randint(10, 28)
        if c["family"] == "dense":
            c["n"] = rng.choice([n for n in range(15, 29) if any((n - 6 * a) % 5 == 0 for a in range(n // 6 + 1))])
        c["size"] = rng.randint(2, 3) if c["family"] == "dense" else rng.randint(4, 10)
        c["k_max"] = 6 if c["family"] == "dense" else rng.randint(4, 6)
    elif kind == "blocked":
        c.update(family=rng.choice(("qft", "hes", "iqp", "rqc")), size=rng.randint(3, 8), n=rng.randint(16, 28),
                 k_max=rng.randint(3, 5))
    elif kind == "expval":
        c.update(n=rng.randint(10, 28), ham=rng.choice(("vqa", "strings")))
    elif kind == "adjoint":
        c.update(n=rng.randint(8, 21), layers=rng.randint(2, 6))
    elif kind == "vqa":
        c["n"] = rng.randint(10, 20)
        c["layers"] = rng.randint(2, 8)
        c["sets"] = int(round(2.0 ** rng.uniform(1, 6 + min(2, 20 - c["n"]))))
        c["mode"] = rng.choice(("graph", "persistent"))
    else:
        c.update(n=rng.randint(13, 21), steps=rng.randint(8, 24), mode=rng.choice(("graph", "persistent")))
    return c


# ------------------------------------------------------------------ inputs
def _random_state(n, seed, dtype):
    """i.i.d. complex Gaussian amplitudes, normalised."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = torch.empty(1 << n, dtype=dtype, device=DEV)
    sq = 0.0
    for part in torch.view_as_real(out).split(1 << 26):
        part.normal_(generator=g)
        sq = sq + part.double().square().sum()
    torch.view_as_real(out).mul_(1.0 / math.sqrt(float(sq)))
    return out


def _product_state(n, seed, dtype):
    """A product of random one-qubit states plus some noise: an energy of order n, as a variational state has."""
    rng = np.random.default_rng([7, seed])
    out = torch.ones(1, dtype=torch.complex128, device=DEV)
    for th, ph in zip(rng.uniform(0, math.pi, n), rng.uniform(0, 2 * math.pi, n)):
        one = torch.tensor([math.cos(th / 2), math.sin(th / 2) * np.exp(1j * ph)], dtype=torch.complex128, device=DEV)
        out = torch.outer(one, out).reshape(-1)   # the new qubit is the highest bit
    out += 0.1 * _random_state(n, seed, torch.complex128)
    return (out / torch.linalg.vector_norm(out)).to(dtype)


def _gates(case, seed):
    n, fam = case["n"], case.get("family")
    if case["kind"] == "gates":
        return rqc_u3_cx(n, layers=1, seed=seed)
    if fam == "qft":
        return qft(n)
    if fam == "rqc":
        return rqc_u3_cx(n, layers=case["size"], seed=seed)
    if fam == "iqp":
        return iqp(n, seed=seed)
    if fam == "ala":
        return ala(n, layers=case["size"], seed=seed)
    if fam == "qvc":
        return qvc(n, depth=case["size"], seed=seed)
    if fam == "hes":
        return hes(n, steps=case["size"], seed=seed)
    return dense_haar_layers(n, depth=case["size"], seed=seed)


def _hamiltonian(case, seed):
    if case.get("ham", "vqa") == "vqa":
        return vqa_hamiltonian(case["n"])
    # Pauli strings of weight 1 to 4, some of which flip the same qubits
    rng = np.random.default_rng([8, seed])
    flips = [rng.choice(case["n"], rng.integers(0, 4), replace=False) for _ in range(10)]
    terms = []
    for _ in range(30):
        fl = flips[rng.integers(len(flips))]
        ops = {int(q): "XY"[rng.integers(2)] for q in fl}
        q = int(rng.integers(case["n"]))
        ops.setdefault(q, "Z")
        terms.append(PauliTerm(float(rng.normal()), tuple(sorted(ops.items()))))
    return terms


def _tfim_sizes(case):
    return [case["n"] - 9, case["n"] - 6, case["n"] - 3, case["n"]]


def _thetas(case, seed):
    rng = np.random.default_rng([9, seed])
    if case["kind"] == "tfim":
        return [rng.uniform(0.5, 1.5, n) for n in _tfim_sizes(case)]
    p = 2 * case["n"] * case["layers"]
    return list(rng.uniform(-math.pi, math.pi, (case.get("sets", 1), p)))


def prepare(case, seed):
    n, dtype, kind = case["n"], DTYPES[case["dtype"]], case["kind"]
    s = {"kind": kind}
    if kind == "gates":
        s["sv"] = cast.StateVector(n, tensor=_random_state(n, seed, dtype))
        s["gates"] = [(g.qubits, cast.std_matrix(g.name, g.params).view(np.complex128)[..., 0])
                      for g in _gates(case, seed)]
    elif kind in ("circuit", "blocked"):
        s["sv"] = cast.StateVector(n, tensor=_random_state(n, seed, dtype))
        s["fused"] = cast.FusedCircuit(n, _gates(case, seed), k_max=case["k_max"])
    elif kind == "expval":
        s["sv"] = cast.StateVector(n, tensor=_product_state(n, seed, dtype))
        s["ham"] = _hamiltonian(case, seed)
    elif kind == "adjoint":
        s["init"] = cast.StateVector(n, dtype=dtype)
        s["gates"] = hea_vqa(n, case["layers"])[0]
        s["theta"], s["ham"] = _thetas(case, seed)[0], _hamiltonian(case, seed)
    elif kind == "vqa":
        g, p = hea_vqa(n, case["layers"])
        b = case["sets"]
        s["thetas"] = _thetas(case, seed)
        s["batch"] = cast.Batch([g] * b, [n] * b, [p] * b, [vqa_hamiltonian(n)] * b, dtype=dtype,
                                mode=MODES[case["mode"]])
    else:
        ns = _tfim_sizes(case)
        s["thetas"] = _thetas(case, seed)
        s["batch"] = cast.Batch([tfim_trotter(m, case["steps"]) for m in ns], ns, ns,
                                [[PauliTerm(1.0, ((0, "Z"),))] for m in ns], dtype=dtype, init=["plus"] * len(ns),
                                mode=MODES[case["mode"]])
    return s


def run(s):
    kind = s["kind"]
    if kind == "gates":
        for qubits, matrix in s["gates"]:
            s["sv"].apply_gate(qubits, matrix)
        return s["sv"].tensor
    if kind == "circuit":
        s["sv"].apply_circuit(s["fused"])
        return s["sv"].tensor
    if kind == "blocked":
        s["sv"].apply_circuit_blocked(s["fused"])
        return s["sv"].tensor
    if kind == "expval":
        return np.float64(s["sv"].expval(s["ham"]).real)
    if kind == "adjoint":
        energy, grad = cast.adjoint(s["init"], s["gates"], s["theta"], s["ham"])
        return {"energy": np.float64(energy), "grad": grad}
    energies, grads = s["batch"].run(s["thetas"])
    return {"energies": energies, "grads": np.concatenate(grads)}


# ------------------------------------------------------------------ work
_FLOPS = {"h": 4, "u3": 14, "ry": 6, "rx": 6, "rz": 6, "cp": 1.5, "rxx": 6, "cx": 0, "cz": 0, "swap": 0}


def _gate_flops(g):
    """Flops per amplitude."""
    return 8 * (1 << len(g.qubits)) - 2 if g.name == "unitary" else _FLOPS[g.name]


def work(case):
    """States read and written once; each gate's multiplications and additions on every amplitude (three times
    where there is a gradient: psi forward, psi and lambda backward, and the inner product)."""
    amp = 16 if case["dtype"] == "c128" else 8
    kind = case["kind"]
    if kind in ("gates", "circuit", "blocked"):
        N = 1 << case["n"]
        return {"bytes": 2 * amp * N, "flops": N * sum(_gate_flops(g) for g in _gates(case, 0))}
    if kind == "expval":
        N = 1 << case["n"]
        return {"bytes": amp * N, "flops": N * (3 + len(_hamiltonian(case, 0)))}
    if kind == "tfim":
        insts = [(m, tfim_trotter(m, case["steps"])) for m in _tfim_sizes(case)]
    else:
        insts = [(case["n"], hea_vqa(case["n"], case["layers"])[0])] * case.get("sets", 1)
    per = {}
    for m, g in insts:
        if m not in per:
            per[m] = sum(3 * _gate_flops(x) + (4 if x.param >= 0 else 0) for x in g)
    return {"bytes": sum(2 * amp << m for m, _ in insts), "flops": sum(per[m] * (1 << m) for m, _ in insts)}


# ------------------------------------------------------------------ exact
def _u3(th, ph, la):
    c, s = math.cos(th / 2), math.sin(th / 2)
    return np.array([[c, -np.exp(1j * la) * s], [np.exp(1j * ph) * s, np.exp(1j * (ph + la)) * c]])


def _matrix(g):
    """Matrix of a fixed gate, bit i of the index belonging to qubits[i]."""
    if g.name == "unitary":
        return np.asarray(g.matrix)
    if g.name == "u3":
        return _u3(*g.params)
    if g.name == "h":
        return np.array([[1, 1], [1, -1]]) / math.sqrt(2)
    if g.name == "cx":
        return np.eye(4)[[0, 3, 2, 1]]
    if g.name == "cz":
        return np.diag([1.0, 1, 1, -1])
    if g.name == "swap":
        return np.eye(4)[[0, 2, 1, 3]]
    a = g.params[0]
    if g.name == "cp":
        return np.diag([1, 1, 1, np.exp(1j * a)])
    if g.name == "rz":
        return np.diag([np.exp(-0.5j * a), np.exp(0.5j * a)])
    c, s = math.cos(a / 2), math.sin(a / 2)
    if g.name == "ry":
        return np.array([[c, -s], [s, c]])
    if g.name == "rxx":
        return c * np.eye(4) - 1j * s * np.fliplr(np.eye(4))
    raise ValueError(g.name)


def _apply(psi, n, qubits, m):
    """psi (2^n amplitudes) with the matrix m applied: a sum over its nonzero entries."""
    hi = sorted(qubits, reverse=True)
    shape, last = [], n
    for q in hi:
        shape += [1 << (last - 1 - q), 2]
        last = q
    x = psi.reshape(shape + [1 << last])
    k = len(qubits)

    def plane(j):
        ix = [slice(None)] * x.dim()
        for i, q in enumerate(qubits):
            ix[2 * hi.index(q) + 1] = (j >> i) & 1
        return tuple(ix)

    if k > 2:   # dense: one product
        rows = torch.stack([x[plane(j)].reshape(-1) for j in range(1 << k)])
        rows = torch.tensor(m, dtype=torch.complex128, device=psi.device) @ rows
        for j in range(1 << k):
            x[plane(j)] = rows[j].reshape(x[plane(j)].shape)
        return psi
    old = [x[plane(j)].clone() for j in range(1 << k)]
    for r in range(1 << k):
        if m[r][r] == 1 and np.count_nonzero(m[r]) == 1:
            continue
        acc = None
        for c in range(1 << k):
            if m[r][c] != 0:
                t = old[c] * complex(m[r][c])
                acc = t if acc is None else acc.add_(t)
        x[plane(r)] = acc
    return psi


_PAULI = {"rx": "X", "ry": "Y", "rz": "Z", "rxx": "XX", "ryy": "YY", "rzz": "ZZ"}


def _pauli(psi, n, ops):
    """A Pauli string on psi of shape [sets, 2^n]."""
    out = psi
    for q, p in ops:
        x = out.reshape(psi.shape[0], 1 << (n - 1 - q), 2, 1 << q)
        if p == "Z":
            out = torch.stack([x[:, :, 0], -x[:, :, 1]], 2)
        elif p == "X":
            out = torch.stack([x[:, :, 1], x[:, :, 0]], 2)
        else:
            out = torch.stack([-1j * x[:, :, 1], 1j * x[:, :, 0]], 2)
        out = out.reshape(psi.shape)
    return out


def _rotate(psi, n, g, angles):
    """exp(-i angle P / 2) on every set."""
    a = torch.as_tensor(angles, dtype=torch.float64, device=psi.device).reshape(-1, 1) / 2
    p = _pauli(psi, n, tuple(zip(g.qubits, _PAULI[g.name])))
    return torch.cos(a) * psi - 1j * torch.sin(a) * p


def _energy_grad(n, gates, thetas, terms, plus):
    """Energies [sets] and gradients [sets, parameters] by the adjoint method."""
    th = np.asarray(thetas)
    psi = torch.zeros((len(th), 1 << n), dtype=torch.complex128, device=DEV)
    if plus:
        psi.fill_(2.0 ** (-n / 2))
    else:
        psi[:, 0] = 1

    def go(v, g, sign):
        if g.param >= 0:
            return _rotate(v, n, g, sign * g.coeff * th[:, g.param])
        if g.params:
            return _rotate(v, n, g, np.full(len(th), sign * g.params[0]))
        x = v.reshape(len(th), -1, 2, 1 << max(g.qubits) - min(g.qubits) - 1, 2, 1 << min(g.qubits))   # cz
        x[:, :, 1, :, 1] *= -1
        return v

    for g in gates:
        psi = go(psi, g, 1.0)
    lam = sum(t.coeff * _pauli(psi, n, t.ops) for t in terms)
    energy = (psi.conj() * lam).sum(1).real
    grad = torch.zeros(th.shape, dtype=torch.float64, device=DEV)
    for g in reversed(gates):
        if g.param >= 0:
            inner = (lam.conj() * _pauli(psi, n, tuple(zip(g.qubits, _PAULI[g.name])))).sum(1).imag
            grad[:, g.param] += g.coeff * inner
        psi, lam = go(psi, g, -1.0), go(lam, g, -1.0)
    return energy.cpu().numpy(), grad.cpu().numpy()


def exact(case, seed):
    n, kind, dtype = case["n"], case["kind"], DTYPES[case["dtype"]]
    if kind in ("gates", "circuit", "blocked"):
        psi = _random_state(n, seed, dtype).to(torch.complex128)
        if case.get("family") == "qft":
            return torch.fft.ifft(psi, norm="ortho")
        for g in _gates(case, seed):
            psi = _apply(psi, n, g.qubits, _matrix(g))
        return psi
    if kind == "expval":
        psi = _product_state(n, seed, dtype).to(torch.complex128).reshape(1, -1)
        return np.float64(sum(t.coeff * float((psi.conj() * _pauli(psi, n, t.ops)).sum().real)
                              for t in _hamiltonian(case, seed)))
    if kind == "adjoint":
        e, g = _energy_grad(n, hea_vqa(n, case["layers"])[0], _thetas(case, seed), _hamiltonian(case, seed), False)
        return {"energy": e[0], "grad": g[0]}
    if kind == "vqa":
        e, g = _energy_grad(n, hea_vqa(n, case["layers"])[0], _thetas(case, seed), vqa_hamiltonian(n), False)
        return {"energies": e, "grads": g.reshape(-1)}
    es, gs = [], []
    for m, th in zip(_tfim_sizes(case), _thetas(case, seed)):
        e, g = _energy_grad(m, tfim_trotter(m, case["steps"]), [th], [PauliTerm(1.0, ((0, "Z"),))], True)
        es.append(e[0])
        gs.append(g[0])
    return {"energies": np.array(es), "grads": np.concatenate(gs)}
