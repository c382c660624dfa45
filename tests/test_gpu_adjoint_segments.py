"""adjoint_grad as segments (complex128, one- and two-qubit gates): every
rotation generator on one and two qubits, both ends of the tile sizes, fixed
gates of each matrix form, equal rotations that meet, a non-zero initial
state, and the general path's circuits, against the oracle's adjoint."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import Gate, PauliTerm, haar_unitary, random_state  # noqa: E402


def _circuit(n, seed, length):
    """Rotations (some repeated at once, some with a shared parameter) between
    fixed gates of every form the segments tell apart."""
    rng = np.random.default_rng([n, seed])
    gates, p = [], 0
    fixed1 = ("h", "x", "y", "z", "s", "t", "u3", "p", "rx", "ry", "rz", "haar")
    fixed2 = ("cx", "cz", "cp", "swap", "rxx", "ryy", "rzz", "haar", "diag", "phase_rxx")
    for _ in range(length):
        a, b = (int(q) for q in rng.permutation(n)[:2])
        ang = tuple(float(v) for v in rng.uniform(-7, 7, 3))
        r = rng.integers(4)
        if r == 0:
            name = fixed1[rng.integers(len(fixed1))]
            m = haar_unitary(2, rng) if name == "haar" else None
            gates.append(Gate("unitary", (a,), matrix=m) if m is not None else
                         Gate(name, (a,), ang[:{"u3": 3, "p": 1, "rx": 1, "ry": 1, "rz": 1}.get(name, 0)]))
        elif r == 1:
            name = fixed2[rng.integers(len(fixed2))]
            if name == "haar":
                gates.append(Gate("unitary", (a, b), matrix=haar_unitary(4, rng)))
            elif name == "diag":
                gates.append(Gate("unitary", (a, b), matrix=np.diag(np.exp(1j * rng.uniform(0, 6, 4)))))
            elif name == "phase_rxx":   # e^{i c} RXX: a Pauli pair that is no rotation
                x = np.fliplr(np.eye(4))
                gates.append(Gate("unitary", (a, b), matrix=np.exp(0.4j) * (0.6 * np.eye(4) - 0.8j * x)))
            else:
                gates.append(Gate(name, (a, b), ang[:1] if name in ("cp", "rxx", "ryy", "rzz") else ()))
        elif r == 2:
            name = ("rx", "ry", "rz")[rng.integers(3)]
            for _ in range(int(rng.integers(1, 3))):
                gates.append(Gate(name, (a,), param=p, coeff=float(rng.uniform(-2, 2))))
                p += int(rng.integers(2))
        else:
            name = ("rxx", "ryy", "rzz")[rng.integers(3)]
            for _ in range(int(rng.integers(1, 3))):
                gates.append(Gate(name, (a, b), param=p, coeff=float(rng.uniform(-2, 2))))
                p += int(rng.integers(2))
    return gates, p + 1


@pytest.mark.parametrize("n,length", [(3, 40), (4, 150), (9, 150), (10, 80), (11, 60), (13, 60), (17, 25)])
def test_adjoint_segments_vs_oracle(n, length):
    gates, P = _circuit(n, 1, length)
    rng = np.random.default_rng([n, 2])
    theta = rng.uniform(-9, 9, P)
    psi0 = random_state(n, seed=n, workload=13)
    H = [PauliTerm(float(rng.normal()), tuple((int(q), "XYZ"[rng.integers(3)])
                                              for q in rng.permutation(n)[:rng.integers(1, min(n, 4) + 1)]))
         for _ in range(9)]
    print(f"adjoint segments n={n} gates={len(gates)} params={P}", flush=True)
    init = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=torch.complex128, device="cuda"))
    e, g = cast.adjoint(init, gates, theta, H)
    ew, gw = oracle.adjoint_grad(n, gates, theta, H, psi0)
    # each gate rounds psi and lambda by a few 2^-53; coefficients are at most 2
    tol = 1e-15 * len(gates) * 10 * sum(abs(t.coeff) for t in H)
    assert abs(e - ew) <= tol and np.max(np.abs(g - gw)) <= tol
    # the initial state is copied, not modified
    assert np.array_equal(init.numpy(), psi0)


@pytest.mark.parametrize("gen", range(1, 16))
def test_every_generator(gen):
    """exp(-i c theta G / 2) for each Pauli string G on two qubits (raw
    generator codes, X / Y / Z with or without identity) and both orders."""
    n = 5
    letters = [(gen >> (2 * i)) & 3 for i in range(2)]
    P = {0: np.eye(2), 1: np.array([[0, 1], [1, 0]]), 2: np.array([[0, -1j], [1j, 0]]), 3: np.diag([1.0, -1])}
    psi0 = random_state(n, seed=gen, workload=14)
    H = [PauliTerm(1.0, ((0, "X"), (3, "Y"))), PauliTerm(0.5, ((1, "Z"), (4, "Z"))), PauliTerm(-0.7, ((3, "Z"),))]
    init = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=torch.complex128, device="cuda"))
    for qubits in ((1, 3), (4, 0)):
        ga = cast.GateArray([Gate("rxx", qubits, param=0, coeff=1.3), Gate("cx", (qubits[1], 2)),
                             Gate("rxx", qubits, param=1, coeff=-0.6)])
        for i in (0, 2):
            ga.arr[i].generator = gen
        theta = np.array([0.9, -2.1])
        import ctypes
        e, g = ctypes.c_double(), np.zeros(2)
        cast.adjoint_grad(init.handle, ga.arr, 3, cast._dptr(theta), 2, cast.pauli_terms(H), 3, ctypes.byref(e),
                          cast._dptr(g))
        full = np.kron(P[letters[1]], P[letters[0]])   # bit i of the index <-> qubits[i]

        def energy(th):
            us = [np.cos(c * t / 2) * np.eye(4) - 1j * np.sin(c * t / 2) * full for c, t in ((1.3, th[0]), (-0.6, th[1]))]
            psi = psi0
            for u, q in ((us[0], qubits), (None, None), (us[1], qubits)):
                if u is None:
                    psi = oracle.run_circuit(n, [Gate("cx", (qubits[1], 2))], psi)
                else:
                    psi = oracle.run_circuit(n, [Gate("unitary", q, matrix=u)], psi)
            return oracle.expval(psi, H).real

        assert abs(e.value - energy(theta)) <= 1e-13
        for i, c in enumerate((1.3, -0.6)):   # parameter shift: exact for these generators
            d = np.zeros(2)
            d[i] = np.pi / 2 / c
            assert abs(g[i] - c * (energy(theta + d) - energy(theta - d)) / 2) <= 1e-13
