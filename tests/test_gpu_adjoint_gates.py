"""adjoint_grad one gate at a time (complex64, and gates of three and more
qubits): both states in one launch, inner products finished in sets, on the
smallest states and on ones whose sets fill the scratch several times, against
the oracle's adjoint."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import Gate, PauliTerm, haar_unitary, random_state  # noqa: E402

# a gate rounds the state to the type's precision (relative, in norm), forward
# and backward for both states; four times that
EPS = {torch.complex64: 2.0**-24, torch.complex128: 2.0**-53}


@pytest.mark.parametrize("n,length,dtype", [(1, 12, torch.complex64), (2, 20, torch.complex64),
                                            (5, 40, torch.complex64), (11, 60, torch.complex64),
                                            (17, 90, torch.complex64), (20, 40, torch.complex64),
                                            (2, 20, torch.complex128), (7, 30, torch.complex128)])
def test_adjoint_gates_vs_oracle(n, length, dtype):
    rng = np.random.default_rng([n, 5])
    gates, P = [], 0
    for i in range(length):
        qs = tuple(int(q) for q in rng.permutation(n))
        r = int(rng.integers(5))
        if r == 0:
            k = int(rng.integers(1, min(n, 4) + 1))
            gates.append(Gate("unitary", qs[:k], matrix=haar_unitary(1 << k, rng)))
        elif r == 1 and n > 1:
            gates.append(Gate(("cx", "cz", "swap")[i % 3], qs[:2]))
        elif r == 2 and n > 1:
            gates.append(Gate(("rxx", "ryy", "rzz")[i % 3], qs[:2], param=P, coeff=float(rng.uniform(-2, 2))))
            P += 1
        else:
            gates.append(Gate(("rx", "ry", "rz")[i % 3], qs[:1], param=P, coeff=float(rng.uniform(-2, 2))))
            P += 1
    if dtype == torch.complex128 and n > 2:
        gates.insert(3, Gate("unitary", (0, 2, 1), matrix=haar_unitary(8, rng)))
    theta = rng.uniform(-4, 4, P)
    psi0 = random_state(n, seed=n, workload=13)
    H = [PauliTerm(float(rng.normal()), tuple((int(q), "XYZ"[rng.integers(3)])
                                              for q in rng.permutation(n)[:rng.integers(1, min(n, 3) + 1)]))
         for _ in range(6)]
    init = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=dtype, device="cuda"))
    e, g = cast.adjoint(init, gates, theta, H)
    we, wg = oracle.adjoint_grad(n, gates, theta, H, psi0.copy())
    scale = sum(abs(t.coeff) for t in H) * 2   # gradients: |coeff| <= 2
    tol = 4 * EPS[dtype] * 4 * (len(gates) + 2) * scale
    print(f"n={n} gates={len(gates)} params={P} de={abs(e - we):.1e} dg={np.abs(g - wg).max():.1e} tol={tol:.1e}", flush=True)
    assert abs(e - we) <= tol
    assert np.abs(g - wg).max() <= tol
