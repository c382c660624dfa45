"""apply_gate with the matrix in the kernel arguments: matrices on both sides
of the 1 KiB line, several blocks, diagonals, low and high targets, many
different matrices queued back to back, and no place in a captured graph."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import haar_unitary, random_state  # noqa: E402

TOL = {torch.complex128: 1e-12, torch.complex64: 1e-5}


def _matrix(k, kind, rng):
    if kind == "dense":
        return haar_unitary(1 << k, rng)
    if kind == "diag":
        return np.diag(np.exp(1j * rng.uniform(0, 6, 1 << k)))
    m = np.eye(1 << k, dtype=np.complex128)   # controlled: a dense 2 x 2 block under k - 1 controls, and another
    m[-2:, -2:] = haar_unitary(2, rng)
    m[:2, :2] = haar_unitary(2, rng)
    return m


@pytest.mark.parametrize("dtype", sorted(TOL, key=str), ids=lambda d: str(d)[6:])
@pytest.mark.parametrize("n", [1, 2, 5, 7, 12, 17])
def test_gates_one_at_a_time(n, dtype):
    rng = np.random.default_rng([n, 7])
    psi = random_state(n, seed=n)
    sv = cast.StateVector(n, tensor=torch.tensor(psi, dtype=dtype, device="cuda"))
    for k in range(1, min(n, 6) + 1):
        for kind in ("dense", "diag", "controlled"):
            for qs in (range(k), range(n - k, n), rng.permutation(n)[:k]):
                qs = tuple(int(q) for q in qs)
                m = _matrix(k, kind, rng)
                sv.apply_gate(qs, m)
                psi = oracle.apply_gate(psi, qs, m)
    got = sv.tensor.cpu().numpy()
    assert np.abs(got - psi).max() <= TOL[dtype]


def test_refused_while_capturing():
    s = torch.cuda.Stream()
    t = torch.zeros(1 << 8, dtype=torch.complex64, device="cuda")
    t[0] = 1
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        sv = cast.StateVector(8, tensor=t)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        t.mul_(1)
        with pytest.raises(cast.CastError):
            sv.apply_gate((0,), np.array([[0, 1], [1, 0]]))
    torch.cuda.synchronize()
    assert t[0].item() == 1
