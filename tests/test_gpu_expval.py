"""Expectation values of many Pauli strings in few passes: tile sizes of every
state size class, x masks inside one tile, over several tiles and too wide for
any tile, both parities of |x & z|, and more strings than one launch holds,
against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import PauliTerm, random_state, vqa_hamiltonian  # noqa: E402


def _string(rng, n, weight):
    return tuple((int(q), "XYZ"[rng.integers(3)]) for q in rng.permutation(n)[:weight])


def _terms(n, kind):
    rng = np.random.default_rng([n, 5])
    if kind == "ring":      # one x mask per qubit, all diagonal terms together
        return vqa_hamiltonian(n)
    if kind == "wide":      # masks that flip more qubits than a tile holds above its window
        ops = [tuple((q, "XY"[(q + s) % 2]) for q in range(n)) for s in range(2)]
        return [PauliTerm(0.7 - s, o) for s, o in enumerate(ops)] + [PauliTerm(0.3, _string(rng, n, n))]
    return [PauliTerm(float(rng.normal()), _string(rng, n, int(rng.integers(1, min(n, 6) + 1)))) for _ in range(200)]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 11, 16, 17, 18, 19, 20, 21])
@pytest.mark.parametrize("kind", ["ring", "wide", "many"])
def test_expval_passes(dtype, n, kind):
    if kind == "ring" and n < 3:
        pytest.skip("no ring")
    terms = _terms(n, kind)
    psi = random_state(n, seed=n, workload=12).astype(np.complex64 if dtype == torch.complex64 else np.complex128)
    print(f"expval n={n} {kind} terms={len(terms)} {dtype}", flush=True)
    sv = cast.StateVector(n, tensor=torch.tensor(psi, device="cuda"))
    got = sv.expval(terms)
    # the oracle sees the same (rounded) amplitudes; products and sums are
    # FP64 on both sides: n 2^-53 per term leaves 1e-13 per unit of coefficient
    want = oracle.expval(psi.astype(np.complex128), terms)
    assert got.imag == 0.0
    assert abs(got.real - want.real) <= 1e-13 * sum(abs(t.coeff) for t in terms)
