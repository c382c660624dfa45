"""Expectation values of strings that share one x mask (a single string among
them): flips within a wave's amplitudes, within a tile, across the state and
none, both parities, more strings than a launch holds and more partial sums than
the scratch, the allocation-free entry point, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import PauliTerm, random_state  # noqa: E402

DTYPES = [torch.complex128, torch.complex64]


def _check(n, terms, dtype, seed=0):
    psi = random_state(n, seed=seed, workload=24).astype(np.complex64 if dtype == torch.complex64 else np.complex128)
    sv = cast.StateVector(n, tensor=torch.tensor(psi, device="cuda"))
    want = oracle.expval(psi.astype(np.complex128), terms)
    # as for many strings: FP64 products and sums on the same rounded amplitudes
    tol = 1e-13 * sum(abs(t.coeff) for t in terms)
    for got in (sv.expval(terms), sv.expval_noalloc(terms[:4096])):
        assert got.imag == 0.0
        assert abs(got.real - want.real) <= tol


def _strings(n, x, count, rng):
    """`count` strings that flip the qubits of x, their other letters at random."""
    out = []
    for _ in range(count):
        ops = [(q, "XY"[rng.integers(2)]) if (x >> q) & 1 else (q, "IZ"[rng.integers(2)]) for q in range(n)]
        out.append(PauliTerm(float(rng.normal()), tuple((q, p) for q, p in ops if p != "I")))
    return out


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("n", [1, 2, 5, 6, 7, 10, 17, 21])
def test_single_string(dtype, n):
    rng = np.random.default_rng(n)
    full = (1 << n) - 1
    for x in sorted({0, 1, 2 & full, 32 & full, 63 & full, 64 & full, 0x60 & full, 1 << (n - 1), full ^ 1, full}):
        print(f"one string n={n} x={x:#x} {dtype}", flush=True)
        _check(n, _strings(n, x, 1, rng), dtype, seed=n)


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("n,count", [(13, 2), (13, 16), (13, 17), (16, 40), (20, 5), (20, 150)])
def test_one_wide_flip(dtype, n, count):
    """Up to ten launches of 512 partial sums (150 strings on 20 qubits)."""
    print(f"{count} strings n={n} {dtype}", flush=True)
    _check(n, _strings(n, (1 << n) - 1, count, np.random.default_rng([n, count])), dtype)


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
def test_partial_sums_fold(dtype):
    """2^22 amplitudes leave 2048 partial sums a launch, the scratch holds eight
    launches' and a ninth finds them folded into one."""
    n, count = 22, 9 * 16
    terms = _strings(n, (1 << n) - 1, count, np.random.default_rng(3))
    g = torch.Generator(device="cuda").manual_seed(5)
    psi = torch.randn(1 << n, dtype=dtype, device="cuda", generator=g)
    psi /= torch.linalg.vector_norm(psi)
    print(f"{count} strings n={n} {dtype}", flush=True)
    sv = cast.StateVector(n, tensor=psi)
    # one at a time the strings need no fold
    want = sum(sv.expval([t]).real for t in terms)
    assert abs(sv.expval(terms).real - want) <= 1e-13 * sum(abs(t.coeff) for t in terms)
