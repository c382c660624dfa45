"""apply_circuit's tile groups (several schedule passes per launch): dense 4-
and 5-qubit blocks on the matrix cores inside a tile, blocks selected by
qubits inside and outside it, identity blocks, phase tables rebuilt within a
tile, tiles of every size, against the oracle and the one-launch-per-pass
path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import Gate, dense_haar_layers, haar_unitary, hes, qft, qvc, random_state, rqc_u3_cx  # noqa: E402

TOL = {torch.complex128: 1e-12, torch.complex64: 1e-5}
DTYPES = [torch.complex128, torch.complex64]


def _selected(n, seed, count):
    """Gates of k qubits with dense blocks of d < k: the other k - d qubits
    select the block, some of which are the identity; diagonals between."""
    rng = np.random.default_rng([n, seed])
    gates = []
    for _ in range(count):
        k = int(rng.integers(2, 7))
        d = int(rng.integers(1, min(k, 5) + 1))
        qs = tuple(int(q) for q in rng.permutation(n)[:k])
        m = np.eye(1 << k, dtype=np.complex128)
        for b in range(1 << (k - d)):   # the selecting qubits are the high bits of the index
            if b and rng.integers(3) == 0:
                continue
            s = slice(b << d, (b + 1) << d)
            m[s, s] = haar_unitary(1 << d, rng)
        gates.append(Gate("unitary", qs, matrix=m))
        for _ in range(int(rng.integers(0, 3))):
            q2 = tuple(int(q) for q in rng.permutation(n)[:5])
            gates.append(Gate("unitary", q2, matrix=np.diag(np.exp(1j * rng.uniform(0, 6, 32)))))
    return gates


CASES = {
    "qft": (lambda n: qft(n), 5),
    "rqc5": (lambda n: rqc_u3_cx(n, 5, seed=2), 5),
    "rqc4": (lambda n: rqc_u3_cx(n, 5, seed=2), 4),
    "qvc": (lambda n: qvc(n, 4, seed=1), 5),
    "hes": (lambda n: hes(n, 2), 4),
    "dense": (lambda n: dense_haar_layers(n, 2, seed=1), 6),
    "selected": (lambda n: _selected(n, 3, 24), 6),
}


def _run(fc, psi0, n, dtype, groups):
    old = cast.get_tuning("tile_groups", dtype)
    try:
        cast.set_tuning("tile_groups", groups, dtype)
        sv = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=dtype, device="cuda"))
        sv.apply_circuit(fc)
        return sv.numpy()
    finally:
        cast.set_tuning("tile_groups", old, dtype)


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("n", [10, 11, 12, 13, 16, 17])
@pytest.mark.parametrize("case", list(CASES))
def test_groups_vs_oracle(case, n, dtype):
    make, k_max = CASES[case]
    if case == "dense" and n == 13:
        pytest.skip("no 5/6-qubit partition of 13")
    gates = make(n)
    fc = cast.FusedCircuit(n, gates, k_max=k_max)
    psi0 = random_state(n, seed=n, workload=15)
    print(f"tile groups {case} n={n} {dtype}: {fc.num_passes(dtype)} passes", flush=True)
    want = oracle.run_circuit(n, gates, psi0)
    got = _run(fc, psi0, n, dtype, 1)
    assert np.max(np.abs(got - want)) <= TOL[dtype]
    assert np.max(np.abs(_run(fc, psi0, n, dtype, 0) - want)) <= TOL[dtype]
    # the list's groups do not depend on the state they were planned with
    psi1 = random_state(n, seed=n + 1, workload=15)
    assert np.max(np.abs(_run(fc, psi1, n, dtype, 1) - oracle.run_circuit(n, gates, psi1))) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("bits", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("threads", [256, 1024])
def test_group_tile_sizes(dtype, bits, threads):
    n = 15
    old = {k: cast.get_tuning(k, dtype) for k in ("blocked_tile_bits", "blocked_threads")}
    psi0 = random_state(n, seed=bits, workload=16)
    try:
        cast.set_tuning("blocked_tile_bits", bits, dtype)
        cast.set_tuning("blocked_threads", threads, dtype)
        for case in ("qft", "rqc4", "selected"):
            make, k_max = CASES[case]
            gates = make(n)
            print(f"tile bits {bits} threads {threads} {case} {dtype}", flush=True)
            got = _run(cast.FusedCircuit(n, gates, k_max=k_max), psi0, n, dtype, 1)
            assert np.max(np.abs(got - oracle.run_circuit(n, gates, psi0))) <= TOL[dtype]
    finally:
        for k, v in old.items():
            cast.set_tuning(k, v, dtype)
