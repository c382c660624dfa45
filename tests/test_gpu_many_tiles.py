"""Kernels whose workgroups take several tiles (the next tile's loads in flight
while one is worked on, tables rebuilt for each, sums carried over): tile groups
with more whole-size tiles than workgroups, of every tile size up to the dtype's
largest, against the oracle, and expectation values of states large enough that
each workgroup takes two and four tiles, against FP64 torch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import PauliTerm, random_state, random_state_torch, vqa_hamiltonian  # noqa: E402
from tests.test_gpu_tile_groups import CASES, TOL  # noqa: E402

DTYPES = [torch.complex128, torch.complex64]
WORKGROUPS = 512   # of a pass, at most: two on each of 256 compute units
LARGEST = {torch.complex128: 12, torch.complex64: 13}


def _apply(fc, psi0, n, dtype):
    sv = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=dtype, device="cuda"))
    sv.apply_circuit(fc)
    return sv.numpy()


def _tiles(fc, n, dtype):
    """(tile bits, tiles, gates) of the launches that are tile groups."""
    groups = [x for x in fc.launches(dtype) if x["tile_bits"]]
    assert groups and len(fc.launches(dtype)) < fc.num_passes(dtype)
    return [(x["tile_bits"], 1 << (n - x["tile_bits"]), x["count"]) for x in groups]


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("case", ["qft", "rqc5", "selected"])
def test_largest_tiles(case, dtype):
    n = 22 if dtype == torch.complex128 else 23
    make, k_max = CASES[case]
    gates = make(n)
    psi0 = random_state(n, seed=n, workload=21)
    fc = cast.FusedCircuit(n, gates, k_max=k_max)
    tiles = _tiles(fc, n, dtype)
    print(f"largest tiles {case} n={n} {dtype}: {tiles}", flush=True)
    assert max(tiles)[0] == LARGEST[dtype] and max(t for _, t, _ in tiles) > WORKGROUPS
    assert np.max(np.abs(_apply(fc, psi0, n, dtype) - oracle.run_circuit(n, gates, psi0))) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("bits", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("case", ["qft", "rqc4", "selected"])
def test_tile_sizes(case, dtype, bits):
    """Tiles of at most 2^bits amplitudes, on the smallest state that has more
    of them than there are workgroups."""
    n = bits + 10
    make, k_max = CASES[case]
    gates = make(n)
    psi0 = random_state(n, seed=bits, workload=22)
    old = cast.get_tuning("blocked_tile_bits", dtype)
    try:
        cast.set_tuning("blocked_tile_bits", bits, dtype)
        fc = cast.FusedCircuit(n, gates, k_max=k_max)
        tiles = _tiles(fc, n, dtype)
        print(f"tile bits {bits} {case} n={n} {dtype}: {tiles}", flush=True)
        assert max(tiles)[0] <= bits and max(t for _, t, _ in tiles) > WORKGROUPS
        got = _apply(fc, psi0, n, dtype)
    finally:
        cast.set_tuning("blocked_tile_bits", old, dtype)
    assert np.max(np.abs(got - oracle.run_circuit(n, gates, psi0))) <= TOL[dtype]


def _reference(psi, terms):
    """sum_m c_m <psi|P_m|psi> by index arithmetic in FP64."""
    y = torch.arange(psi.numel(), device="cuda")
    psi = psi.to(torch.complex128)
    e = 0.0
    for t in terms:
        x = sum(1 << q for q, p in t.ops if p in "XY")
        odd = torch.zeros_like(y)
        for q, p in t.ops:
            if p in "YZ":
                odd ^= (y >> q) & 1
        # (P psi)[y ^ x] = i^{#Y} (-1)^{|z & y|} psi[y]
        phase = 1j ** sum(p == "Y" for _, p in t.ops)
        s = torch.sum(psi[y ^ x].conj() * torch.where(odd == 1, -psi, psi)).item()
        e += t.coeff * (phase * s).real
    return e


@pytest.mark.parametrize("dtype", DTYPES, ids=["c128", "c64"])
@pytest.mark.parametrize("n", [22, 23])
@pytest.mark.parametrize("kind", ["ring", "wide", "many"])
def test_expval(dtype, n, kind):
    rng = np.random.default_rng([n, 6])

    def string(weight):
        return tuple((int(q), "XYZ"[rng.integers(3)]) for q in rng.permutation(n)[:weight])

    if kind == "ring":      # one x mask per qubit, all diagonal terms together
        terms = vqa_hamiltonian(n)
    elif kind == "wide":    # masks that flip more qubits than a tile holds above its window
        terms = [PauliTerm(0.7 - s, tuple((q, "XY"[(q + s) % 2]) for q in range(n))) for s in range(2)]
        terms.append(PauliTerm(0.3, string(n)))
    else:                   # more strings than a launch holds
        terms = [PauliTerm(float(rng.normal()), string(int(rng.integers(1, 7)))) for _ in range(120)]
    psi = random_state_torch(n, seed=n, device="cuda", dtype=dtype, workload=23)
    print(f"expval n={n} {kind} terms={len(terms)} {dtype}", flush=True)
    got = cast.StateVector(n, tensor=psi).expval(terms)
    # products and sums are FP64 on both sides: n 2^-53 per term leaves 1e-13
    # per unit of coefficient
    assert got.imag == 0.0
    assert abs(got.real - _reference(psi, terms)) <= 1e-13 * sum(abs(t.coeff) for t in terms)
