"""Tile groups at the edges of what reaches them: knobs from the environment,
which no range check has seen, a stream that is being captured, and amplitudes
that are not finite, against the oracle."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2503_19894_amd as cast  # noqa: E402
from circuits import Gate, qft, random_state, rqc_u3_cx  # noqa: E402

TOL = {torch.complex128: 1e-12, torch.complex64: 1e-5}

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = """
import numpy as np, torch, oracle, paper_2503_19894_amd as cast
from circuits import qft, random_state, rqc_u3_cx
n = 15
for dt, tol in ((torch.complex128, 1e-12), (torch.complex64, 1e-5)):
    for gates in (qft(n), rqc_u3_cx(n, 5, seed=2)):
        psi = random_state(n, seed=1, workload=18)
        sv = cast.StateVector(n, tensor=torch.tensor(psi, dtype=dt, device="cuda"))
        fc = cast.FusedCircuit(n, gates, k_max=4)
        assert len(fc.launches(dt)) < fc.num_passes(dt)
        sv.apply_circuit(fc)
        assert np.max(np.abs(sv.numpy() - oracle.run_circuit(n, gates, psi))) <= tol, (dt, fc.launches(dt))
print("agree")
"""


@pytest.mark.parametrize("bits,threads", [(13, 512), (13, 300), (40, 128)])
def test_environment_knobs(bits, threads):
    env = dict(os.environ, CAST_BLOCKED_TILE_BITS=str(bits), CAST_BLOCKED_THREADS=str(threads))
    print(f"tile bits {bits} threads {threads}", flush=True)
    r = subprocess.run([sys.executable, "-c", PROBE], cwd=ROOT, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "agree" in r.stdout, r.stderr[-2000:]


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
@pytest.mark.parametrize("n", [10, 14, 18])
@pytest.mark.parametrize("bad", [(np.inf, 0.0), (-np.inf, np.inf), (np.nan, 1.0)])
def test_untouched_amplitudes(dtype, n, bad):
    """No gate acts on amplitude 0 (every phase is 1, every control 0, and the
    fused gates' blocks with it are the identity): it keeps its value, infinite
    or not, and no other amplitude meets it."""
    rng = np.random.default_rng(n)
    gates = []
    for q in range(4, n):
        gates += [Gate("cp", (q, int(p)), (float(rng.uniform(0.1, 3)),)) for p in rng.permutation(np.setdiff1d(range(4, n), q))[:3]]
        gates.append(Gate("cx", (q, q - 1)))
    psi = random_state(n, seed=n, workload=19)
    psi[0] = complex(*bad)
    fc = cast.FusedCircuit(n, gates, k_max=2)
    assert len(fc.launches(dtype)) < fc.num_passes(dtype)
    print(f"amplitude {bad} n={n} {dtype}: {len(fc.launches(dtype))} launches", flush=True)
    sv = cast.StateVector(n, tensor=torch.tensor(psi, dtype=dtype, device="cuda"))
    sv.apply_circuit(fc)
    out = sv.numpy()
    assert np.array_equal([out[0].real, out[0].imag], bad, equal_nan=True)
    assert np.isfinite(out[1:]).all()


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
@pytest.mark.parametrize("before", ["tune", "timed", "apply"])
def test_captured_after(before, dtype):
    """A list that any earlier call has put on the device can be captured."""
    n = 13
    gates = qft(n) + rqc_u3_cx(n, 3, seed=4)
    psi0 = random_state(n, seed=3, workload=20)
    fc = cast.FusedCircuit(n, gates, k_max=4)
    psi = torch.tensor(psi0, dtype=dtype, device="cuda")
    sv = cast.StateVector(n, tensor=psi)
    {"tune": sv.tune_circuit, "timed": sv.apply_circuit_timed, "apply": sv.apply_circuit}[before](fc)
    torch.cuda.synchronize()
    print(f"capture after {before} {dtype}", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cast.StateVector(n, tensor=psi).apply_circuit(fc)
    want = oracle.run_circuit(n, gates, psi0)
    for i in range(3):
        psi.copy_(torch.tensor(psi0, dtype=dtype))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.max(np.abs(psi.cpu().numpy() - want)) <= TOL[dtype]
        other = cast.StateVector(n, tensor=torch.tensor(psi0, dtype=dtype, device="cuda"))   # eager work between
        other.apply_circuit(fc)
        assert np.max(np.abs(other.numpy() - want)) <= TOL[dtype]
