"""Tile groups at the edges of what reaches them: knobs from the environment,
which no range check has seen, against the oracle."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

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
