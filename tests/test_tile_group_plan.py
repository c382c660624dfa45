"""The launches apply_circuit plans (no GPU: grouping is planned on the host):
tiles and workgroups stay within what the kernel takes whatever an environment
variable, which no range check has seen, asks for, and blocks that the knobs
keep off the matrix cores keep a launch of their own."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2503_19894_amd as cast
from circuits import qft, rqc_u3_cx

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE_BYTES = 64 << 10
AMP = {torch.complex128: 16, torch.complex64: 8}

PROBE = """
import torch, paper_2503_19894_amd as cast
from circuits import qft
for dt in (torch.complex128, torch.complex64):
    for n in (9, 13, 20, 30):
        l = cast.FusedCircuit(n, qft(n), k_max=5).launches(dt)
        print(n, 16 if dt == torch.complex128 else 8, max(x["tile_bits"] for x in l),
              *sorted({x["threads"] for x in l if x["tile_bits"]}))
"""


@pytest.mark.parametrize("bits,threads", [("13", "512"), ("14", "300"), ("40", "128"), ("1000", "512"), ("8", "4096"),
                                          ("9", "300"), ("3", "300"), ("0", "0"), ("-2", "512")])
def test_environment_knobs(bits, threads):
    env = dict(os.environ, CAST_BLOCKED_TILE_BITS=bits, CAST_BLOCKED_THREADS=threads, CAST_NO_TUNING_FILE="1")
    r = subprocess.run([sys.executable, "-c", PROBE], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    rows = [[int(v) for v in line.split()] for line in r.stdout.strip().splitlines()]
    assert len(rows) == 8
    for n, amp, tb, *nt in rows:
        assert amp << tb <= TILE_BYTES and tb <= n
        assert (tb == 0) == (int(bits) < 8)
        assert set(nt) <= {256, 512, 1024} and all(t <= 1 << tb for t in nt)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
def test_launches_cover_the_list(dtype):
    n = 20
    fc = cast.FusedCircuit(n, qft(n), k_max=5)
    launches = fc.launches(dtype)
    assert len(launches) < fc.num_passes(dtype)
    at = 0
    for x in launches:
        assert x["first"] == at and AMP[dtype] << x["tile_bits"] <= TILE_BYTES
        at += x["count"]
    assert at == len(fc)
    cast.set_tuning("tile_groups", 0, dtype)
    try:
        assert [(x["first"], x["count"], 0, 0) for x in fc.schedule(dtype)] == [tuple(x.values()) for x in fc.launches(dtype)]
    finally:
        cast.set_tuning("tile_groups", 1, dtype)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
@pytest.mark.parametrize("knob,value,kept_out", [("mfma_min_d", 7, (4, 5)), ("mfma_min_d", 5, (4,)),
                                                 ("mfma_3m_min_d", 4, (4, 5)), ("mfma_3m_min_d", 5, (5,))])
def test_matrix_core_knobs(dtype, knob, value, kept_out):
    n = 16
    fc = cast.FusedCircuit(n, rqc_u3_cx(n, 5, seed=2), k_max=5)

    def grouped():
        return {fc.gate(g)["d"] for x in fc.launches(dtype) if x["tile_bits"]
                for g in range(x["first"], x["first"] + x["count"])}

    before = grouped()
    assert {4, 5} <= before
    old = cast.get_tuning(knob, dtype)
    cast.set_tuning(knob, value, dtype)
    try:
        assert not grouped() & set(kept_out)
    finally:
        cast.set_tuning(knob, old, dtype)
    assert grouped() == before


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64], ids=["c128", "c64"])
def test_tiles_of_256_lanes_cost_more(dtype):
    """A 9-qubit Fourier transform shares a launch in one tile of 2^9
    amplitudes, not in two of 2^8 on workgroups of 256 lanes."""
    fc = cast.FusedCircuit(9, qft(9), k_max=6)
    launches = fc.launches(dtype)
    assert {x["tile_bits"] for x in launches} == {0, 9}, launches
