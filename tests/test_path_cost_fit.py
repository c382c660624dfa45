"""The calibration of in-tile gate costs (no GPU): a fit in which more gates took
no longer is no measurement and is not stored, and the stored costs are of the
order of what a gate does to 2^30 amplitudes in a tile."""
import json
import os

import pytest

import paper_2503_19894_amd as cast
from paper_2503_19894_amd.autotune import gate_slope


def test_slope():
    assert gate_slope([(4, 2.0), (24, 6.0)]) == pytest.approx((0.2, 1.2))
    assert gate_slope([(4, 2.0), (24, 2.0)]) is None
    assert gate_slope([(4, 2.0), (24, 1.9)]) is None


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_stored_gate_costs(dtype):
    """One pass over LDS: 2^30 amplitudes read and written at the 256 compute
    units' 128 bytes a cycle and 2.4 GHz take 0.22 ms in complex64; gates share
    passes (two- and more-qubit tables), but not tens of them."""
    with open(os.path.join(os.path.dirname(cast.__file__), "tuning_gfx950.json")) as f:
        cost = json.load(f)["path_cost"][dtype]
    for d in range(4):
        assert 0.01 < cost[f"seg_gate{d}"] < 20, (d, cost[f"seg_gate{d}"])
