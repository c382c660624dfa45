"""The single-pass kernels of apply_circuit, one launch per pass (tile_groups
off): the tests that name a kernel, a knob or a pass shape, run again where
those decide what is launched.  By default most of their passes share launches,
and the QFT on 30 qubits is seven of them."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2503_19894_amd as cast  # noqa: E402
from tests import test_gpu_fullsize as fullsize  # noqa: E402
from tests.test_gpu_blocked import test_blocked_matches_per_pass_path  # noqa: E402,F401
from tests.test_gpu_dense import (test_dense_haar_22_vs_oracle, test_dense_mfma_product_forms,  # noqa: E402,F401
                                  test_low_target_mfma_placement)
from tests.test_gpu_diag_runs import (knobs, test_run_knobs_vs_oracle, test_runs_on_and_off_agree,  # noqa: E402,F401
                                      test_runs_vs_oracle)
from tests.test_gpu_families import test_family_all_paths  # noqa: E402,F401
from tests.test_gpu_parity import (test_bitwise_deterministic, test_config1_rqc12_unfused,  # noqa: E402,F401
                                   test_direct_block_runs, test_direct_rotated_order, test_fused_circuits,
                                   test_guard_region_untouched, test_mfma_pass_rotation, test_pass_shapes_and_tuner,
                                   test_qft_closed_form_via_fft, test_small_states, test_tile_idle_runs_skipped)

DTYPES = [torch.complex128, torch.complex64]


@pytest.fixture(autouse=True)
def one_launch_per_pass():
    old = {dt: cast.get_tuning("tile_groups", dt) for dt in DTYPES}
    for dt in DTYPES:
        cast.set_tuning("tile_groups", 0, dt)
    yield
    for dt, v in old.items():
        cast.set_tuning("tile_groups", v, dt)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-12), (torch.complex64, 1e-5)], ids=["c128", "c64"])
def test_qft30(dtype, tol):
    fullsize.test_qft30_closed_form_and_inverse(dtype, tol, "per_pass")
    torch.cuda.empty_cache()
    fullsize.test_qft30_full_state_vs_fft(dtype, tol, "per_pass")
