"""The QR of sketches whose rows are factored in the order of where they start: what it
refuses, its fallback panels and its look-ahead."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R

pytestmark = pytest.mark.gpu


# A panel's grid holds 512 rows a compute unit.  One row more is refused whether or not
# most rows are empty and would never reach a panel; at the limit R^T R = (SA)^T SA to
# the gate of the other factorisations, 20 n u.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_qr_refuses_rows_beyond_a_panel_grid(dtype):
    n, live = 64, 3000
    most = 512 * torch.cuda.get_device_properties(0).multi_processor_count
    td = torch.float64 if dtype == "f64" else torch.float32
    M = np.random.default_rng(3).standard_normal((live, n)).astype(np.float64 if dtype == "f64" else np.float32)
    h = R.Handle(device="cuda:0")

    def sketch(s):
        SA = torch.zeros((s, n), dtype=td, device="cuda")
        SA[:: s // live][:live] = torch.tensor(M, device="cuda")
        return SA

    with pytest.raises(R.RfmlsError) as e:
        R.rfmls_precond(h, sketch(most + 1), dtype, dtype)
    assert e.value.status == -1
    P = R.rfmls_precond(h, sketch(most), dtype, dtype)
    Rm = R.rfmls_precond_export_R(h, P).cpu().numpy()
    M = M.astype(np.float64)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    assert np.linalg.norm(Rm.T @ Rm - M.T @ M) <= 20 * n * u * np.linalg.norm(M) ** 2
