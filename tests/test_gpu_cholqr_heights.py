"""CholeskyQR2 panels at the least heights that take them, 128 rows, and their fallbacks
there."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R

pytestmark = pytest.mark.gpu


def _factor(handle, SA, mode, dtype):
    R.rfmls_qr_panel_mode(handle, mode)
    try:
        P = R.rfmls_precond(handle, torch.tensor(SA, device="cuda"), dtype, dtype)
        Rm = R.rfmls_precond_export_R(handle, P).cpu().numpy()
        P.free()
    finally:
        R.rfmls_qr_panel_mode(handle, 0)
    return Rm


# One panel of 127 rows (unblocked), 128 (one slab) and 129 (a ragged second slab); two
# whose last has 127, 128 or 129; three whose last has 129.  Modes 2 and 3 fail the first
# and the second Cholesky of every panel that CholeskyQR2 takes: then the unblocked
# kernel's R bit for bit, and Q1's R times R1.  R^T R = (SA)^T SA to 20 n u, and R to
# what that leaves open, 20 n u kappa^2 of a row.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n", [(127, 64), (128, 64), (129, 64), (191, 128), (192, 128), (193, 128), (257, 192)])
def test_panels_at_128_rows(handle, m, n, dtype):
    SA = np.random.default_rng(m + n).standard_normal((m, n)).astype(np.float64 if dtype == "f64" else np.float32)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    Sd = SA.astype(np.float64)
    tol = 20 * n * u
    kappa = np.linalg.cond(Sd)
    R1 = _factor(handle, SA, 1, dtype)
    scale = np.abs(R1).max(axis=1, keepdims=True)
    for mode in (0, 1, 2, 3):
        Rm = _factor(handle, SA, mode, dtype)
        assert np.all(np.diag(Rm) > 0) and not np.tril(Rm, -1).any()
        assert np.linalg.norm(Rm.T @ Rm - Sd.T @ Sd) <= tol * np.linalg.norm(Sd) ** 2, mode
        assert (np.abs(Rm - R1) / scale).max() <= tol * kappa ** 2, mode
        if mode == 2:
            assert np.array_equal(Rm, R1)
