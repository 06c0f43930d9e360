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
    n, live = 256, 3000
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


def _staircase(s, n, width, seed, dtype):
    """Rows with entries in two random blocks of `width` columns; every 50th row empty."""
    rng = np.random.default_rng(seed)
    M = np.zeros((s, n), np.float64 if dtype == "f64" else np.float32)
    nb = -(-n // width)
    for i in range(s):
        if i % 50 == 49:
            continue
        for q in rng.choice(nb, size=2, replace=False):
            M[i, q * width:(q + 1) * width] = rng.standard_normal(min(n, (q + 1) * width) - q * width)
    return M


# Both forced fallbacks over sorted rows: the first Cholesky failed leaves the unblocked
# kernel's R bit for bit, the second its R of Q1 times R1.  Gates as for dense sketches.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("s,n,width", [(9000, 300, 25), (5200, 577, 40)])
def test_fallback_panels_over_sorted_rows(handle, s, n, width, dtype):
    M = _staircase(s, n, width, s, dtype)
    Md = M.astype(np.float64)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    Rs = []
    for mode in (1, 2, 3):
        R.rfmls_qr_panel_mode(handle, mode)
        try:
            P = R.rfmls_precond(handle, torch.tensor(M, device="cuda"), dtype, dtype)
            Rs.append(R.rfmls_precond_export_R(handle, P).cpu().numpy())
        finally:
            R.rfmls_qr_panel_mode(handle, 0)
        assert np.linalg.norm(Rs[-1].T @ Rs[-1] - Md.T @ Md) <= 20 * n * u * np.linalg.norm(Md) ** 2, mode
    assert np.array_equal(Rs[0], Rs[1])


# Look-ahead over sorted rows, outer blocks of 256 and 512 columns, the last ragged: the
# whole factored sketch bit for bit the plain schedule's.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_lookahead_over_sorted_rows(handle, dtype):
    n = 1100 if dtype == "f64" else 1690
    M = _staircase(3 * n, n, 90, 5, dtype)
    F = []
    for la in (False, True, True):
        R.rfmls_qr_lookahead(handle, la)
        try:
            SA = torch.tensor(M, device="cuda")
            P = R.rfmls_precond(handle, SA, dtype, dtype)
            torch.cuda.synchronize()
            F.append((SA.cpu().numpy(), R.rfmls_precond_export_R(handle, P).cpu().numpy()))
        finally:
            R.rfmls_qr_lookahead(handle, False)
    for f in F[1:]:
        assert np.array_equal(F[0][0], f[0]) and np.array_equal(F[0][1], f[1])


# The count of the rows by their panel: one chunk of 4,096 and several with a ragged last,
# every row of one panel, and empty panels, against the dense factorisation's gate.
@pytest.mark.parametrize("s,n,first", [(8192, 256, lambda i, n: 0 * i), (8193, 300, lambda i, n: i * n // 9000),
                                       (20001, 321, lambda i, n: np.where(i % 2 == 0, 0, n - 60))])
def test_rows_by_their_panels(handle, s, n, first):
    rng = np.random.default_rng(s)
    M = rng.standard_normal((s, n))
    M[np.arange(n)[None, :] < np.minimum(first(np.arange(s), n), n - 1)[:, None]] = 0.0
    M = M[rng.permutation(s)]
    P = R.rfmls_precond(handle, torch.tensor(M, device="cuda"))
    Rm = R.rfmls_precond_export_R(handle, P).cpu().numpy()
    assert np.all(np.diag(Rm) > 0) and not np.tril(Rm, -1).any()
    assert np.linalg.norm(Rm.T @ Rm - M.T @ M) <= 20 * n * 2.0 ** -53 * np.linalg.norm(M) ** 2
