"""The plane rotations of the SVD preconditioner at the ends of float64's range and
to its last bits, against LAPACK's SVD of the oracle's sketch."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R
from oracle import countsketch
from rfmgen import csr_from_dense, dense_with_condition

pytestmark = pytest.mark.gpu


def _sketch(Ad, s, seed):
    m, n = Ad.shape
    rp, col, val = csr_from_dense(Ad, keep_zeros=True)
    h, sign = countsketch.hash_sign(m, s, seed)
    return countsketch.sketch_dense(rp, col, val, h, sign, s, n)[0]


# All columns so short that twice a pair's product is subnormal near convergence:
# scaling by a power of two scales every rounding, so the singular values are those of
# the unscaled sketch to the usual 2e-12 of sigma_1.
@pytest.mark.parametrize("exponent", [-498, -250, 400])
def test_svd_of_a_scaled_sketch(exponent):
    n = 20
    SA = _sketch(dense_with_condition(200, n, 1e3, seed=3), 60, 5)
    want = np.linalg.svd(SA, compute_uv=False)
    h = R.Handle(device="cuda:0")
    P = R.rfmls_precond_svd(h, torch.tensor(SA * 2.0 ** exponent, device="cuda"), n)
    sig = np.sort(R.rfmls_precond_export_sigma(h, P).cpu().numpy())[::-1]
    assert P.status == 0 and P.rank == n and P.off <= 1.0
    assert np.max(np.abs(sig * 2.0 ** -exponent - want)) <= 2e-12 * want[0]
    U = SA @ (R.rfmls_precond_export_P(h, P).cpu().numpy() * 2.0 ** exponent)
    assert np.max(np.abs(U.T @ U - np.eye(n))) <= n * 2.0 ** -53 * want[0] / want[-1] + 1e-12


# One rotation makes two columns orthogonal: formed to the last bits it leaves a cosine
# of some 4 u from t and 3 u each from applying it and from its measurement, against
# the tolerance of 16 u for two columns, so the second sweep rotates nothing.
def test_svd_of_two_columns_takes_one_rotation():
    h = R.Handle(device="cuda:0")
    sweeps = []
    for seed in range(24):
        SA = np.random.default_rng(seed).standard_normal((16, 2)) @ np.array([[1.0, 0.5], [0.0, 0.7]])
        P = R.rfmls_precond_svd(h, torch.tensor(SA, device="cuda"), 2)
        assert P.status == 0 and P.rank == 2 and P.off <= 16 * 2.0 ** -53
        sweeps.append(P.sweeps)
    assert max(sweeps) <= 2, sweeps


# Beyond the sizes whose blocks are few: P = V Sigma^{-1} of a sketch of 2,500 and 4,200
# columns, kappa 1e4.  V = P Sigma is orthogonal and U = SA P has orthonormal columns, to
# 8 n u and to what kappa amplifies; the singular values' squares sum to the sketch's.
@pytest.mark.parametrize("n", [2500, 4200])
def test_svd_of_many_columns(n):
    s = 2 * n
    gen = torch.Generator("cuda").manual_seed(n)
    SA = torch.randn((s, n), dtype=torch.float64, device="cuda", generator=gen)
    SA *= torch.logspace(0, -3, n, dtype=torch.float64, device="cuda")
    h = R.Handle(device="cuda:0")
    P = R.rfmls_precond_svd(h, SA.clone(), n)
    sig = R.rfmls_precond_export_sigma(h, P)
    X = R.rfmls_precond_export_P(h, P)
    u = 2.0 ** -53
    assert P.status == 0 and P.rank == n
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    V, U = X * sig, SA @ X
    assert float((V.T.contiguous() @ V - eye).abs().max()) <= 8 * n * u
    kappa = float(sig.max() / sig.min())
    assert float((U.T.contiguous() @ U - eye).abs().max()) <= n * u * kappa + 1e-12
    assert abs(float((sig ** 2).sum() / (SA ** 2).sum()) - 1.0) <= 8 * n * u


# Few columns, whose sweeps run in one launch up to 32: one column, padding inside the
# pairs' rounds, the whole group, and one column more.  kappa 1e4; the sweeps' limit is
# kept to, and what it leaves is still an SVD's V to rounding.
@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 16, 31, 32, 33])
def test_svd_of_few_columns(n):
    SA = _sketch(dense_with_condition(8 * n + 30, n, 1e4 if n > 1 else 1.0, seed=n), 4 * n + 5, 3)
    want = np.linalg.svd(SA, compute_uv=False)
    h = R.Handle(device="cuda:0")
    P = R.rfmls_precond_svd(h, torch.tensor(SA, device="cuda"), n)
    sig = R.rfmls_precond_export_sigma(h, P).cpu().numpy()
    X = R.rfmls_precond_export_P(h, P).cpu().numpy()
    assert P.status == 0 and P.rank == n and P.sweeps >= 1 and P.off <= max(8.0, n ** 0.5) * 2.0 ** -52
    assert np.max(np.abs(np.sort(sig)[::-1] - want)) <= 2e-12 * want[0]
    U = SA @ X
    assert np.max(np.abs(U.T @ U - np.eye(n))) <= n * 2.0 ** -53 * want[0] / want[-1] + 1e-12
    for most in range(1, P.sweeps + 1):
        Q = R.rfmls_precond_svd(h, torch.tensor(SA, device="cuda"), n, max_sweeps=most)
        assert Q.sweeps == most and Q.status == (0 if most == P.sweeps else 1) and Q.off <= 1.0
        V = R.rfmls_precond_export_P(h, Q).cpu().numpy() * R.rfmls_precond_export_sigma(h, Q).cpu().numpy()
        assert np.max(np.abs(V.T @ V - np.eye(n))) <= 64 * n * 2.0 ** -53
