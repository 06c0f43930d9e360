"""Kernels at the sizes where they change path: slice and tile remainders, the
smallest and the largest of a range, through the C-ABI against plain numpy."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R
from rfmgen import csr_from_dense, dense_with_condition

pytestmark = pytest.mark.gpu


def _csr(Ad):
    rp, col, val = csr_from_dense(Ad, keep_zeros=True)
    return R.CSR.from_numpy(rp, col, val, *Ad.shape)


# B^T u by row slices: fewer rows than a slice holds, row remainders of the
# eight-row steps, column counts at the edges of a 256-column block.  kappa = 10
# and LSQR stopped at 1e-13 leave x within about 10 * 1e-13 ||b|| / ||A x||;
# 1e-10 allows a hundred times that.
@pytest.mark.parametrize("m,n", [(3, 1), (63, 20), (65, 64), (400, 255), (513, 256), (1031, 257), (1999, 520)])
def test_explicit_operator_slices(m, n):
    Ad = dense_with_condition(m, n, 10.0, seed=m)
    b = np.random.default_rng(n).standard_normal(m)
    h = R.Handle(device="cuda:0")
    A = _csr(Ad)
    opts = R.default_opts(atol=1e-13, btol=1e-13)
    AT = R.rfmls_transpose(h, A)
    P = R.rfmls_precond_import_R(h, torch.tensor(np.abs(np.diag(np.diag(np.linalg.qr(Ad)[1]))) +
                                                 np.eye(n), device="cuda"))
    x, res, _, rc = R.rfmls_solve_explicit(h, A, AT, P, R.rfmls_form_B(h, A, P), torch.tensor(b, device="cuda"), opts)
    want = np.linalg.lstsq(Ad, b, rcond=None)[0]
    assert rc == 0
    assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
    assert np.linalg.norm(res.cpu().numpy() - (b - Ad @ want)) <= 1e-10 * np.linalg.norm(b)
