"""The 32-column products of matrices without long pieces of rows with equal column
runs: windows of the input staged in LDS, row groups split by columns, the gradient
entry by entry, and the autotuner's window widths."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R

pytestmark = pytest.mark.gpu


def _scattered(m, n, k, seed):
    """Rows of k entries, one at a random place of each k-th of the columns."""
    rng = np.random.default_rng(seed)
    e = np.arange(k + 1) * n // k
    col = e[:-1] + (rng.random((m, k)) * np.diff(e)).astype(np.int64)
    return np.arange(m + 1) * k, col.reshape(-1).astype(np.int32), rng.standard_normal(m * k)


def _dense(ptr, col, val, m, n):
    Ad = np.zeros((m, n))
    Ad[np.repeat(np.arange(m), np.diff(ptr)), col] = val
    return Ad


# A matrix in pieces of rows with one run and a scattered one of the same rows, columns
# and entries on one handle: each is tuned among its own kernel's shapes.
def test_tuning_keeps_kinds_of_matrices_apart():
    m, n, k = 640, 100, 10
    rng = np.random.default_rng(1)
    pieces = np.repeat(rng.integers(0, n - k, size=m // 64), 64)[:, None] + np.arange(k)
    h = R.Handle(device="cuda:0")
    P = R.rfmls_precond_import_R(h, torch.eye(n, dtype=torch.float64, device="cuda"))
    for ptr, col, val in ((np.arange(m + 1) * k, pieces.reshape(-1).astype(np.int32), rng.standard_normal(m * k)),
                          _scattered(m, n, k, 2)):
        B = R.rfmls_form_B(h, R.CSR.from_numpy(ptr, col, val, m, n), P)
        assert np.array_equal(B.cpu().numpy(), _dense(ptr, col, val, m, n))
    rec = R.rfmls_tune_read(h)
    assert [(r["rows"], r["cols"], r["nnz"]) for r in rec] == [(m, n, m * k)] * 2
    assert rec[0]["choice"].startswith("runs") and "window" in rec[1]["choice"]


# Pieces of h rows at random places, cut by the 64-row groups: the run kernel from an
# average of six rows on, the windowed one below, the bits of A (B = A I) on either.
@pytest.mark.parametrize("runs,length", [(1, 37), (8, 3)])
@pytest.mark.parametrize("h", [3, 6, 7, 8, 16, 64])
def test_the_line_between_the_kernels(h, runs, length):
    m, n = 1500, 300
    rng = np.random.default_rng(h)
    gap = n // runs
    first = rng.integers(0, gap - length, size=(-(-m // h), runs)) + gap * np.arange(runs)
    col = (first[:, :, None] + np.arange(length)).reshape(len(first), -1).repeat(h, axis=0)[:m]
    k = runs * length
    ptr, col, val = np.arange(m + 1) * k, col.reshape(-1).astype(np.int32), rng.standard_normal(m * k)
    hd = R.Handle(device="cuda:0")
    P = R.rfmls_precond_import_R(hd, torch.eye(n, dtype=torch.float64, device="cuda"))
    B = R.rfmls_form_B(hd, R.CSR.from_numpy(ptr, col, val, m, n), P)
    assert np.array_equal(B.cpu().numpy(), _dense(ptr, col, val, m, n))
    pieces = len(set(range(0, m, h)) | set(range(0, m, 64)))
    (rec,) = R.rfmls_tune_read(hd)
    assert rec["choice"].startswith("runs") == (6 * pieces <= m), (pieces, rec["choice"])
