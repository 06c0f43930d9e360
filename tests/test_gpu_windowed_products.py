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


def _clustered(m, n, seed):
    """Every other column of a stretch of 39 (past the last column from the first on) that
    the rows of a group of 64 share, the stretches 13 columns apart."""
    rng = np.random.default_rng(seed)
    col = np.sort((13 * (np.arange(m) // 64)[:, None] + np.arange(0, 40, 2)) % n, axis=1)
    return np.arange(m + 1) * 20, col.reshape(-1).astype(np.int32), rng.standard_normal(20 * m)


# Lockstep solve, from zero and from a given start, and backward on the windowed kernel:
# both matrices in whole groups; a transpose whose rows are long enough for the groups to
# be split by columns (1,125 entries a row, nsplit = 4); rows of twenty runs; one and two
# blocks of right-hand sides.  kappa is O(10) and LSQR stops at 1e-13, as for the
# products over pieces: 1e-10 allows a hundred times that.
@pytest.mark.parametrize("nrhs", [2, 33])
@pytest.mark.parametrize("make,m,n", [(lambda: _scattered(700, 96, 12, 3), 700, 96),
                                      (lambda: _scattered(9000, 96, 12, 4), 9000, 96),
                                      (lambda: _clustered(1500, 101, 5), 1500, 101)])
def test_windowed_solve_and_gradients(make, m, n, nrhs):
    from oracle import backward

    ptr, col, val = make()
    Ad = _dense(ptr, col, val, m, n)
    rng = np.random.default_rng(6)
    B, G = rng.standard_normal((nrhs, m)), rng.standard_normal((nrhs, n))
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    AT = R.rfmls_transpose(h, A)
    P = R.rfmls_precond(h, R.rfmls_sketch(h, A, 4 * n, 2)[0])
    opts = R.default_opts(atol=1e-13, btol=1e-13)
    Bt = torch.tensor(B, device="cuda")
    want = np.linalg.lstsq(Ad, B.T, rcond=None)[0].T
    for x0 in (None, torch.tensor(want + 0.1 * rng.standard_normal(want.shape), device="cuda")):
        X, Res, info, rc = R.rfmls_solve(h, A, AT, P, Bt, opts, x0=x0)
        assert rc == 0
        assert np.linalg.norm(X.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
        assert np.linalg.norm(Res.cpu().numpy() - (B - want @ Ad.T)) <= 1e-10 * np.linalg.norm(B)
        for k in range(nrhs):
            r = B[k] - Ad @ want[k]
            assert abs(info[k]["normb"] - np.linalg.norm(B[k])) <= 1e-13 * np.linalg.norm(B[k])
            assert abs(info[k]["normr"] - np.linalg.norm(r)) <= 1e-10 * np.linalg.norm(r)
    dB, dA, _, rc = R.rfmls_solve_backward(h, A, AT, P, X, Res, torch.tensor(G, device="cuda"), opts)
    dBo, dAo = np.zeros((nrhs, m)), np.zeros(len(col))
    for k in range(nrhs):
        x, r, w, lam = backward.dense_gradients(Ad, B[k], G[k])
        dBo[k] = lam
        dAo += backward.pattern_grad(ptr, col, r, w, lam, x)
    assert rc == 0
    assert np.linalg.norm(dB.cpu().numpy() - dBo) <= 1e-10 * np.linalg.norm(dBo)
    assert np.linalg.norm(dA.cpu().numpy() - dAo) <= 1e-10 * np.linalg.norm(dAo)
    assert sorted((q["rows"], q["cols"]) for q in R.rfmls_tune_read(h)) == sorted([(m, n), (n, m)])
    assert all("window" in q["choice"] for q in R.rfmls_tune_read(h))


# Whatever width the tuner keeps (windows of 128 where a row's columns lie far apart, of
# 32 where a group's lie together), solve and gradients are bitwise those of the
# hand-picked 64.
@pytest.mark.parametrize("make,m,n", [(lambda: _scattered(6400, 900, 10, 8), 6400, 900),
                                      (lambda: _clustered(6400, 400, 9), 6400, 400)])
def test_window_widths_change_no_bit(make, m, n):
    ptr, col, val = make()
    B = torch.tensor(np.random.default_rng(1).standard_normal((5, m)), device="cuda")
    G = torch.tensor(np.random.default_rng(2).standard_normal((5, n)), device="cuda")
    out = []
    for tune in (False, True):
        h = R.Handle(device="cuda:0")
        R.rfmls_tune_enable(h, tune)
        A = R.CSR.from_numpy(ptr, col, val, m, n)
        AT = R.rfmls_transpose(h, A)
        P = R.rfmls_precond(h, R.rfmls_sketch(h, A, 4 * n, 2)[0])
        X, Res, _, _ = R.rfmls_solve(h, A, AT, P, B)
        dB, dA, _, _ = R.rfmls_solve_backward(h, A, AT, P, X, Res, G)
        rec = R.rfmls_tune_read(h)
        assert len(rec) == (2 if tune else 0) and all(q["candidates"] == 3 and "window" in q["choice"] for q in rec)
        print([(q["rows"], q["choice"]) for q in rec], flush=True)
        out.append((X.clone(), Res.clone(), dB.clone(), dA.clone()))
        h.close()
    assert all(torch.equal(a, b) for a, b in zip(*out))
