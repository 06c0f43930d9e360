"""Kernels at the sizes where they change path: slice and tile remainders, the
smallest and the largest of a range, through the C-ABI against plain numpy."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R
from oracle import backward
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
    U = np.linalg.qr(Ad)[1]
    P = R.rfmls_precond_import_R(h, torch.tensor(np.sign(np.diag(U))[:, None] * U, device="cuda"))
    x, res, _, rc = R.rfmls_solve_explicit(h, A, AT, P, R.rfmls_form_B(h, A, P), torch.tensor(b, device="cuda"), opts)
    want = np.linalg.lstsq(Ad, b, rcond=None)[0]
    assert rc == 0
    assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
    assert np.linalg.norm(res.cpu().numpy() - (b - Ad @ want)) <= 1e-10 * np.linalg.norm(b)


def _blocks(pieces, n, seed):
    """CSR rows by (rows, [(first column, length), ...]) pieces, values N(0, 1)."""
    rng = np.random.default_rng(seed)
    ptr, col, val = [0], [], []
    for rows, runs in pieces:
        cols = np.concatenate([np.arange(c, c + k) for c, k in runs]) if runs else np.zeros(0, int)
        for _ in range(rows):
            col.append(cols)
            val.append(rng.standard_normal(cols.size))
            ptr.append(ptr[-1] + cols.size)
    return np.array(ptr, np.int64), np.concatenate(col).astype(np.int32), np.concatenate(val)


# 32-column products over pieces of dense runs: row counts at the edges of the
# 16-row tiles and of a 64-row group, run lengths at the edges of a 16-entry
# step, rows without entries, one to eight runs a row, and (the last two) rows
# of nine runs and pieces too short, which take the windowed kernel.  B = A X
# with X = I: every output is one product a_ij * 1 plus zeros, so B equals A bit
# for bit on either kernel.
RUN_CASES = [
    (40, [(64, [(0, 40)]), (64, [(0, 16)])]),
    (131, [(15, [(0, 15)]), (17, [(3, 17)]), (33, [(0, 1)]), (1, [(130, 1)]), (63, [(5, 33), (60, 70)])]),
    (300, [(100, [(0, 300)]), (49, []), (16, [(1, 31), (40, 47), (90, 16), (200, 100)]), (70, [(299, 1)])]),
    (90, [(48, [(10 * k, 5) for k in range(8)]), (32, [(0, 64)])]),
    (90, [(48, [(10 * k, 5) for k in range(9)]), (60, [(0, 64)])]),
    (64, [(1, [(k, 1 + k % 3)]) for k in range(62)]),
]


@pytest.mark.parametrize("case", range(len(RUN_CASES)))
def test_run_products_reproduce_the_matrix(case):
    n, pieces = RUN_CASES[case]
    ptr, col, val = _blocks(pieces, n, case)
    m = len(ptr) - 1
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    P = R.rfmls_precond_import_R(h, torch.eye(n, dtype=torch.float64, device="cuda"))
    want = np.zeros((m, n))
    want[np.repeat(np.arange(m), np.diff(ptr)), col] = val
    assert np.array_equal(R.rfmls_form_B(h, A, P).cpu().numpy(), want)


# The transposed product with long rows, split into K chunks that are then
# merged, and more right-hand sides than one block of 32: per column the
# lockstep solution is the single-column one (another summation order), both
# within 10 * 1e-13 of the least-squares solution at kappa = O(10).
@pytest.mark.parametrize("nrhs", [2, 33])
def test_run_products_in_chunks(nrhs):
    n = 96
    pieces = [(900, [(0, 48)]), (700, [(48, 48)]), (333, [(0, 96)]), (5, [])]
    ptr, col, val = _blocks(pieces, n, 7)
    m = len(ptr) - 1
    Ad = np.zeros((m, n))
    Ad[np.repeat(np.arange(m), np.diff(ptr)), col] = val
    B = np.random.default_rng(1).standard_normal((nrhs, m))
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    AT = R.rfmls_transpose(h, A)
    SA, _, _, _ = R.rfmls_sketch(h, A, 4 * n, 2)
    P = R.rfmls_precond(h, SA)
    X, Res, _, rc = R.rfmls_solve(h, A, AT, P, torch.tensor(B, device="cuda"), R.default_opts(atol=1e-13, btol=1e-13))
    want = np.linalg.lstsq(Ad, B.T, rcond=None)[0].T
    assert rc == 0
    assert np.linalg.norm(X.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
    assert np.linalg.norm(Res.cpu().numpy() - (B - want @ Ad.T)) <= 1e-10 * np.linalg.norm(B)


# The matrix gradient over pieces of rows with common column runs: pieces and runs
# with remainders of 16, one-entry runs, empty rows, and a second block of 32
# right-hand sides added to the first.  Oracle and bound as above (kappa = O(10)).
# The wide matrix's rows are long enough for K chunks.
GRADIENT_CASES = [
    (96, [(450, [(0, 48)]), (350, [(48, 48)]), (333, [(0, 96)]), (70, [(3, 17), (40, 1), (60, 33)]), (5, []),
          (17, [(95, 1)])]),
    (700, [(1500, [(0, 700)]), (70, [(3, 517), (540, 1), (560, 133)]), (5, [])]),
]


@pytest.mark.parametrize("nrhs", [2, 33])
@pytest.mark.parametrize("case", range(len(GRADIENT_CASES)))
def test_matrix_gradient_over_run_pieces(case, nrhs):
    n, pieces = GRADIENT_CASES[case]
    ptr, col, val = _blocks(pieces, n, 9)
    m = len(ptr) - 1
    Ad = np.zeros((m, n))
    Ad[np.repeat(np.arange(m), np.diff(ptr)), col] = val
    rng = np.random.default_rng(2)
    B, G = rng.standard_normal((nrhs, m)), rng.standard_normal((nrhs, n))
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    AT = R.rfmls_transpose(h, A)
    SA, _, _, _ = R.rfmls_sketch(h, A, 4 * n, 2)
    P = R.rfmls_precond(h, SA)
    opts = R.default_opts(atol=1e-13, btol=1e-13)
    X, Res, _, _ = R.rfmls_solve(h, A, AT, P, torch.tensor(B, device="cuda"), opts)
    dB, dA, _, rc = R.rfmls_solve_backward(h, A, AT, P, X, Res, torch.tensor(G, device="cuda"), opts)
    dBo, dAo = np.zeros((nrhs, m)), np.zeros(len(col))
    for k in range(nrhs):
        x, r, w, lam = backward.dense_gradients(Ad, B[k], G[k])
        dBo[k] = lam
        dAo += backward.pattern_grad(ptr, col, r, w, lam, x)
    assert rc == 0
    assert np.linalg.norm(dB.cpu().numpy() - dBo) <= 1e-10 * np.linalg.norm(dBo)
    assert np.linalg.norm(dA.cpu().numpy() - dAo) <= 1e-10 * np.linalg.norm(dAo)


def _staircase(s, n, width, per_row, seed, zero_rows=0):
    """Rows with entries in `per_row` random blocks of `width` columns, as a count
    sketch of box-structured rows has them; the last zero_rows rows empty."""
    rng = np.random.default_rng(seed)
    M = np.zeros((s, n))
    nb = -(-n // width)
    for i in range(s - zero_rows):
        for q in rng.choice(nb, size=min(nb, per_row), replace=False):
            M[i, q * width:(q + 1) * width] = rng.standard_normal(min(n, (q + 1) * width) - q * width)
    return M


# QR of sketches whose rows start late, factored in sorted row order: the last
# panel ragged, one to three outer blocks, entries that start inside a panel, the
# moving slabs smaller than the matrix, empty rows, and the right-hand sides' extra
# columns.  R^T R = (SA)^T SA to the gate of the dense factorisations, 20 n u.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("s,n,width,per_row,zero_rows", [
    (9000, 250, 25, 1, 0), (6000, 400, 40, 2, 500), (5200, 577, 30, 2, 0), (3300, 640, 64, 1, 3),
    (33500, 320, 20, 1, 100)])
def test_qr_of_rows_that_start_late(s, n, width, per_row, zero_rows, dtype):
    SA = _staircase(s, n, width, per_row, s + n, zero_rows)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    td = torch.float64 if dtype == "f64" else torch.float32
    h = R.Handle(device="cuda:0")
    gram = SA.T @ SA
    Rs = []
    for extra in (0, 2):
        buf = R.sketch_buffer(s, n + extra, dtype)
        buf.zero_()
        buf[:, :n] = torch.tensor(SA, device="cuda", dtype=td)
        if extra:
            Sb = torch.randn((extra, s), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
            P, X0 = R.rfmls_precond_x0(h, buf, n, Sb, dtype, dtype)
            if dtype == "f64":  # kappa(SA) is a few tens: the least-squares solution to 1e-11
                want = np.linalg.lstsq(SA, Sb.cpu().numpy().T, rcond=None)[0].T
                assert np.linalg.norm(X0.cpu().numpy() - want) <= 1e-11 * np.linalg.norm(want)
        else:
            P = R.rfmls_precond(h, buf[:, :n], dtype, dtype)
        Rm = R.rfmls_precond_export_R(h, P).cpu().numpy()
        assert np.all(np.diag(Rm) > 0) and np.array_equal(Rm, np.triu(Rm))
        ref = gram if dtype == "f64" else None
        if ref is None:
            S32 = SA.astype(np.float32).astype(np.float64)
            ref = S32.T @ S32
        assert np.linalg.norm(Rm.T @ Rm - ref) <= 20 * n * u * np.linalg.norm(SA) ** 2
        Rs.append(Rm)


# Transposes of at least 2^20 entries, which are sorted piece by piece where the
# rows' runs allow it: pieces cut by the 64-row groups, runs that leave a 64-entry
# tile, empty rows, more columns than one counting pass holds (16,384); and the two
# kinds that are not (a row of nine runs; every row with runs of its own).  Whole
# numbers and copies: equal to scipy's transpose bit for bit.
TRANSPOSES = [
    (700, [(900, [(0, 333)]), (37, []), (1501, [(10, 64), (200, 65), (699, 1)]), (1, [(5, 7)]), (3000, [(333, 200)])]),
    (20000, [(5000, [(100 * k, 30) for k in range(7)]), (130, [(16000, 2000)]), (63, [(19999, 1)]), (65, [(0, 20000)])]),
    (400, [(4000, [(0, 300)]), (64, [(10 * k, 5) for k in range(9)])]),
    (2000, [(1, [(k % 1500, 200 + k % 300)]) for k in range(4000)]),
]


@pytest.mark.parametrize("case", range(len(TRANSPOSES)))
def test_transpose_piece_by_piece(case):
    import scipy.sparse as sp

    n, pieces = TRANSPOSES[case]
    ptr, col, val = _blocks(pieces, n, case)
    m = len(ptr) - 1
    assert ptr[-1] >= 1 << 20
    h = R.Handle(device="cuda:0")
    T = R.rfmls_transpose(h, R.CSR.from_numpy(ptr, col, val, m, n))
    ref = sp.csr_matrix((val, col, ptr), shape=(m, n)).T.tocsr()
    ref.sort_indices()
    assert np.array_equal(T.row_ptr.cpu().numpy(), ref.indptr)
    assert np.array_equal(T.col.cpu().numpy(), ref.indices)
    assert np.array_equal(T.val.cpu().numpy(), ref.data)


# Sketch rows whose buckets hold rows of two distant gapless halves, odd and even
# entry counts, single entries, empty rows and rows with gaps, with windows below and
# above both window sizes: the same adds in the same order as the oracle, so equal
# bit for bit.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("s,big", [(7, False), (40, False), (7, True), (300, True)])
def test_sketch_of_two_span_rows(s, big, dtype):
    from oracle import countsketch

    n = 9001 if big else 1203
    w = 900 if big else 40
    runs = [[(0, w)], [(5, w), (n - w, w)], [(0, w + 1), (2 * w + 3, w)], [(n - 1, 1)], [],
            [(w, 1), (n - 2, 1)], [(3, 2), (9, 2), (20, 2)], [(w // 2, 7), (n // 2, 8)]]
    ptr, col, val = _blocks([(5 if k % 2 else 2, runs[k % len(runs)]) for k in range(24)], n, s)
    m = len(ptr) - 1
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    SA, hg, sg, _ = R.rfmls_sketch(h, A, s, 11, dtype=dtype, want_maps=True)
    ho, so = countsketch.hash_sign(m, s, 11)
    ref, _ = countsketch.sketch_dense(ptr, col, val, ho, so, s, n)
    assert np.array_equal(hg.cpu().numpy(), ho) and np.array_equal(sg.cpu().numpy(), so)
    assert np.array_equal(SA.cpu().numpy(), ref if dtype == "f64" else ref.astype(np.float32))


# X = R^{-1} over outer blocks of 1,024 rows whose near sums are carried from block
# row to block row: one outer block with a ragged tail, exactly one, and two or three
# with the last ragged.  Each column is a back substitution: |R X - I| <= n u |R||X|
# and as much again for the product taken here; 4 n u allows twice that.
@pytest.mark.parametrize("n", [1, 64, 65, 200, 1024, 1025, 1100, 2112, 2113])
def test_inverse_over_outer_blocks(n):
    rng = np.random.default_rng(n)
    U = np.triu(rng.standard_normal((n, n)), 1) / np.sqrt(n) + np.diag(1.0 + rng.random(n))
    h = R.Handle(device="cuda:0")
    P = R.rfmls_precond_import_R(h, torch.tensor(U, device="cuda"))
    X = R.rfmls_precond_export_Rinv(h, P).cpu().numpy()
    err = np.linalg.norm(U @ X - np.eye(n))
    assert err <= 4 * n * 2.0 ** -53 * np.linalg.norm(np.abs(U) @ np.abs(X)), err
