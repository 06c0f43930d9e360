"""Matrices whose rows have the same column runs in pieces in some of their 64-row groups
only: the sample that is looked at first may see the one kind or the other, and whichever
kernels then run give the same bytes."""

import numpy as np
import pytest
import scipy.sparse as sp
import torch

import paper_2409_15818_amd as R

pytestmark = pytest.mark.gpu


def _mixed(groups, in_pieces, k, n, tail, seed):
    """Rows of k entries by 64-row groups: one run that all rows of the group share where
    in_pieces(group), else a random place in each k-th of the columns; then `tail` rows."""
    rng = np.random.default_rng(seed)
    e = np.arange(k + 1) * n // k
    cols = []
    for g in range(groups + (tail > 0)):
        rows = 64 if g < groups else tail
        if in_pieces(g):
            c = np.tile(rng.integers(0, n - k) + np.arange(k), (rows, 1))
        else:
            c = e[:-1] + (rng.random((rows, k)) * np.diff(e)).astype(np.int64)
        cols.append(c)
    col = np.concatenate(cols).reshape(-1).astype(np.int32)
    m = 64 * groups + tail
    return m, np.arange(m + 1) * k, col, rng.standard_normal(m * k)


# 192 groups are sampled at every twelfth.  All pieces, none, pieces only where the sample
# looks, only where it does not, every eighth of the sampled groups scattered, and fewer
# groups than the sample takes, with a ragged last one.  At least 2^20 entries, from where
# the transpose takes pieces at all.
CASES = [
    (192, lambda g: True, 90, 0), (192, lambda g: False, 90, 13), (192, lambda g: g % 12 == 0, 90, 1),
    (192, lambda g: g % 12 != 0, 90, 63), (192, lambda g: g % 96 != 0, 90, 5), (13, lambda g: True, 1300, 17),
    (13, lambda g: g % 2 == 0, 1300, 0),
]

# The sample is taken from 2^18 rows on: one row fewer and no more, the sampled
# groups in pieces and the others not and the other way round.
TALL = [(4096, lambda g: True, 0), (4095, lambda g: True, 63), (4096, lambda g: False, 1), (4096, lambda g: g % 256 == 0, 0),
        (4096, lambda g: g % 256 != 0, 7)]


@pytest.mark.parametrize("case", range(len(TALL)))
def test_many_rows(case):
    groups, kind, tail = TALL[case]
    n = 150
    m, ptr, col, val = _mixed(groups, kind, 5, n, tail, case)
    assert len(col) >= 1 << 20
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    T = R.rfmls_transpose(h, A)
    order = np.argsort(col, kind="stable")
    assert np.array_equal(T.row_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))]))
    assert np.array_equal(T.col.cpu().numpy(), np.repeat(np.arange(m), 5)[order])
    assert np.array_equal(T.val.cpu().numpy(), val[order])
    P = R.rfmls_precond_import_R(h, torch.eye(n, dtype=torch.float64, device="cuda"))
    dense = torch.zeros((m, n), dtype=torch.float64, device="cuda")
    dense[torch.arange(m, device="cuda").repeat_interleave(5), A.col.long()] = A.val
    assert torch.equal(R.rfmls_form_B(h, A, P), dense)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_pieces_in_some_groups(case):
    groups, kind, k, tail = CASES[case]
    n = 2900 if k == 1300 else 700
    m, ptr, col, val = _mixed(groups, kind, k, n, tail, case)
    assert len(col) >= 1 << 20
    h = R.Handle(device="cuda:0")
    A = R.CSR.from_numpy(ptr, col, val, m, n)
    T = R.rfmls_transpose(h, A)
    ref = sp.csr_matrix((val, col, ptr), shape=(m, n))
    tr = ref.T.tocsr()
    tr.sort_indices()
    assert np.array_equal(T.row_ptr.cpu().numpy(), tr.indptr)
    assert np.array_equal(T.col.cpu().numpy(), tr.indices)
    assert np.array_equal(T.val.cpu().numpy(), tr.data)
    # B = A I: every output one product a_ij * 1 plus zeros, the bits of A
    P = R.rfmls_precond_import_R(h, torch.eye(n, dtype=torch.float64, device="cuda"))
    assert np.array_equal(R.rfmls_form_B(h, A, P).cpu().numpy(), ref.toarray())
