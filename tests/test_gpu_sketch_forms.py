"""The forms of the sketch-row kernel at the lines between them, bit for bit against the
oracle: the same adds in the same order."""

import numpy as np
import pytest
import torch

import paper_2409_15818_amd as R
from oracle import countsketch

pytestmark = pytest.mark.gpu


def _two_boxes(m, n, w, seed):
    """Rows over one gapless stretch of w columns or two of them far apart, every seventh
    row empty, every fifth with gaps."""
    rng = np.random.default_rng(seed)
    ptr, col, val = [0], [], []
    for i in range(m):
        a = int(rng.integers(0, n // 2 - w))
        c = np.arange(a, a + w)
        if i % 3 == 0:
            c = np.concatenate([c, c + n // 2])
        if i % 5 == 0:
            c = c[rng.random(len(c)) < 0.5]
        if i % 7 == 0:
            c = c[:0]
        col.append(c)
        val.append(rng.standard_normal(len(c)))
        ptr.append(ptr[-1] + len(c))
    return np.array(ptr, np.int64), np.concatenate(col).astype(np.int32), np.concatenate(val)


# Fewer than three rows a bucket, three, more; rows short and long against the wide
# window's line (256 entries, 1,024 a bucket, 4,096 columns); buckets of more rows than
# are sorted; aligned rows and rows that are not.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("m,n,w,s", [(299, 5001, 40, 100), (300, 5001, 40, 100), (301, 5001, 40, 100), (900, 5001, 60, 30),
                                     (200, 5001, 700, 40), (200, 5001, 160, 16), (200, 3000, 160, 16), (400, 9000, 30, 4)])
def test_sketch_forms(m, n, w, s, pad, dtype):
    ptr, col, val = _two_boxes(m, n, w, m + n + s)
    td = torch.float64 if dtype == "f64" else torch.float32
    SA = torch.full((s, n + 8 + pad), 7.0, dtype=td, device="cuda")[:, :n]
    h = R.Handle(device="cuda:0")
    R.rfmls_sketch(h, R.CSR.from_numpy(ptr, col, val, m, n), s, 11, dtype=dtype, SA=SA)
    ho, so = countsketch.hash_sign(m, s, 11)
    ref, _ = countsketch.sketch_dense(ptr, col, val, ho, so, s, n)
    assert np.array_equal(SA.cpu().numpy(), ref if dtype == "f64" else ref.astype(np.float32))


# Rows of one or two columns at every second place: more intervals than wavefronts, a
# column between them, so that the 16-byte segments of the output hold parts of two, and
# one span a row or, past the window, two.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n,far", [(37, 0), (64, 0), (2045, 0), (4999, 2498), (9000, 4500), (9001, 6000)])
def test_sketch_of_many_intervals(n, far, pad, dtype):
    m, s = 96, 9
    rng = np.random.default_rng(n)
    near = n - far if far else n
    first = 2 * rng.integers(0, min(near, 60) // 2, size=m)
    col = np.stack([first, first + far], 1).astype(np.int32) if far else first[:, None].astype(np.int32)
    ptr = np.arange(m + 1) * col.shape[1]
    val = rng.standard_normal(col.size)
    td = torch.float64 if dtype == "f64" else torch.float32
    SA = torch.full((s, n + 8 + pad), 7.0, dtype=td, device="cuda")[:, :n]
    h = R.Handle(device="cuda:0")
    R.rfmls_sketch(h, R.CSR.from_numpy(ptr, col.reshape(-1), val, m, n), s, 5, dtype=dtype, SA=SA)
    ho, so = countsketch.hash_sign(m, s, 5)
    ref, _ = countsketch.sketch_dense(ptr, col.reshape(-1), val, ho, so, s, n)
    assert np.array_equal(SA.cpu().numpy(), ref if dtype == "f64" else ref.astype(np.float32))
