"""Edges of the bitset kernel sums: rows beyond a chunk's end add nothing whatever gamma is."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def csr(rows, d, y):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col = np.concatenate([np.asarray(r, np.int32) for r in rows]).astype(np.int32)
    return g.SvmData("bits", len(rows), d, "csr", np.asarray(y, np.int8), row_ptr=rp, col=col,
                     val=np.ones(len(col), np.float32))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
def test_gamma_beyond_fp32(n):
    """gamma is finite and infinite as an FP32 number: every kernel value between different rows is 0."""
    from paper_1406_5161_amd import svmhip as S
    d = 40
    n += 1
    train = csr([[i % d] for i in range(n)], d, [1 if i % 2 else -1 for i in range(n)])
    queries = csr([[], [0, 1, 2], list(range(d)), []], d, [1, 1, 1, 1])
    out = S.decision_data(train, np.full(n, 0.5), 0.25, 1e39, queries, kernel_precision=S.SVM_KERNEL_FP32)
    assert np.array_equal(out, np.full(4, -0.25))


@pytest.mark.parametrize("d", [1, 40, 1023, 1024])
@pytest.mark.parametrize("prec", [0, 1])
def test_largest_distance(d, prec):
    """Rows of every column against rows of none: distance d, the last of the table."""
    from paper_1406_5161_amd import svmhip as S
    train = csr([list(range(d)), [], list(range(d)), [d - 1]], d, [1, -1, 1, -1])
    queries = csr([[], list(range(d)), [0]], d, [1, 1, 1])
    gamma = 1.0 / d
    alpha = np.array([1.0, 2.0, 0.5, 0.25])
    x, q = train.to_dense().astype(np.float64), queries.to_dense().astype(np.float64)
    d2 = ((q[:, None, :] - x[None, :, :]) ** 2).sum(2)
    assert d2.max() == d
    out = S.decision_data(train, alpha, 0.25, gamma, queries, kernel_precision=prec)
    want = np.exp(-gamma * d2) @ (alpha * train.y) - 0.25
    # |K / e^v - 1| <= (|v| + 1) 2^-21 in FP32 (|v| <= 1), a few ulp in FP64
    tol = alpha.sum() * (2.0 * 2.0 ** -21 if prec == S.SVM_KERNEL_FP32 else 1e-15) + 1e-15
    assert np.abs(out - want).max() <= tol
