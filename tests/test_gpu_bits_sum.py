"""The bitset kernel sum (whole-number distances on the matrix cores, kernel values from a table) at the
edges of its tiles, chunks and widths, against NumPy in 64 bits."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def check(n, nq, d, share=0.7):
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, nq, d])
    train = g.gen_sparse_binary(n, d, 0.2, r)
    query = g.gen_sparse_binary(nq, d, 0.2, r)
    alpha = r.uniform(0.0, 1.0, n) * (r.random(n) < share)
    gamma, beta = 1.0 / d, 0.25
    a, b = train.to_dense().astype(np.float64), query.to_dense().astype(np.float64)
    v = -gamma * (b.sum(1)[:, None] + a.sum(1)[None, :] - 2.0 * (b @ a.T))
    c = alpha * train.y
    want = np.exp(v) @ c - beta
    for prec in (S.SVM_KERNEL_FP32, S.SVM_KERNEL_FP64):
        got = S.decision_data(train, alpha, beta, gamma, query, kernel_precision=prec)
        # |K / e^v - 1| <= (|v| + 1) 2^-21 in FP32 (|v| <= 2), a few ulp in FP64; sums in FP64
        tol = np.abs(c).sum() * (3.0 * 2.0 ** -21 if prec == S.SVM_KERNEL_FP32 else 1e-14) + 1e-13
        assert np.abs(got - want).max() <= tol


@pytest.mark.parametrize("d", [1, 2, 31, 63, 64, 65, 128, 129, 192, 256, 300, 320, 321, 384, 385, 512, 513, 768, 769,
                               1000, 1024])
def test_widths(d):
    check(150, 140, d)


@pytest.mark.parametrize("nq", [1, 15, 17, 63, 64, 65, 127, 129, 700])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1100])
def test_tiles(n, nq):
    check(n, nq, 300, share=1.0)
    check(n, nq, 700, share=0.5)


def test_all_bits():
    """The largest distance (2 d) and the least: rows of every column against rows of one."""
    import torch  # noqa: F401
    from paper_1406_5161_amd import svmhip as S
    d = 1024
    y = np.array([1, -1, 1], np.int8)
    rp = np.array([0, d, d + 1, 2 * d + 1], np.int32)
    col = np.concatenate([np.arange(d), [d - 1], np.arange(d)]).astype(np.int32)
    s = g.SvmData("all", 3, d, "csr", y, row_ptr=rp, col=col, val=np.ones(len(col), np.float32))
    x = s.to_dense().astype(np.float64)
    d2 = ((x[:, None, :] - x[None, :, :]) ** 2).sum(2)
    got = S.decision_data(s, np.ones(3), 0.0, 1.0 / d, s, kernel_precision=S.SVM_KERNEL_FP64)
    assert np.abs(got - np.exp(-d2 / d) @ y).max() <= 1e-14
