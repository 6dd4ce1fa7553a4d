"""The dense FP32 kernel sum (products on the matrix cores, norms from a pass of their own) against NumPy in
64 bits, at the edges of its tiles, chunks and widths."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nq,d", [(2, 1, 1), (63, 64, 4), (64, 63, 5), (65, 65, 20), (130, 17, 33), (500, 129, 48),
                                    (1100, 15, 64), (300, 200, 65), (400, 70, 100), (1000, 300, 128), (5000, 3, 28)])
def test_against_64_bits(n, nq, d):
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, nq, d])
    train, query = g.gen_blobs(n, d, r), g.gen_blobs(nq, d, r)
    alpha = r.uniform(0.0, 1.0, n) * (r.random(n) < 0.8)
    gamma, beta = 1.0 / d, 0.25
    x, z = train.x.astype(np.float64), query.x.astype(np.float64)
    x2, z2 = (x * x).sum(1), (z * z).sum(1)
    d2 = np.maximum(z2[:, None] + x2[None, :] - 2.0 * (z @ x.T), 0.0)
    k = np.exp(-gamma * d2)
    got = S.decision_data(train, alpha, beta, gamma, query, kernel_precision=S.SVM_KERNEL_FP32)
    # each of |a|^2, |b|^2 and 2 a.b is a sum of d FP32 products, then two additions: at most d + 3 roundings of
    # at most |a|^2 + |b|^2 each way; |K / e^v - 1| <= (|v| + 1) 2^-21 for the exponential
    err = gamma * (d + 3) * 2.0 ** -23 * (z2[:, None] + x2[None, :]) + (gamma * d2 + 1.0) * 2.0 ** -21
    tol = (k * np.expm1(err)) @ alpha + 1e-13
    assert np.all(np.abs(got - (k @ (alpha * train.y) - beta)) <= tol)


@pytest.mark.parametrize("d", [3, 40, 128, 160])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 130])
def test_gamma_beyond_fp32(n, d):
    """gamma is finite and infinite as an FP32 number: every kernel value between different rows is 0, and rows
    beyond a chunk's end add nothing, against a query of zeros too."""
    from paper_1406_5161_amd import svmhip as S
    x = np.zeros((n, d), np.float32)
    x[:, 0] = 1.0 + np.arange(n)
    y = np.where(np.arange(n) % 2, 1, -1).astype(np.int8)
    train = g.SvmData("t", n, d, "dense", y, x=x)
    query = g.SvmData("q", 3, d, "dense", np.ones(3, np.int8),
                      x=np.stack([np.zeros(d), np.full(d, -1.0), np.zeros(d)]).astype(np.float32))
    out = S.decision_data(train, np.full(n, 0.5), 0.25, 1e39, query, kernel_precision=S.SVM_KERNEL_FP32)
    assert np.array_equal(out, np.full(3, -0.25))
