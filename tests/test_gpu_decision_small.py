"""Decision calls at the edges of the one-launch list of support vectors and of the place that the
validation's parts take, against NumPy in 64 bits; refused inputs stay refused."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("n", [2, 3, 63, 65, 1023, 1024, 1025, 2048, 4095, 4096, 4097])
def test_list_edges(n, share):
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, int(10 * share)])
    for train, query in ((g.gen_blobs(n, 3, r), g.gen_blobs(5, 3, r)),
                         (g.gen_sparse_binary(n, 40, 0.2, r), g.gen_sparse_binary(5, 40, 0.2, r))):
        alpha = r.uniform(0.1, 1.0, n) * (r.random(n) < share)
        a, b = train.to_dense().astype(np.float64), query.to_dense().astype(np.float64)
        d2 = ((b[:, None, :] - a[None, :, :]) ** 2).sum(2)
        want = np.exp(-0.1 * d2) @ (alpha * train.y) - 0.25
        got = S.decision_data(train, alpha, 0.25, 0.1, query, kernel_precision=S.SVM_KERNEL_FP64)
        assert np.abs(got - want).max() <= 1e-13 * (1.0 + alpha.sum())
        # FP32: |a|^2 + |b|^2 - 2ab of squares up to 50 to 2^-23 each, times gamma, and the exponential
        got = S.decision_data(train, alpha, 0.25, 0.1, query)
        assert np.abs(got - want).max() <= 2e-6 * (1.0 + alpha.sum())


@pytest.mark.parametrize("n,d", [(2, 1), (5, 1), (70, 3), (3000, 20)])
def test_refused(n, d):
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng(n)

    def call(**bad):
        x = r.normal(size=(n, d)).astype(np.float32)
        q = r.normal(size=(9, d)).astype(np.float32)
        y = np.where(np.arange(n) % 2, 1, -1).astype(np.int8)
        if "label" in bad:
            y[n - 1] = bad["label"]
        if "row" in bad:
            x[n - 1, d - 1] = bad["row"]
        if "query" in bad:
            q[8, 0] = bad["query"]
        train = S.to_device(g.SvmData("t", n, d, "dense", y, x=x))
        query = S.to_device(g.SvmData("q", 9, d, "dense", None, x=q), with_labels=False)
        out = torch.full((9,), 7.0, dtype=torch.float64, device="cuda")
        alpha = torch.ones(n, dtype=torch.float64, device="cuda")
        rc = S.svm_decision(train, alpha, 0.0, 0.5, query, out, S.SVM_KERNEL_FP32)
        return rc, bool((out == 7.0).all())

    assert call()[0] == S.SVM_OK
    assert call(label=0) == (S.SVM_EINVAL, True)
    assert call(row=np.inf) == (S.SVM_ENONFINITE, True)
    assert call(query=np.nan) == (S.SVM_ENONFINITE, True)
