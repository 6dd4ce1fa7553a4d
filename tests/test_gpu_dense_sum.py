"""The dense FP32 matrix-core kernel sum at the edges of its tiles (64 queries, 64 support vectors) and
row widths, against FP64 kernel values."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def check(n, nq, d, layout=0, share=0.7):
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, nq, d])
    train, query = g.gen_blobs(n, d, r), g.gen_blobs(nq, d, r)
    alpha = r.uniform(0.0, 1.0, n) * (r.random(n) < share)
    tp, qp = S.to_device(train, layout=layout), S.to_device(query, layout=layout, with_labels=False)
    a = torch.from_numpy(alpha).cuda()
    out = {}
    for prec in (S.SVM_KERNEL_FP32, S.SVM_KERNEL_FP64):
        o = torch.full((nq,), float("nan"), dtype=torch.float64, device="cuda")
        assert S.svm_decision(tp, a, 0.5, 0.05, qp, o, prec) == S.SVM_OK
        out[prec] = o.cpu().numpy()
    # FP32 sums of d products each in |a|^2, |b|^2 and a.b: gamma (d + 8) 2^-24 of the four terms' size
    big = max(float((train.x.astype(np.float64) ** 2).sum(1).max()), float((query.x.astype(np.float64) ** 2).sum(1).max()))
    tol = np.abs(alpha).sum() * (0.05 * (d + 8) * 4 * big + 4) * 2.0 ** -24 + 1e-12
    assert np.abs(out[0] - out[1]).max() <= tol


@pytest.mark.parametrize("d", [1, 4, 5, 8, 12, 13, 20, 24, 28, 29, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129])
def test_widths(d):
    check(130, 70, d)
    check(70, 130, d, layout=1)


@pytest.mark.parametrize("nq", [1, 15, 16, 17, 63, 64, 65, 129, 2000])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 1500])
def test_tiles(n, nq):
    check(n, nq, 28, share=1.0)


def test_no_support_vectors():
    check(50, 20, 28, share=0.0)
