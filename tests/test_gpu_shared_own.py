"""svm_train_shared where its problems run side by side on workgroups of their own, on both sides of the
line to the common pass: alpha, f and the summary equal those of svm_train bit for bit."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


# the line: 256 / k workgroups of 512 threads that hold four rows of 32 words each, or one of 128 floats
@pytest.mark.parametrize("kind,d,n,k,prec,own", [
    ("dense", 4, 2, 8, 0, True), ("dense", 20, 511, 3, 0, True), ("dense", 20, 513, 1, 0, True),
    ("dense", 128, 16384, 8, 0, True), ("dense", 128, 16385, 8, 0, False), ("dense", 132, 2000, 2, 0, False),
    ("dense", 20, 4500, 7, 1, True), ("bits", 300, 2049, 5, 0, True), ("bits", 1000, 4000, 8, 1, True),
    ("bits", 1024, 32768, 8, 0, True), ("bits", 1024, 32769, 8, 0, True), ("bits", 1024, 65536, 8, 0, True),
    ("bits", 1024, 65537, 8, 0, False)])
def test_side_by_side(kind, d, n, k, prec, own):
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, d, k])
    data = g.gen_blobs(n, d, r) if kind == "dense" else g.gen_sparse_binary(n, d, 0.03, r)
    dp = S.to_device(data)
    ys = []
    for p in range(k):
        y = data.y.copy()
        if p and n > 2:
            flip = r.choice(n, n // 10, replace=False)
            y[flip] = -y[flip]
        ys.append(torch.as_tensor(y, device="cuda"))
    prec = (S.SVM_KERNEL_FP32, S.SVM_KERNEL_FP64)[prec]
    # problems stop at different iterations: by the tolerance or by caps of their own
    pars = [S.make_params(2.0, 0.5 * (p + 1) / d, 1e-3, 0, 0, 0.0, 150 + 60 * p, prec) for p in range(k)]
    alphas, fs = ([torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(k)] for _ in range(2))
    rc, res = S.svm_train_shared(dp, ys, pars, alphas, fs)
    assert rc >= 0, S.strerror(rc)
    assert (res[0].rows_streamed >= sum(x.iterations for x in res) * n) == own or k == 1
    for p in range(k):
        s1 = dp.s
        one = S.DeviceProblem(S.svm_problem_t(s1.n, s1.d, s1.layout, 0, s1.x, s1.ldx, s1.row_ptr, s1.col, s1.val,
                                              ys[p].data_ptr()), dp, n, d)
        a, f = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        rc, x = S.svm_train(one, pars[p], a, f)
        assert rc >= 0, S.strerror(rc)
        assert torch.equal(a, alphas[p]) and torch.equal(f, fs[p])
        assert (x.iterations, x.n_sv, x.n_bsv, x.status) == (res[p].iterations, res[p].n_sv, res[p].n_bsv,
                                                             res[p].status)
        assert x.beta == res[p].beta and x.dual_obj == res[p].dual_obj
