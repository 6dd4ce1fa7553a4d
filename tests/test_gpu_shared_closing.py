"""svm_train_shared through its closing recompute where one pass serves all problems: the re-test and the
thresholds are taken over every row, so the result is that of svm_train, b_up and b_low included."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


# (dense: one row past what fits the chip eight times; bits: payload flag, which asks for the common pass)
@pytest.mark.parametrize("kind,d,n,k,payload", [("dense", 128, 16385, 8, True), ("dense", 64, 33000, 8, True),
                                                ("dense", 20, 6000, 3, False), ("bits", 300, 6000, 3, False),
                                                ("bits", 300, 6000, 3, True)])
def test_closing_test_over_all_rows(kind, d, n, k, payload):
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, d, k])
    data = g.gen_blobs(n, d, r) if kind == "dense" else g.gen_sparse_binary(n, d, 0.12, r)
    dp = S.to_device(data)
    ys = []
    for p in range(k):
        y = data.y.copy()
        flip = r.choice(n, n // 20 * (p % 3), replace=False)
        y[flip] = -y[flip]
        ys.append(torch.as_tensor(y, device="cuda"))
    flags = 0 if payload else S.SVM_FLAG_NO_LDS_PAYLOAD
    pars = [S.make_params(1.0, (0.5 + 0.25 * p) / d, 1e-3, 0, 0, 0.0, 10**9, S.SVM_KERNEL_FP32, flags)
            for p in range(k)]
    alphas, fs = ([torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(k)] for _ in range(2))
    rc, res = S.svm_train_shared(dp, ys, pars, alphas, fs)
    assert rc == S.SVM_OK, S.strerror(rc)
    for p in range(k):
        s = dp.s
        one = S.DeviceProblem(S.svm_problem_t(s.n, s.d, s.layout, 0, s.x, s.ldx, s.row_ptr, s.col, s.val,
                                              ys[p].data_ptr()), dp, n, d)
        a, f = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        rc, x = S.svm_train(one, pars[p], a, f)
        assert rc == S.SVM_OK
        assert (x.iterations, x.n_launches) == (res[p].iterations, res[p].n_launches)
        assert torch.equal(a, alphas[p]) and torch.equal(f, fs[p])
        assert (x.b_up, x.b_low, x.beta, x.dual_obj) == (res[p].b_up, res[p].b_low, res[p].beta, res[p].dual_obj)
        # the thresholds are those of the returned f over all rows
        al, fv, y = a.cpu().numpy(), f.cpu().numpy(), ys[p].cpu().numpy()
        up = ((y > 0) & (al < 1.0)) | ((y < 0) & (al > 0.0))
        low = ((y > 0) & (al > 0.0)) | ((y < 0) & (al < 1.0))
        assert (res[p].b_up, res[p].b_low) == (fv[up].min(), fv[low].max())
