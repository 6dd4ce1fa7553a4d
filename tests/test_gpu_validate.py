"""Input validation on the device: one bad value anywhere in the samples is found, whatever share of
the rows the workgroup that checks it holds, and nothing else is reported."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# one row, around one workgroup's share (64 rows), around the most workgroups (256)
SIZES = [2, 63, 64, 65, 129, 16384, 16385, 20011]


def _call(n, d, layout, x=None, ldx=0, csr=None, y=None):
    import torch
    from paper_1406_5161_amd import svmhip as S
    dev = [torch.from_numpy(a).cuda() for a in ((x, y) if csr is None else (*csr, y))]
    if csr is None:
        s = S.svm_problem_t(n, d, layout, 0, dev[0].data_ptr(), ldx, None, None, None, dev[1].data_ptr())
    else:
        s = S.svm_problem_t(n, d, S.SVM_CSR, 0, None, 0, dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(),
                            dev[3].data_ptr())
    p = S.DeviceProblem(s, tuple(dev), n, d)
    alpha = torch.zeros(n, dtype=torch.float64, device="cuda")
    rc, r = S.svm_train(p, S.make_params(1.0, 0.1, max_iter=1, flags=S.SVM_FLAG_NO_FINAL_RECOMPUTE), alpha)
    return rc, r


def _labels(n):
    y = np.ones(n, np.int8)
    y[1::2] = -1
    return y


@pytest.mark.parametrize("layout", ["rows", "strided", "features"])
@pytest.mark.parametrize("n", SIZES)
def test_dense(n, layout):
    from paper_1406_5161_amd import svmhip as S
    d = 5
    rng = np.random.default_rng([n, 1])
    x = rng.standard_normal((n, d)).astype(np.float32)

    def run(x, y):
        if layout == "rows":
            return _call(n, d, S.SVM_DENSE_ROW_MAJOR, x, d, y=y)[0]
        if layout == "strided":   # the padding is not part of the samples
            w = np.full((n, d + 3), np.nan, np.float32)
            w[:, :d] = x
            return _call(n, d, S.SVM_DENSE_ROW_MAJOR, w, d + 3, y=y)[0]
        return _call(n, d, S.SVM_DENSE_FEATURE_MAJOR, np.ascontiguousarray(x.T), n, y=y)[0]

    assert run(x, _labels(n)) in (S.SVM_OK, S.SVM_NOT_CONVERGED)
    for i, k in ((0, 0), (n - 1, d - 1), (n // 2, 2), (min(n - 1, 64), 0)):
        for v in (np.nan, np.inf, -np.inf):
            bad = x.copy()
            bad[i, k] = v
            assert run(bad, _labels(n)) == S.SVM_ENONFINITE
    for i in (0, n - 1, n // 2):
        y = _labels(n)
        y[i] = 0
        assert run(x, y) == S.SVM_EINVAL
    assert run(x, np.ones(n, np.int8)) == S.SVM_EONECLASS


@pytest.mark.parametrize("n", SIZES)
def test_csr(n):
    from paper_1406_5161_amd import svmhip as S
    d = 40
    rng = np.random.default_rng([n, 2])
    lens = rng.integers(0, 35, n)     # empty rows among them, and more than one step of a row's lanes
    lens[0] = lens[-1] = 34
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.permutation(d)[:m]) for m in lens]).astype(np.int32)
    ones = np.ones(len(col), np.float32)
    y = _labels(n)
    rc, r = _call(n, d, S.SVM_CSR, csr=(rp, col, ones), y=y)
    assert rc in (S.SVM_OK, S.SVM_NOT_CONVERGED) and r.pattern_only == 1
    rows = np.flatnonzero(lens >= 2)
    for i in (rows[0], rows[-1], rows[len(rows) // 2]):
        last = rp[i + 1] - 1
        v = ones.copy()
        v[last] = 2.0
        rc, r = _call(n, d, S.SVM_CSR, csr=(rp, col, v), y=y)
        assert rc in (S.SVM_OK, S.SVM_NOT_CONVERGED) and r.pattern_only == 0
        v[last] = np.nan
        assert _call(n, d, S.SVM_CSR, csr=(rp, col, v), y=y)[0] == S.SVM_ENONFINITE
        for p, c in ((last, d), (rp[i], -1), (last, col[last - 1])):
            bad = col.copy()
            bad[p] = c
            assert _call(n, d, S.SVM_CSR, csr=(rp, bad, ones), y=y)[0] == S.SVM_EINVAL
    bad = rp.copy()
    bad[0] = 1
    assert _call(n, d, S.SVM_CSR, csr=(bad, col, ones), y=y)[0] == S.SVM_EINVAL
    if n > 2:
        bad = rp.copy()
        bad[n // 2] = rp[n // 2 + 1] + 1   # the next pointer falls
        assert _call(n, d, S.SVM_CSR, csr=(bad, col, ones), y=y)[0] == S.SVM_EINVAL
