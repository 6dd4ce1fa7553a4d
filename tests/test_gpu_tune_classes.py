"""A tuned grid is used where it was measured: by the loop that ran it, and never with fewer workgroups than
hold a problem's rows."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


@pytest.fixture
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1406_5161_amd import svmhip
    svmhip.svm_autotune_reset()
    yield svmhip
    svmhip.svm_autotune_reset()


def solve(S, dp, n, par):
    import torch
    a, f = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
    rc, _ = S.svm_train(dp, par, a, f)
    assert rc >= 0, S.strerror(rc)
    return (a, f), S.svm_debug_step_info()


def equal(x, y):
    import torch
    return all(torch.equal(a, b) for a, b in zip(x, y))


def test_larger_size_of_a_class_keeps_its_loop(S):
    d, small, large = 100, 16400, 32768     # one class; the small size's candidates end at 49, the large needs 64
    par = S.make_params(1.0, 0.01, 1e-3, 0, 0, 0.0, 200, S.SVM_KERNEL_FP32)
    dp = S.to_device(g.gen_blobs(large, d, np.random.default_rng(1)))
    before, info = solve(S, dp, large, par)
    assert info[0] == 2
    rc, _ = S.svm_autotune(S.to_device(g.gen_blobs(small, d, np.random.default_rng(2))), par, S.SVM_TUNE_GRID)
    assert rc == S.SVM_OK
    after, info = solve(S, dp, large, par)
    assert info[0] == 2 and info[1] >= 64
    assert equal(before, after)


def test_the_other_loop_keeps_its_rule(S):
    n, d = 20000, 64
    dp = S.to_device(g.gen_blobs(n, d, np.random.default_rng(3)))
    par = S.make_params(1.0, 0.01, 1e-3, 0, 0, 0.0, 200, S.SVM_KERNEL_FP32)
    cached = S.make_params(1.0, 0.01, 1e-3, 0, 0, 0.0, 200, S.SVM_KERNEL_FP32, cache_mb=1700)
    before, info = solve(S, dp, n, cached)
    rc, _ = S.svm_autotune(dp, par, S.SVM_TUNE_GRID)     # measures the loop with its rows in registers
    assert rc == S.SVM_OK
    after, again = solve(S, dp, n, cached)
    assert again == info and equal(before, after)


@pytest.mark.parametrize("kind", ["text", "values", "dense"])
def test_tuned_grid_is_no_slower_than_the_one_taken_without(S, kind):
    """The grid that a solve takes by itself is among the candidates, and the tuned solve gives its bits."""
    r = np.random.default_rng(4)
    n = 6000
    if kind == "dense":
        data = g.gen_blobs(n, 40, r)
    else:
        data = g.gen_text_like(n, 20000, 60, r) if kind == "text" else g.gen_sparse_binary(n, 300, 0.12, r)
        data.val = (data.val * r.uniform(0.5, 1.5, len(data.val))).astype(np.float32)
    par = S.make_params(2.0, 0.05 if kind == "dense" else 0.5, 1e-3, 0, 0, 0.0, 400, S.SVM_KERNEL_FP32)
    dp = S.to_device(data)
    before, info = solve(S, dp, n, par)
    rc, tune = S.svm_autotune(dp, par, S.SVM_TUNE_GRID)
    assert rc == S.SVM_OK
    print(kind, info, tune, flush=True)
    us = {c["shape"]: c["us_per_iter"] for c in tune["candidates"]}
    assert len(us) == len(tune["candidates"]) and info[1] in us
    assert us[tune["chosen"]] <= us[info[1]]
    after, again = solve(S, dp, n, par)
    assert again[1] == tune["chosen"] and again[2] == info[2]
    assert equal(before, after)


def test_malformed_rows_are_refused(S):
    dp = S.to_device(g.gen_sparse_binary(500, 300, 0.12, np.random.default_rng(6)))
    par = S.make_params(1.0, 0.01, 1e-3, 0, 0, 0.0, 50, S.SVM_KERNEL_FP32)
    rp = dp.keep[0]
    rp[200] = rp[201] + 1      # the next pointer falls
    for target in (S.SVM_TUNE_GRID, S.SVM_TUNE_TEAM):
        assert S.svm_autotune(dp, par, target)[0] == S.SVM_EINVAL
