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
