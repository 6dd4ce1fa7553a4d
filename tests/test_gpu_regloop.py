"""The SMO loop with its rows in registers (dense and bitset rows) against the loop that streams them
from HBM: the same pairs, alpha, f and counts bit for bit, at the edges of its row widths, rows per
thread, waves, records per load and records per merging wave."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu

CAP = 3000


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1406_5161_amd import svmhip
    svmhip.lib()
    return svmhip


def make(kind, n, d, seed, dup=False):
    r = np.random.default_rng([n, d, seed])
    if kind == "dense":
        data = g.gen_blobs(n, d, r)
        if dup:                      # equal rows: ties in f, decided by the lowest id
            k = n // 2
            data.x[k:2 * k] = data.x[:k]
            data.y[k:2 * k] = data.y[:k]
    else:
        data = g.gen_sparse_binary(n, d, 0.12, r)
        if dup:
            data = data.subset(np.concatenate([np.arange(n - n // 2), np.arange(n // 2)]))
    return data


def run(S, data, prec, grid, flags, shrink):
    import torch
    tr = [torch.zeros(CAP, dtype=torch.int32, device="cuda") for _ in range(2)]
    tb = [torch.zeros(CAP, dtype=torch.float64, device="cuda") for _ in range(2)]
    S.svm_debug_set_trace(CAP, *tr, *tb)
    try:
        out = S.train_data(data, 1.0, 0.05 if data.layout == "dense" else 1.0 / data.d, max_iter=CAP,
                           kernel_precision=prec, grid_blocks=grid, flags=flags, shrink_mode=2 if shrink else 0,
                           shrink_param=2.0)
    finally:
        S.svm_debug_set_trace(0)
    return out, [t.cpu().numpy() for t in tr + tb]


def check(S, data, prec, grid, shrink):
    old, tr0 = run(S, data, prec, grid, S.SVM_FLAG_NO_LDS_PAYLOAD, shrink)
    assert S.svm_debug_step_info()[0] == 1
    new, tr1 = run(S, data, prec, grid, 0, shrink)
    assert new.rc == old.rc and new.rc in (S.SVM_OK, S.SVM_NOT_CONVERGED)
    assert S.svm_debug_step_info()[0] == 2
    if grid:
        assert new.result["grid_blocks"] == min(grid, data.n)
    for a, b in zip(tr0, tr1):
        assert np.array_equal(a, b)
    assert np.array_equal(old.alpha, new.alpha) and np.array_equal(old.f, new.f)
    for k in ("iterations", "n_recon", "shrink_passes", "shrunk_total", "rows_streamed", "nnz_streamed", "beta",
              "dual_obj", "b_up", "b_low", "n_sv", "n_bsv"):
        assert old.result[k] == new.result[k], k


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "fp64"])
@pytest.mark.parametrize("d", [1, 4, 5, 8, 12, 15, 20, 23, 28, 32, 33, 48, 49, 64, 65, 96, 97, 128])
def test_dense_widths(S, d, prec):
    check(S, make("dense", 700, d, 1), prec, 3, True)
    check(S, make("dense", 300, d, 2), prec, 0, False)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "fp64"])
@pytest.mark.parametrize("d", [3, 128, 129, 256, 300, 500, 700, 1000, 1024])
def test_bitset_widths(S, d, prec):
    check(S, make("bits", 700, d, 1), prec, 3, True)
    check(S, make("bits", 300, d, 2), prec, 0, False)


@pytest.mark.parametrize("kind,d", [("dense", 20), ("bits", 300)])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 511, 512, 513, 1024, 1025, 2047, 2048])
def test_rows_of_one_workgroup(S, kind, d, n):
    check(S, make(kind, n, d, 3), 0, 1, n > 100)


@pytest.mark.parametrize("kind,d", [("dense", 28), ("bits", 300)])
@pytest.mark.parametrize("grid", [2, 7, 8, 9, 31, 33, 63, 64, 65, 127, 129, 192, 193, 255, 256])
def test_grids(S, kind, d, grid):
    check(S, make(kind, 3001, d, 4), 0, grid, True)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind,d", [("dense", 20), ("bits", 60)])
def test_ties(S, kind, d, prec):
    for grid in (1, 5, 70):
        check(S, make(kind, 500, d, 5, dup=True), prec, grid, True)
