"""The automatic grid of CSR problems spreads the same work over more workgroups than a grid of 700 rows
each: residency of the rows, lanes per row, and so every sum, stay those of that grid, and alpha and f
are equal bit for bit."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def make(kind, n):
    r = np.random.default_rng([n, len(kind)])
    if kind == "text":           # slot map, rows from HBM
        return g.gen_text_like(n, 20_000, 75.0, r)
    if kind == "short":          # column table, rows that fit the LDS
        return g.gen_text_like(n, 3000, 6.0, r)
    data = g.gen_sparse_binary(n, 2000, 0.02, r)   # values all 1.0, too wide for bitsets
    return data


@pytest.mark.parametrize("prec", [0, 1], ids=["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["text", "short", "ones"])
@pytest.mark.parametrize("n", [100, 255, 257, 1025, 4096, 4097, 9001])
def test_same_results(kind, n, prec):
    from paper_1406_5161_amd import svmhip as S
    data = make(kind, n)
    kw = dict(kernel_precision=prec, shrink_mode=2, shrink_param=2.0, max_iter=1500)
    old = S.train_data(data, 2.0, 1.0 if kind != "ones" else 0.02, grid_blocks=1 if n <= 4096 else (n + 350) // 700, **kw)
    mode0, G0, L0 = S.svm_debug_step_info()
    new = S.train_data(data, 2.0, 1.0 if kind != "ones" else 0.02, **kw)
    mode1, G1, L1 = S.svm_debug_step_info()
    print(kind, n, "mode", mode0, mode1, "grid", G0, G1, "lanes", L0, L1, flush=True)
    assert L0 == L1 and G1 >= G0 and (mode0 == 2) == (mode1 == 2)
    assert old.rc == new.rc and old.result["iterations"] == new.result["iterations"]
    assert np.array_equal(old.alpha, new.alpha) and np.array_equal(old.f, new.f)
