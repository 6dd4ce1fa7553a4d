"""The head/tail kernel sum at the edges of its tables: tiles of 64, 32 and 16 target rows and rows too
long for any, columns at both ends, equal column counts, empty and one-element rows, fewer columns in
use than the head has, and row and support-vector counts around its tiles and chunks; decision values
against FP64 kernel values."""
import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def rows(r, n, d, nnz, pool=None):
    """n rows of nnz[i] distinct columns, values exp(N(0, 0.5)), unit norm."""
    cols = [np.sort(r.choice(pool if pool is not None else d, size=k, replace=False)) for k in nnz]
    vals = [np.exp(0.5 * r.standard_normal(k)) for k in nnz]
    vals = [v / np.linalg.norm(v) if len(v) else v for v in vals]
    rp = np.concatenate([[0], np.cumsum(nnz)]).astype(np.int32)
    y = np.ones(n, np.int8)
    y[1::2] = -1
    return g.SvmData("edges", n, d, "csr", y, row_ptr=rp, col=np.concatenate(cols).astype(np.int32),
                     val=np.concatenate(vals).astype(np.float32))


CASES = {
    # name: (d, training rows, queries, nonzeros per training row, per query, columns used)
    "least_d": (12289, 300, 100, 20, 20, None),
    "most_d": (65535, 300, 100, 20, 20, None),
    "one_query": (20000, 300, 1, 30, 30, None),
    "tile_63": (20000, 129, 63, 30, 30, None),
    "tile_65": (20000, 127, 65, 30, 30, None),
    "chunk_64": (20000, 64, 64, 30, 30, None),
    "one_sv": (20000, 2, 70, 30, 30, None),
    "tile_full": (65535, 200, 128, 40, 88, None),        # 64 rows of 88: 5632, the table's size
    "tile_of_32": (65535, 200, 128, 40, 89, None),
    "tile_of_16": (65535, 200, 100, 40, 200, None),
    "no_tile": (65535, 200, 100, 40, 400, None),
    "few_columns": (30000, 300, 100, 20, 20, 60),         # all of them in the head
    "dense_columns": (30000, 300, 200, 60, 60, 160),      # every tail column in most rows of a tile
    "long_sv": (40000, 400, 64, 900, 20, None),           # more tail entries a chunk than are held ahead
}


@pytest.mark.parametrize("name", CASES)
def test_decision(name):
    from paper_1406_5161_amd import svmhip as S
    d, n, nq, kt, kq, used = CASES[name]
    r = np.random.default_rng([n, nq, d])
    pool = None if used is None else r.choice(d, size=used, replace=False)
    nt, qt = np.full(n, kt), np.full(nq, kq)
    if name in ("least_d", "most_d"):
        nt[3], qt[5], nt[9], qt[7] = 0, 0, 1, 1
    train, query = rows(r, n, d, nt, pool), rows(r, nq, d, qt, pool)
    # the first and last columns, in rows of both sides
    for s in (train, query):
        if used is None:
            p = s.row_ptr[0]
            s.col[p], s.col[s.row_ptr[1] - 1] = 0, d - 1
    alpha = r.uniform(0.0, 4.0, n) * (r.random(n) < 0.8)
    alpha[0] = 1.0
    gamma, beta = 1.0, 0.25
    lo = S.decision_data(train, alpha, beta, gamma, query)
    hi = S.decision_data(train, alpha, beta, gamma, query, kernel_precision=S.SVM_KERNEL_FP64)
    # a kernel value is e^v of v = -gamma d^2, |v| <= 4 here: norms and dots summed in FP32 over at most
    # 900 products of magnitude <= 1 in all (error <= 900 ulp of 1 at worst, some ulp in practice), and
    # exp and its argument a few ulp more: 1e-5 of each value covers the sums' usual rounding
    tol = 1e-5 * np.abs(alpha).sum()
    assert np.abs(lo - hi).max() <= tol
    assert np.isfinite(lo).all()
