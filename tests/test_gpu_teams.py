"""Teams enlarged where a batch leaves workgroups idle: the solution and the summary are those of a team
of one, alone or beside other launches that take the workgroups first."""
import threading

import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu


def problems(S, ns, prec):
    import torch
    data, par = [], []
    for j, n in enumerate(ns):
        r = np.random.default_rng([n, j])
        data.append(g.gen_blobs(n, (20, 128)[j % 2], r) if j % 3 else g.gen_sparse_binary(n, 300, 0.12, r))
        par.append(S.make_params(1.0, 0.01, 1e-3, 2, 1, 0.05, 3000, prec))
    return [S.to_device(x) for x in data], par, [torch.zeros(n, dtype=torch.float64, device="cuda") for n in ns]


def solve(S, made, team):
    import torch
    probs, par, alphas = made
    for p in par:
        p.grid_blocks = team
    fs = [torch.zeros_like(a) for a in alphas]
    rc, res = S.svm_train_batch(probs, par, alphas, fs)
    assert rc >= 0, S.strerror(rc)
    return res, [a.cpu().numpy().copy() for a in alphas], [f.cpu().numpy() for f in fs]


def same(x, y):
    for j, (p, q) in enumerate(zip(x[0], y[0])):
        assert np.array_equal(x[1][j], y[1][j]) and np.array_equal(x[2][j], y[2][j])
        assert (p.iterations, p.n_sv, p.n_bsv, p.beta, p.dual_obj) == (q.iterations, q.n_sv, q.n_bsv, q.beta,
                                                                       q.dual_obj)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ns", [(2, 3), (63, 64, 65), (512, 513, 1025, 2049), (5000,), (700,) * 40])
def test_enlarged_teams(ns, prec):
    from paper_1406_5161_amd import svmhip as S
    made = problems(S, ns, (S.SVM_KERNEL_FP32, S.SVM_KERNEL_FP64)[prec])
    one, auto = solve(S, made, 1), solve(S, made, 0)
    assert sum(r.grid_blocks for r in auto[0]) <= 256
    if ns == (5000,):
        assert auto[0][0].grid_blocks > 4
    same(one, auto)


def test_launches_that_overlap():
    """Four host threads, each with a stream of its own: a team takes what is free and gives the same."""
    import torch
    from paper_1406_5161_amd import svmhip as S
    mades = [problems(S, ns, S.SVM_KERNEL_FP32) for ns in ((3000, 2500), (4000,), (1500, 2000, 900), (3500, 600))]
    ref = [solve(S, m, 1) for m in mades]
    got, err = [None] * 4, []

    def work(t):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(2):
                    got[t] = solve(S, mades[t], 0)
        except Exception as e:   # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not err
    for a, b in zip(ref, got):
        same(a, b)


@pytest.mark.parametrize("kind", ["dense", "wide", "bits", "values"])
def test_rows_per_member(kind):
    """Members with rows for one, two and four rows a lane group, in LDS or streamed, with room for alpha
    in LDS or not; 17 members and up read the records with every wave."""
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([7, len(kind)])
    n = 4200
    data = (g.gen_blobs(n, 20, r) if kind == "dense" else g.gen_blobs(n, 160, r) if kind == "wide"
            else g.gen_sparse_binary(n, 300, 0.12, r))
    if kind == "values":
        data.val = (data.val * r.uniform(0.5, 1.5, len(data.val))).astype(np.float32)
    dp = S.to_device(data)
    a0, f0 = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
    base = None
    for team in (1, 2, 3, 4, 5, 8, 9, 16, 17, 33, 63, 64):
        p = S.make_params(3.0, 0.01, 1e-3, 2, 1, 0.05, 1200, S.SVM_KERNEL_FP32)
        p.grid_blocks = team
        rc, res = S.svm_train_batch([dp], [p], [a0], [f0])
        assert rc >= 0 and res[0].grid_blocks == team
        got = (res[0].iterations, res[0].shrink_passes, res[0].shrunk_total, res[0].n_sv, res[0].beta)
        if base is None:
            base = (got, a0.clone(), f0.clone())
        assert got == base[0]
        assert torch.equal(a0, base[1]) and torch.equal(f0, base[2])
