"""Elementwise kernels of the caller and small classifier calls run beside a live serving loop: they do not
wait until it stops, which it does after two seconds without work.

The calls run in one child process, whose streams are few: HIP maps streams onto four hardware queues, and a
stream that shares the loop's queue waits for it, whatever the kernels are."""
import json
import os
import subprocess
import sys
import time

import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DECISIONS = [("dense", 400, 8, 400, 0), ("dense", 2000, 20, 16, 0), ("dense", 5000, 20, 16, 0),
             ("dense", 2000, 20, 16, 1), ("dense", 2000, 200, 16, 0), ("bits", 2000, 300, 16, 0),
             ("values", 1000, 300, 16, 0)]


def _elementwise():
    import torch
    x = torch.zeros(1 << 22, device="cuda")         # thousands of workgroups

    def call():
        x.zero_()
        for _ in range(5):
            x.add_(1.0)
        torch.cuda.current_stream().synchronize()
        return [float(x[0]), float(x[-1])]
    return call


def _decision(kind, n, d, nq, prec):
    import torch
    from paper_1406_5161_amd import svmhip as S
    r = np.random.default_rng([n, d, nq])

    def make(m):
        if kind == "dense":
            return g.gen_blobs(m, d, r)
        x = g.gen_sparse_binary(m, d, 0.12, r)
        if kind == "values":
            x.val = (x.val * r.uniform(0.5, 1.5, len(x.val))).astype(np.float32)
        return x

    train, queries = S.to_device(make(n)), S.to_device(make(nq))
    alpha = torch.from_numpy(np.where(r.random(n) < 0.3, r.random(n), 0.0)).cuda()
    ws = torch.empty(S.svm_decision_workspace_size(train, queries, prec), dtype=torch.uint8, device="cuda")
    out = torch.zeros(nq, dtype=torch.float64, device="cuda")

    def call():
        assert S.svm_decision(train, alpha, 0.1, 0.5 / d, queries, out, prec, workspace=ws) == 0
        return out.cpu().tolist()
    return call


def main():
    import torch
    from paper_1406_5161_amd import svmhip as S
    for name, call in [("elementwise", _elementwise())] + [(repr(c), _decision(*c)) for c in DECISIONS]:
        ref = call()
        torch.cuda.synchronize()
        with S.Server(1 << 28, max_slots=4):
            time.sleep(0.05)                        # the loop holds its compute units
            t0 = time.perf_counter()
            got = call()
            dt = time.perf_counter() - t0
        print(json.dumps([name, dt, got == ref]), flush=True)


def test_calls_run_beside_the_loop():
    out = subprocess.check_output([sys.executable, "-u", "-m", "tests.test_gpu_server_beside"], text=True, cwd=ROOT,
                                  timeout=100)
    lines = [json.loads(x) for x in out.splitlines() if x.startswith("[")]
    print(lines)
    assert len(lines) == 1 + len(DECISIONS)
    for name, dt, same in lines:
        assert same and dt < 1.0, (name, dt, same)


@pytest.mark.parametrize("n", [16, 17, 4095, 4096, 4097, 8191, 8192, 8193])
def test_validation_around_its_workgroup_sizes(n):
    from tests import test_gpu_validate as v
    for layout in ("rows", "strided", "features"):
        v.test_dense(n, layout)
    v.test_csr(n)


if __name__ == "__main__":
    main()
