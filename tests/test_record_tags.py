"""The 16-bit tags of the register loop's selection records: a reader never takes cleared words or a record
of another iteration for the one it waits for, wherever a launch starts."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1406_5161_amd import datagen as g

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "svm_internal.h"
#include <cstdio>
// one writer's two record places (by iteration parity); a launch at `start`, its places cleared or not
static int run(int64_t start, int64_t end, bool clear, unsigned (&slot)[2]) {
    if (clear) slot[0] = slot[1] = 0u;
    for (int64_t i = start; i < end; ++i) {
        const unsigned tag = svm::rec_tag(i);
        if (tag > 0xffffu) return 1;
        if (slot[i & 1] == tag) return 2;      // matches before it is written
        slot[i & 1] = tag;
    }
    return 0;
}
int main() {
    const int64_t wraps[] = {0, 32767, 32768, 65534, 65535, 65536, 131069, 131070, 131072, 1ll << 40};
    for (int64_t w : wraps)
        for (int64_t start = w > 4 ? w - 4 : 0; start < w + 4; ++start)
            for (int relaunch = 0; relaunch < 6; ++relaunch) {   // cleared, then continued some iterations on
                unsigned slot[2];
                int rc = run(start, start + relaunch, true, slot);
                if (!rc) rc = run(start + relaunch, start + relaunch + 140000, false, slot);
                if (rc) { std::printf("start %lld relaunch %d: %d\n", (long long)start, relaunch, rc); return 1; }
            }
    std::puts("ok");
    return 0;
}
"""


def test_no_cleared_or_old_word_matches(tmp_path):
    cxx = shutil.which("g++")
    src, exe = tmp_path / "tags.cpp", tmp_path / "tags"
    src.write_text(PROGRAM)
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_1406_5161_amd", "csrc"), "-o", str(exe), str(src)])
    assert subprocess.check_output([str(exe)], text=True).strip() == "ok"


@pytest.mark.gpu
def test_solve_beyond_the_wrap():
    """70,000 iterations on 11 workgroups: the loop that keeps rows elsewhere has 32-bit tags."""
    import torch
    from paper_1406_5161_amd import svmhip as S
    n, d, cap = 2600, 6, 70_000
    r = np.random.default_rng(5)
    data = g.gen_blobs(n, d, r)
    data.y[:] = r.permutation(data.y)
    dp = S.to_device(data)
    got = []
    for flags in (0, S.SVM_FLAG_NO_LDS_PAYLOAD):
        par = S.make_params(1000.0, 0.2, 1e-13, 0, 0, 0.0, cap, S.SVM_KERNEL_FP32, flags)
        a, f = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        rc, x = S.svm_train(dp, par, a, f)
        assert rc == S.SVM_NOT_CONVERGED and x.iterations == cap
        assert flags or x.grid_blocks > 1
        got.append((a, f))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
