"""Elementwise kernels of the caller run beside a live serving loop: they do not wait until it stops, which
it does after two seconds without work."""
import time

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own_stream", [False, True])
def test_elementwise_kernels_run_beside_the_loop(own_stream):
    import torch
    from paper_1406_5161_amd import svmhip as S
    x = torch.zeros(1 << 22, device="cuda")         # thousands of workgroups
    st = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    with torch.cuda.stream(st):
        x.add_(1.0)
    torch.cuda.synchronize()
    with S.Server(1 << 28, max_slots=4):
        time.sleep(0.05)                            # the loop holds its compute units
        t0 = time.perf_counter()
        with torch.cuda.stream(st):
            for _ in range(5):
                x.add_(1.0)
            st.synchronize()
        dt = time.perf_counter() - t0
    assert float(x.min()) == float(x.max()) == 6.0
    assert dt < 1.0
