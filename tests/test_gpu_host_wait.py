"""What a call does with the host core while it waits for the device."""
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_long_wait_gives_the_core_away():
    """A call that has to wait some 200 ms for work ahead of it on its stream uses less than half of a core
    meanwhile (the first 20 ms are polled without a pause: 10 %), and returns the same results."""
    import torch
    import paper_2506_06122_amd as R
    z = torch.from_numpy(workloads.random_logits(4, 5000, seed=1, scale=2.0)).cuda()
    x = workloads.uniform_words(4, seed=2)
    want = R.rollout_sample(z, 1.0, 0.9, x)
    stream = torch.cuda.Stream()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    cycles = 1_000_000
    with torch.cuda.stream(stream):
        torch.cuda._sleep(cycles)
        start.record()
        torch.cuda._sleep(cycles)
        end.record()
    stream.synchronize()
    cycles = int(cycles * 200.0 / start.elapsed_time(end))
    assert cycles < 10 ** 10
    with torch.cuda.stream(stream):
        torch.cuda._sleep(cycles)
    wall, cpu = time.perf_counter(), time.thread_time()
    got = R.rollout_sample(z, 1.0, 0.9, x, stream=stream.cuda_stream)
    wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
    print(f"waited {1e3 * wall:.1f} ms with {1e3 * cpu:.1f} ms of the core")
    assert wall > 0.05 and cpu < 0.5 * wall
    for a, b in zip(want, got):
        np.testing.assert_array_equal(a, b)
