"""The context-free calls report their own failures, not an error that earlier HIP work of the thread left behind."""
import ctypes

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def leave_an_error():
    """An error that nobody has asked for: a device index no machine has (refused by the runtime on the host)."""
    with open("/proc/self/maps") as fh:
        path = next(line.split()[-1] for line in fh if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    assert hip.hipSetDevice(1 << 20) != 0
    assert hip.hipPeekAtLastError() != 0


def test_sample_after_a_stale_error():
    import torch
    import paper_2506_06122_amd as R
    z = torch.from_numpy(workloads.random_logits(5, 1000, seed=1, scale=2.0)).cuda()
    x = workloads.uniform_words(5, seed=2)
    want = R.rollout_sample(z, 1.0, 0.9, x)
    leave_an_error()
    got = R.rollout_sample(z, 1.0, 0.9, x)
    for a, b in zip(want, got):
        np.testing.assert_array_equal(a, b)


def test_policy_loss_after_a_stale_error():
    import torch
    import paper_2506_06122_amd as R
    old = -torch.rand(40, device="cuda")
    new, mask = old + 0.01, torch.ones(40, dtype=torch.uint8, device="cuda")
    args = ([0, 15, 40], new, old, None, mask, [1.0, -1.0])
    want = R.rollout_policy_loss(*args)
    torch.cuda.synchronize()
    leave_an_error()
    got = R.rollout_policy_loss(*args)
    assert got[0] == want[0] and torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])


def test_tile_product_after_a_stale_error():
    import torch
    from paper_2506_06122_amd import binding as B
    a, w = torch.ones(1, 1, 2, 32, dtype=torch.bfloat16, device="cuda"), torch.ones(16 * 32, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(16, device="cuda")
    torch.cuda.synchronize()
    leave_an_error()
    assert B.rollout_debug_tile_product(shape=0, epilogue=0, splits=1, m=1, n=16, k=32, a=a, w=w, out=out) == 1
    assert out.tolist() == [64.0] * 16
