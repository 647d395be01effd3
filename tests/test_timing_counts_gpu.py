"""Model flops that the per-kernel timer states for the whole-node kernels of the backward pass: 5 n
log2 n per n-point complex transform (half of that for a real signal), 4 per filter multiply-accumulate
and modulus, counted here from the plan's own filter bank."""
import numpy as np
import pytest
import torch

import paper_1812_11214_amd as scat

pytestmark = pytest.mark.gpu


def backward_rows(plan, batch):
    x = torch.randn((batch,) + plan.shape, device="cuda")
    g = torch.randn((batch, plan.K) + plan.out_shape, device="cuda")
    plan.timing_begin(None)
    plan.backward(x, g)
    torch.cuda.synchronize()
    return plan.timing_end()


def listed(plan, wavelets):
    """(block of 256 frequencies, wavelet) pairs on which the wavelet exceeds 1e-8 of its peak."""
    n = 0
    for k in range(wavelets):
        v = np.abs(plan.filter(1, k, 0)).ravel()
        size = min(256, v.size)
        n += int((v.reshape(-1, size).max(axis=1) > 1e-8 * v.max()).sum()) * size
    return n


@pytest.mark.parametrize("shape", [(16, 16), (32, 64), (128, 128)])
def test_plane_kernels(shape):
    L, batch = 3, 4
    plan = scat.Scattering(shape, 1, L, 1)
    try:
        rows = backward_rows(plan, batch)
        n = shape[0] * shape[1]
        lg = np.log2(n)
        node = rows["k_plane_nodes<%d, %d, true>" % shape]
        assert node["launches"] == 1
        # three transforms, filter product, modulus, lowpass
        assert node["model_flops"] == batch * L * n * (15 * lg + 12)
        assert rows["k_plane_end<%d, %d, true>" % shape]["model_flops"] == batch * n * 2.5 * lg
        assert rows["k_plane_end<%d, %d, false>" % shape]["model_flops"] == batch * n * 5 * lg
        assert rows["k_plane_sum"]["model_flops"] == batch * 4 * (n + listed(plan, L))
    finally:
        plan.close()


@pytest.mark.parametrize("n,J,Q", [(64, 1, 2), (1024, 3, 4)])
def test_line_sum(n, J, Q):
    batch = 3
    plan = scat.Scattering((n,), J, Q, 1)
    try:
        rows = backward_rows(plan, batch)
        assert rows["k_line_sum"]["model_flops"] == batch * 4 * (n + listed(plan, J * Q))
        nodes = rows["k_line_nodes<true, false>"]["model_flops"]
        want = sum(batch * Q * (n >> j) * (15 * np.log2(n >> j) + 4 * 2 ** j + 8) for j in range(J))
        assert nodes == want
    finally:
        plan.close()
