"""Whole-node kernels of the 1-D cascade (k_line_nodes): every length they are built for, node counts
that do not fill a workgroup or the last group of eight, padded, oversampled and first-order plans,
forward and backward, against the oracle and against the pass kernels of the same plan."""
import numpy as np
import pytest
import torch

import oracle
import paper_1812_11214_amd as scat

from parity import TOL, order_of_channels, per_order_errors

pytestmark = pytest.mark.gpu


def run(n, J, Q, max_order, x, g, padded=False, o=0, **kw):
    plan = scat.Scattering((n,), J, Q, max_order, padded=padded, oversampling=o, **kw)
    try:
        plan.timing_begin(None)
        xd = torch.from_numpy(x).cuda()
        y = plan.forward(xd)
        gi = plan.backward(xd, torch.from_numpy(g(plan)).cuda())
        torch.cuda.synchronize()
        return y.cpu().numpy(), gi.cpu().numpy(), set(plan.timing_end()), plan.coeff_index(), g(plan)
    finally:
        plan.close()


@pytest.mark.parametrize("n,J,Q,max_order,padded,o,batch", [
    (8192, 5, 8, 2, False, 0, 3),   # 8192 (two workgroups a compute unit) ... 512 samples
    (8192, 8, 1, 2, False, 1, 2),   # 28 pairs of octaves in one launch, 64 alias blocks
    (8192, 7, 1, 2, False, 0, 2),
    (4096, 7, 4, 2, False, 0, 2),   # 4096 ... 64
    (2048, 4, 12, 2, False, 0, 1),  # 2048 ... 256
    (64, 2, 3, 2, False, 0, 5),     # the smallest nodes and outputs: 32 and 16 samples
    (256, 1, 5, 2, False, 0, 3),    # no children
    (1024, 5, 2, 1, False, 0, 17),  # first order only; a last workgroup that is not full
    (1024, 4, 2, 2, False, 2, 2),   # several octaves of one length, output grid 256
    (512, 3, 2, 2, False, 5, 2),    # nothing subsampled: output grid as long as the nodes
    (5000, 5, 8, 2, True, 0, 2),    # odd tails of input and output
    (1501, 4, 3, 2, True, 0, 1),
    (113, 3, 2, 2, True, 0, 4),
    (33, 2, 4, 2, True, 1, 3),
])
def test_line_nodes(n, J, Q, max_order, padded, o, batch):
    rng = np.random.default_rng(n * 100 + 10 * J + Q + o)
    x = rng.standard_normal((batch, n)).astype(np.float32)
    x[0] = np.cumsum(x[0]) * 0.1 + 3
    seed = int(rng.integers(1 << 30))

    def g(plan):
        return np.random.default_rng(seed).standard_normal((batch, plan.K) + plan.out_shape).astype(np.float32)

    print("line", n, J, Q, max_order, padded, o, batch, flush=True)
    got, grad, names, rows, g_of = run(n, J, Q, max_order, x, g, padded, o)
    assert any(s.startswith("k_line_nodes<false") for s in names), names
    assert any(s.startswith("k_line_nodes<true") for s in names), names
    kw = {} if padded else {"oversampling": o}  # (the oracle's padded transforms are not oversampled)
    x64 = x.astype(np.float64)
    if not (padded and o):
        want = (oracle.scattering1d_padded if padded else oracle.scattering1d)(x, J, Q, max_order, **kw)
        errs = per_order_errors(got, want, order_of_channels(rows), x)
        print("oracle", errs, flush=True)
        assert max(errs.values()) <= TOL, errs
    old, grad_old, names, _, _ = run(n, J, Q, max_order, x, g, padded, o, node_kernels=False)
    assert not any(s.startswith("k_line_") for s in names), names
    if not (padded and o):
        # (order 2 of a random walk is 1e-4 of the signal and carries its rounding, in either schedule)
        errs_old = per_order_errors(old, want, order_of_channels(rows), x)
        print("passes", errs_old, flush=True)
        assert max(errs_old.values()) <= TOL, errs_old
        assert all(errs[k] <= max(3e-6, 1.5 * errs_old[k]) for k in errs), (errs, errs_old)
    else:
        errs = per_order_errors(got, old, order_of_channels(rows), x)
        assert max(errs.values()) <= 6e-6, errs  # 3e-6 on either side
    # Gradients pass through y / |y|: the rounding of x's spectrum (1e-7 of its norm) over |y| is the
    # error of that phase, so a random walk, whose |y| at octave 0 is a hundredth of its norm, has
    # 1e-5 in fp32 whatever the schedule; each side is held against 64 bits, and to 1e-6 on noise.
    if padded and o:
        for p in range(1, batch):
            assert rel(grad[p], grad_old[p]) <= 2e-6, p
        return
    back = oracle.scattering1d_padded_backward if padded else oracle.scattering1d_backward
    want = back(x64, g_of.astype(np.float64), J, Q, max_order, **kw)
    for p in range(batch):
        new, before = rel(grad[p], want[p]), rel(grad_old[p], want[p])
        print("gradient", p, new, before, flush=True)
        # (a random walk's 1e-5, see above, with a factor of ten: the passes have a bar of their own)
        assert before <= 1e-4, (p, before)
        assert new <= max(1e-6, 2 * before), (p, new, before)


def rel(a, b):
    return np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b)


def test_special_values():
    n, J, Q = 2048, 4, 3
    x = np.zeros((4, n), dtype=np.float32)
    x[0] = -2.5
    x[1, 77] = 1.0
    x[2] = np.random.default_rng(2).standard_normal(n) * 1e4
    x[3, 0] = np.inf
    got, grad, _, rows, _ = run(n, J, Q, 2, x, lambda p: np.ones((4, p.K) + p.out_shape, dtype=np.float32))
    want = oracle.scattering1d(x[:3], J, Q)
    errs = per_order_errors(got[:3], want, order_of_channels(rows), x[:3])
    assert max(errs.values()) <= TOL, errs
    assert np.isnan(got[3]).all()
    assert np.isfinite(grad[:3]).all()


def test_lengths_out_of_range_keep_the_passes():
    x = np.random.default_rng(1).standard_normal((1, 16384)).astype(np.float32)
    plan = scat.Scattering((16384,), 5, 2, 2)
    try:
        plan.timing_begin(None)
        plan.forward(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        assert not any(s.startswith("k_line_") for s in plan.timing_end())
    finally:
        plan.close()
