"""3-D plans whose nodes go through the fused passes in lists: more nodes than one list takes,
lists cut short by the scratch at hand, one node or one volume per list, output grids that one
workgroup holds and larger ones, each forward and backward against the oracle."""
import numpy as np
import pytest

import paper_1812_11214_amd as scat
from oracle import harmonic3d as o3
from paper_1812_11214_amd import binding

from parity import TOL, order_of_channels, per_order_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,J,L,mo,o,batch", [
    ((16, 16, 16), 4, 6, 2, 0, 2),    # 28 first-order and 42 second-order nodes: two lists each
    ((16, 32, 16), 3, 0, 2, 0, 1),    # degree 0 only: every node one signal
    ((8, 16, 32), 2, 3, 1, 0, 3),     # no second order
    ((4, 64, 16), 1, 2, 2, 0, 5),     # one scale; two slabs of T beside the Nyquist one
    ((32, 64, 64), 1, 1, 2, 0, 1),    # output grid of 16 x 32 x 32: not held by one workgroup
    ((16, 16, 16), 2, 2, 2, 2, 2),    # full-resolution output of 16 x 16 x 16: held whole
])
def test_lists_forward_and_backward(shape, J, L, mo, o, batch):
    import torch
    rng = np.random.default_rng(sum(shape) * 7 + 10 * J + L)
    # positive fields: the degree-0 signals keep away from zero, where their sign (and the
    # gradient) would be decided by rounding
    x = (0.2 + rng.random((batch,) + shape)).astype(np.float32)
    plan = scat.Scattering(shape, J, L, mo, oversampling=o)
    try:
        xd = torch.from_numpy(x).cuda()
        y = plan.forward(xd)
        g = rng.standard_normal(tuple(y.shape)).astype(np.float32)
        gx = plan.backward(xd, torch.from_numpy(g).cuda())
        torch.cuda.synchronize()
        got, ggot = y.cpu().numpy(), gx.cpu().numpy().astype(np.float64)
        rows = plan.coeff_index()
    finally:
        plan.close()
    errs = per_order_errors(got, o3.harmonic_scattering3d(x, J, L, mo, oversampling=o),
                            order_of_channels(rows), x)
    assert max(errs.values()) <= TOL, errs
    want = o3.harmonic_scattering3d_backward(x, g, J, L, mo, oversampling=o)
    emax = np.abs(ggot - want).max() / np.abs(want).max()
    assert emax <= TOL, emax


def test_special_values():
    """A volume of zeros, a constant, large values and an infinity, each beside the others in one call."""
    import torch
    shape, J, L = (16, 32, 16), 2, 2
    rng = np.random.default_rng(11)
    x = np.zeros((4,) + shape, dtype=np.float32)
    x[1] = 2.5
    x[2] = (0.2 + rng.random(shape)) * 1e4
    x[3, 0, 0, 0] = np.inf
    plan = scat.Scattering(shape, J, L)
    try:
        xd = torch.from_numpy(x).cuda()
        y = plan.forward(xd)
        g = rng.standard_normal(tuple(y.shape)).astype(np.float32)
        gx = plan.backward(xd, torch.from_numpy(g).cuda())
        torch.cuda.synchronize()
        got, ggot = y.cpu().numpy(), gx.cpu().numpy().astype(np.float64)
        rows = plan.coeff_index()
    finally:
        plan.close()
    errs = per_order_errors(got[:3], o3.harmonic_scattering3d(x[:3], J, L), order_of_channels(rows), x[:3])
    assert max(errs.values()) <= TOL, errs
    assert (got[0] == 0).all() and np.isnan(got[3]).all()
    want = o3.harmonic_scattering3d_backward(x[:3], g[:3], J, L)
    for p in (0, 2):  # zeros: the lowpass of x alone
        assert np.abs(ggot[p] - want[p]).max() / np.abs(want[p]).max() <= TOL, p
    assert np.isfinite(ggot[1]).all()  # (moduli that vanish up to rounding, which decides their signs)
    assert np.isnan(ggot[3]).all()


def test_lists_cut_by_the_static_buffer():
    """64^3 at J = 3, L = 3 asks for more scratch than the library's static buffer has: the call
    takes fewer nodes at a time there and gives the same coefficients (bit for bit: a node's
    arithmetic does not depend on its list)."""
    import torch
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal((2, 64, 64, 64)).astype(np.float32)).cuda()
    plan = scat.Scattering((64, 64, 64), 3, 3)
    try:
        assert plan.workspace_bytes(1) > binding.SCAT_STATIC_SCRATCH_MB << 20
        ref = plan.forward(x)
        got = torch.full_like(ref, float("nan"))
        binding.scat_forward_static(plan._plan, x.data_ptr(), got.data_ptr(), 2,
                                    torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(ref, got)
    finally:
        plan.close()


def test_workspace_grows_with_the_batch():
    """scat_plan_reserve covers every smaller batch (host arithmetic only)."""
    for shape, J, L in (((64, 64, 64), 2, 3), ((32, 32, 32), 3, 2), ((16, 64, 64), 2, 8)):
        plan = scat.Scattering(shape, J, L, host_only=True)
        fw = [plan.workspace_bytes(b) for b in range(1, 40)]
        bw = [plan.backward_workspace_bytes(b) for b in range(1, 40)]
        plan.close()
        assert fw == sorted(fw) and bw == sorted(bw)
