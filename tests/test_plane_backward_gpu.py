"""Whole-node backward kernels of 2-D plans (k_plane_nodes): every node shape, node counts that do not
fill a workgroup, padded, oversampled and first-order plans, against the oracle in 64 bits and against
the pass kernels of the same plan."""
import numpy as np
import pytest
import torch

import oracle
import paper_1812_11214_amd as scat

pytestmark = pytest.mark.gpu


def run(shape, J, L, max_order, x, g, padded, o, **kw):
    plan = scat.Scattering(shape, J, L, max_order, padded=padded, oversampling=o, **kw)
    try:
        gd = torch.from_numpy(g((plan.K,) + plan.out_shape)).cuda()
        plan.timing_begin(None)
        gi = plan.backward(torch.from_numpy(x).cuda(), gd)
        torch.cuda.synchronize()
        return gi.cpu().numpy(), set(plan.timing_end()), gd.cpu().numpy()
    finally:
        plan.close()


def rel(a, b):
    return np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b)


@pytest.mark.parametrize("shape,J,L,max_order,padded,o,batch", [
    ((32, 32), 1, 8, 2, False, 0, 3),    # a last workgroup that is not full (at J = 2 it is a tree's)
    ((32, 32), 2, 3, 2, False, 1, 5),    # oversampled, so no tree: octaves of one size
    ((64, 64), 3, 3, 2, False, 0, 2),    # 64, 32 and 16 a side
    ((64, 128), 3, 2, 2, False, 0, 1),   # wide
    ((128, 64), 2, 1, 2, False, 0, 5),   # tall; one angle
    ((128, 128), 3, 4, 2, False, 0, 1),  # octave 0 fills a compute unit
    ((128, 128), 4, 2, 2, False, 0, 2),
    ((64, 32), 2, 5, 1, False, 0, 2),    # first order only
    ((32, 64), 1, 4, 2, False, 0, 2),    # no children
    ((64, 64), 3, 2, 2, False, 2, 2),    # oversampled: octaves of one size
    ((28, 27), 1, 8, 2, True, 0, 3),     # padded to 32 x 32
    ((50, 33), 2, 3, 2, True, 0, 2),
])
def test_plane_backward(shape, J, L, max_order, padded, o, batch):
    rng = np.random.default_rng(shape[0] * 1000 + shape[1] * 10 + J + o)
    x = rng.standard_normal((batch,) + shape).astype(np.float32)
    seed = int(rng.integers(1 << 30))

    def g(per):
        return np.random.default_rng(seed).standard_normal((batch,) + per).astype(np.float32)

    print("plane", shape, J, L, max_order, padded, o, flush=True)
    got, names, gg = run(shape, J, L, max_order, x, g, padded, o)
    n1, n2 = ((1 << (n + 2 ** J - 1).bit_length()) for n in shape) if padded else shape
    sides = {(n1 >> max(j - o, 0), n2 >> max(j - o, 0)) for j in range(J)}
    assert {s for s in names if s.startswith("k_plane_nodes<") and s.endswith(", true>")} == {
        "k_plane_nodes<%d, %d, true>" % s for s in sides}, names
    assert {"k_plane_end<%d, %d, true>" % (n1, n2), "k_plane_end<%d, %d, false>" % (n1, n2), "k_plane_sum"} <= names
    old, names, _ = run(shape, J, L, max_order, x, g, padded, o, node_kernels=False)
    assert not any(s.startswith("k_plane_") for s in names), names
    if padded:
        want = oracle.scattering2d_padded_backward(x.astype(np.float64), gg.astype(np.float64), J, L, max_order)
    else:
        want = oracle.scattering2d_backward(x.astype(np.float64), gg.astype(np.float64), J, L, max_order,
                                            oversampling=o)
    for p in range(batch):
        new, before = rel(got[p], want[p]), rel(old[p], want[p])
        mid, mid_before = median(got[p], want[p]), median(old[p], want[p])
        print(p, new, before, mid, mid_before, flush=True)
        # Through y / |y| the rounding of y (3e-7 of its r.m.s.) becomes a phase error of 3e-7 / rho at a
        # sample of rho r.m.s.; of N samples of noise one has rho < N^-1/2 / 10 in a hundred planes, which
        # alone moves the gradient by 3e-6 in relative L2 (in either schedule, by its own rounding: no
        # bound on their ratio).  So the L2 bar is 1e-5, and the median over the pixels, which such a
        # sample does not reach, is held to the rounding of nine chained transforms.
        assert new <= 1e-5 and before <= 1e-5, (p, new, before)
        assert mid <= max(3e-7, 1.5 * mid_before), (p, mid, mid_before)


def median(a, b):
    return np.median(np.abs(a.astype(np.float64) - b)) / np.sqrt(np.mean(b ** 2))


@pytest.mark.parametrize("shape,J,few,many", [((128, 128), 4, 2, 130), ((64, 128), 3, 128, 129), ((128, 128), 1, 1, 3)])
def test_few_nodes_of_one_angle_keep_the_passes(shape, J, few, many):
    """Calls that the whole-node kernels make slower run on the passes, larger ones of the same plan
    do not; neither allocates after scat_plan_reserve for the larger one."""
    rng = np.random.default_rng(shape[0] + J)
    plan = scat.Scattering(shape, J, 1, 2)
    try:
        plan.reserve(many, with_backward=True)
        x = rng.standard_normal((many,) + shape).astype(np.float32)
        g = rng.standard_normal((many, plan.K) + plan.out_shape).astype(np.float32)
        xd, gd = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
        out = torch.empty_like(xd)
        free = torch.cuda.mem_get_info()[0]
        want = oracle.scattering2d_backward(x[:1].astype(np.float64), g[:1].astype(np.float64), J, 1)
        for n, whole in ((few, False), (many, True)):
            plan.timing_begin(None)
            plan.backward(xd[:n], gd[:n], out[:n])
            torch.cuda.synchronize()
            names = set(plan.timing_end())
            assert any(s.startswith("k_plane_nodes<") for s in names) == whole, names
            assert rel(out[:1].cpu().numpy(), want) <= 1e-5   # (the bar of test_plane_backward)
        assert torch.cuda.mem_get_info()[0] == free
    finally:
        plan.close()


def test_special_values():
    """A plane of zeros (no gradient through any modulus), a constant, large noise and an infinity."""
    shape, J, L = (64, 32), 2, 3
    rng = np.random.default_rng(3)
    x = np.zeros((4,) + shape, dtype=np.float32)
    x[1] = -2.5
    x[2] = rng.standard_normal(shape) * 1e4
    x[3, 0, 0] = np.inf
    got, names, g = run(shape, J, L, 2, x, lambda per: rng.standard_normal((4,) + per).astype(np.float32), False, 0)
    assert any(s.startswith("k_plane_nodes<") for s in names), names
    want = oracle.scattering2d_backward(x[:3].astype(np.float64), g[:3].astype(np.float64), J, L)
    assert rel(got[0], want[0]) <= 1e-6          # the lowpass of x alone: two transforms of 2048 points
    assert np.isfinite(got[1]).all()             # (its moduli vanish up to rounding, which decides their phases)
    assert rel(got[2], want[2]) <= 1e-5          # (the bar of test_plane_backward)
    assert np.isnan(got[3]).all()


def test_grids_out_of_range_keep_the_passes():
    for shape, J in (((32, 32), 3), ((256, 128), 2), ((128, 32), 2)):
        plan = scat.Scattering(shape, J, 2, 2)
        try:
            x = torch.randn((1,) + shape, device="cuda")
            g = torch.randn((1, plan.K) + plan.out_shape, device="cuda")
            plan.timing_begin(None)
            plan.backward(x, g)
            torch.cuda.synchronize()
            assert not any(s.startswith("k_plane_") for s in plan.timing_end())
        finally:
            plan.close()
