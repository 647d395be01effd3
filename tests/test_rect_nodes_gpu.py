"""Whole-node kernel for grids of any shape (k_node_rect): every node shape and subsampling that a plan
reaches, source counts that do not fill a workgroup or the last group of eight, padded and
first-order plans, against the oracle and against the pass kernels of the same plan."""
import numpy as np
import pytest
import torch

import oracle
import paper_1812_11214_amd as scat

from parity import TOL, order_of_channels, per_order_errors

pytestmark = pytest.mark.gpu


def run(shape, J, L, max_order, padded, x, **kw):
    plan = scat.Scattering(shape, J, L, max_order, padded=padded, **kw)
    try:
        plan.timing_begin(None)
        y = plan.forward(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        return y.cpu().numpy(), set(plan.timing_end()), plan.coeff_index()
    finally:
        plan.close()


@pytest.mark.parametrize("shape,J,L,max_order,padded,batch", [
    ((128, 128), 3, 8, 2, False, 2),   # 64 x 64 and 32 x 32 nodes, octave 0 by k_node_half
    ((128, 128), 4, 3, 2, False, 1),   # 64, 32 and 16 a side, subsampling 8, 4 and 2
    ((64, 64), 2, 5, 2, False, 3),     # 15 first-order nodes: a last workgroup that is not full
    ((64, 64), 3, 1, 2, False, 9),     # one angle; more sources than a group of eight
    ((128, 64), 3, 3, 2, False, 3),    # tall nodes down to 32 x 16
    ((64, 128), 2, 4, 2, False, 1),    # wide nodes
    ((200, 120), 3, 4, 2, True, 2),    # padded to 256 x 128: 128 x 64 nodes
    ((120, 200), 3, 2, 2, True, 1),    # padded to 128 x 256: 64 x 128 nodes
    ((256, 128), 3, 2, 1, False, 2),   # first order only
    ((256, 256), 4, 2, 2, False, 1),   # octaves 0 and 1 on the passes, their grandchildren whole
])
def test_rect_nodes(shape, J, L, max_order, padded, batch):
    rng = np.random.default_rng(shape[0] * 1000 + shape[1] * 10 + J)
    x = rng.standard_normal((batch,) + shape).astype(np.float32)
    x[0] = np.cumsum(x[0], axis=0) * 0.1 + 3
    got, names, rows = run(shape, J, L, max_order, padded, x)
    assert any(n.startswith("k_node_rect<") for n in names), names
    want = (oracle.scattering2d_padded if padded else oracle.scattering2d)(x, J, L, max_order)
    errs = per_order_errors(got, want, order_of_channels(rows), x)
    print("rect", shape, J, L, errs, flush=True)
    assert max(errs.values()) <= TOL, errs
    old, names, _ = run(shape, J, L, max_order, padded, x, node_kernels=False)
    assert not any(n.startswith("k_node_rect<") for n in names), names
    # five chained transforms and two sums in fp32 on either side: 2 * 3e-6 of the order's maximum
    errs = per_order_errors(got, old, order_of_channels(rows), x)
    assert max(errs.values()) <= 6e-6, errs


# (rows, columns, subsampling) of the variants that each plan's octaves take: together all that a plan reaches
VARIANTS = [
    ((32, 32), 1, 4, 1, [(32, 32, 2)]),
    ((32, 64), 1, 3, 2, [(32, 64, 2)]),
    ((32, 64), 2, 5, 2, [(32, 64, 4), (16, 32, 2)]),
    ((32, 64), 3, 2, 1, [(32, 64, 8), (16, 32, 4)]),   # (8 x 16 nodes on the passes)
    ((64, 32), 1, 2, 2, [(64, 32, 2)]),
    ((64, 32), 2, 3, 2, [(64, 32, 4), (32, 16, 2)]),
    ((64, 64), 1, 7, 2, [(64, 64, 2)]),
    ((64, 64), 2, 3, 2, [(64, 64, 4), (32, 32, 2)]),
    ((64, 64), 3, 2, 2, [(64, 64, 8), (32, 32, 4), (16, 16, 2)]),
    ((64, 128), 1, 3, 1, [(64, 128, 2)]),
    ((64, 128), 2, 2, 2, [(64, 128, 4), (32, 64, 2)]),
    ((64, 128), 3, 2, 2, [(64, 128, 8), (32, 64, 4), (16, 32, 2)]),
    ((128, 64), 1, 2, 2, [(128, 64, 2)]),
    ((128, 64), 2, 1, 2, [(128, 64, 4), (64, 32, 2)]),
    ((128, 64), 3, 2, 2, [(128, 64, 8), (64, 32, 4), (32, 16, 2)]),
]


@pytest.mark.parametrize("shape,J,L,max_order,variants", VARIANTS)
def test_rect_node_variants(shape, J, L, max_order, variants):
    rng = np.random.default_rng(shape[0] * 100 + shape[1] + J)
    x = rng.standard_normal((3,) + shape).astype(np.float32)
    x[0] = np.cumsum(x[0], axis=0) * 0.1 + 3
    got, names, rows = run(shape, J, L, max_order, False, x)
    assert {n for n in names if n.startswith("k_node_rect<")} == {"k_node_rect<%d, %d, %d>" % v for v in variants}
    errs = per_order_errors(got, oracle.scattering2d(x, J, L, max_order), order_of_channels(rows), x)
    print("rect", shape, J, L, errs, flush=True)
    # what the fp32 chain of transforms shows elsewhere in this file: 3e-6 of an order's maximum
    assert max(errs.values()) <= 3e-6, errs


def test_all_variants_are_tested():
    assert len({v for case in VARIANTS for v in case[4]}) == 20


@pytest.mark.parametrize("shape,J,L,max_order,few,many", [
    ((128, 128), 4, 1, 1, 2, 300),
    ((128, 128), 4, 1, 2, 1, 150),
    ((128, 128), 4, 2, 2, 40, 41),    # two angles and second-order nodes: the passes up to 160 nodes
    ((128, 128), 4, 3, 1, None, 1),   # three: whole nodes at any batch
    ((256, 128), 4, 2, 1, 1, 80),
    ((128, 256), 3, 1, 1, 3, 520),
    ((128, 128), 4, 5, 1, None, 1),   # more angles: whole nodes at any batch
])
def test_few_nodes_of_few_angles_keep_the_passes(shape, J, L, max_order, few, many):
    """Calls that k_node_rect makes slower (few first-order nodes of few angles) run on the passes, larger
    ones of the same plan do not; the coefficients are the same."""
    rng = np.random.default_rng(shape[1] + 7 * J + L)
    x = rng.standard_normal((many,) + shape).astype(np.float32)
    got, names, rows = run(shape, J, L, max_order, False, x)
    assert any(n.startswith("k_node_rect<") for n in names), names
    n = min(few or 1, 2)
    want = oracle.scattering2d(x[:n], J, L, max_order)
    errs = per_order_errors(got[:n], want, order_of_channels(rows), x[:n])
    assert max(errs.values()) <= TOL, errs
    if few is None:
        return
    got, names, rows = run(shape, J, L, max_order, False, x[:few])
    assert not any(n.startswith("k_node_rect<") for n in names), names
    errs = per_order_errors(got[:n], want, order_of_channels(rows), x[:n])
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("shape,J,L", [
    ((64, 64), 3, 5),     # 16 x 16 leaves, four nodes to a wavefront
    ((64, 64), 3, 6),
    ((128, 64), 3, 3),    # 32 x 16 leaves, two to a wavefront
    ((64, 128), 3, 5),    # 16 x 32 leaves
])
def test_a_plane_has_the_same_bits_wherever_it_stands(shape, J, L):
    """Nodes of fewer than 64 threads share a wavefront with other planes' nodes, with other filters at
    another place in the batch."""
    x = torch.from_numpy(np.random.default_rng(J + L).standard_normal((7,) + shape).astype(np.float32)).cuda()
    plan = scat.Scattering(shape, J, L)
    try:
        y = plan.forward(x)
        for k in range(len(x)):
            assert torch.equal(plan.forward(x[k:k + 1].contiguous())[0], y[k]), k
    finally:
        plan.close()


def test_oversampled_plans_keep_the_passes():
    x = np.random.default_rng(1).standard_normal((1, 64, 64)).astype(np.float32)
    got, names, rows = run((64, 64), 3, 3, 2, False, x, oversampling=1)
    assert not any(n.startswith("k_node_rect<") for n in names), names
    want = oracle.scattering2d(x, 3, 3, 2, oversampling=1)
    errs = per_order_errors(got, want, order_of_channels(rows), x)
    assert max(errs.values()) <= TOL, errs


def test_special_values():
    x = np.zeros((4, 128, 64), dtype=np.float32)
    x[0] = -2.5
    x[1, 3, 50] = 1.0
    x[2] = np.random.default_rng(2).standard_normal((128, 64)) * 1e4
    x[3, 0, 0] = np.inf
    got, _, rows = run((128, 64), 3, 4, 2, False, x)
    want = oracle.scattering2d(x[:3], 3, 4)
    errs = per_order_errors(got[:3], want, order_of_channels(rows), x[:3])
    assert max(errs.values()) <= TOL, errs
    assert np.isnan(got[3]).all()
