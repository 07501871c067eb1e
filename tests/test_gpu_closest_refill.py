"""Closest-point projection of caller's points: a lane keeps the nodal values of
the cell it evaluates in across its points, and a wave takes new points once
enough of its lanes are idle.  A point's result may depend on neither, so
scattered points give the same bits (tolerance 0) in another order and in calls
of another size: below and above a wave, around the refill threshold, and more
points than the kernel has lanes (every lane then takes several)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpu_util import dev, say

pytestmark = pytest.mark.gpu

vpp = pytest.importorskip("paper_2401_07805_amd")


@pytest.mark.parametrize("use_normal", [False, True])
@pytest.mark.parametrize("k,n", [(2, 8), (3, 5), (4, 4)])
def test_result_of_a_point_depends_on_no_other(k, n, use_normal):
    eps = 0.08
    m = W.unit_cube(n, k, 1000.0, 1.0, bc=(1,) * 6)
    phi = W.droplet_phi(m, 0.3, eps, centre=(0.48, 0.51, 0.5))
    prob = vpp.Problem.from_mesh(m)
    prob.set_phi(dev(phi))
    normal = None
    if use_normal:
        c = oracle.node_coords(m, np.arange(m.ndofs))
        normal = [dev(np.ascontiguousarray(0.48 + 0.01 * d - c[:, d])) for d in range(3)]
    total = 256 * 256 + 4097
    pts = np.random.default_rng(k).uniform(0.1, 0.9, size=(total, 3))
    pts[1] = np.nan

    def run(idx):
        say("closest points", k, use_normal, len(idx))
        y, info = prob.closest_points(eps, pts=dev(np.ascontiguousarray(pts[idx])), max_iter=8, normal=normal)
        return y.view(torch.int64).cpu().numpy(), info.cpu().numpy()

    y, info = run(np.arange(total))
    assert (info > 0).any()
    perm = np.random.default_rng(9).permutation(total)
    yp, ip = run(perm)
    assert np.array_equal(ip, info[perm]) and np.array_equal(yp, y[perm])
    for count in (1, 2, 15, 17, 63, 65, 1000):
        sub = perm[:count]
        ys, isub = run(sub)
        assert np.array_equal(isub, info[sub]) and np.array_equal(ys, y[sub])


@pytest.mark.parametrize("use_normal", [False, True])
@pytest.mark.parametrize("k,n", [(2, 8), (3, 5), (4, 4)])
def test_lanes_that_take_several_points(k, n, use_normal):
    """Four points for every lane the device has (a workgroup of 256 per CU) and some
    more, sorted by cell, so that a lane's next points often lie in the cell it keeps:
    the bits of calls so small that every lane takes one point, and of the same
    points in scattered order."""
    eps = 0.08
    m = W.unit_cube(n, k, 1000.0, 1.0, bc=(1,) * 6)
    prob = vpp.Problem.from_mesh(m)
    prob.set_phi(dev(W.droplet_phi(m, 0.3, eps, centre=(0.48, 0.51, 0.5))))
    normal = None
    if use_normal:
        c = oracle.node_coords(m, np.arange(m.ndofs))
        normal = [dev(np.ascontiguousarray(0.48 + 0.01 * d - c[:, d])) for d in range(3)]
    lanes = 256 * torch.cuda.get_device_properties(0).multi_processor_count
    total = 4 * lanes + 4097
    pts = np.random.default_rng(20 + k).uniform(0.1, 0.9, size=(total, 3))
    cell = np.minimum((pts * n).astype(int), n - 1) @ np.array([1, n, n * n])
    pts = pts[np.argsort(cell, kind="stable")]

    def run(idx):
        say("closest points, sorted", k, use_normal, len(idx))
        y, info = prob.closest_points(eps, pts=dev(np.ascontiguousarray(pts[idx])), max_iter=8, normal=normal)
        return y.view(torch.int64).cpu().numpy(), info.cpu().numpy()

    y, info = run(np.arange(total))
    assert (info > 0).any()
    perm = np.random.default_rng(9).permutation(total)
    yp, ip = run(perm)
    assert np.array_equal(ip, info[perm]) and np.array_equal(yp, y[perm])
    for first in (0, total // 2, total - lanes // 2):
        sub = np.arange(first, first + lanes // 2)
        ys, isub = run(sub)
        assert np.array_equal(isub, info[sub]) and np.array_equal(ys, y[sub])
