"""Tile edges of the plane-per-thread kernels (apply variant 1 and the
reinitialization operator) and of the default configurations: meshes one cell
below, at and one above each instantiated tile, and one with several tiles per
direction, against the FP64 oracle.  Bars as elsewhere: FP64 1e-12, FP32 2e-6
(relative 2-norm)."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu

vpp = pytest.importorskip("paper_2401_07805_amd")


def edge_boxes(tile):
    t = np.array(tile)
    return [tuple(int(v) for v in b) for b in (np.maximum(t - 1, 1), t, t + 1, np.minimum(2 * t + 1, (9, 9, 9)))]


@pytest.mark.parametrize("k", [2, 3, 4])
def test_plane_apply_tile_edges(k):
    cfgs = [c for c in vpp.config_candidates(k) if c["variant"] == 1]
    assert cfgs
    for cfg in cfgs:
        for nc in edge_boxes(cfg["tile"]):
            m = W.Mesh(ncells=nc, degree=k, bc=(0, 1, 1, 0, 0, 1), extent=(1.0, 0.8, 1.1), rho_l=1000.0, rho_g=1.0)
            phi = W.droplet_phi(m, 0.3, 0.1)
            x = W.uniform_vectors(5, 1, m.ndofs)[0]
            yref = oracle.Operator(m, phi=phi).matvec(x)
            p = vpp.Problem.from_mesh(m)
            p.set_phi(dev(phi))
            p.set_config(cfg["variant"], cfg["tile"])
            say("plane apply", k, cfg, nc)
            assert rel(host(p.apply(dev(x))), yref) < 1e-12, (cfg, nc)
            y32 = host(p.apply(dev(x).float()).double())
            assert rel(y32, yref) < 2e-6, (cfg, nc)


# around the tiles 8x4x2 (k = 2), 4x4x2 and 4x4x4 (k = 3), 4x3x2 (k = 4)
@pytest.mark.parametrize("k,ncells", [(2, (1, 1, 1)), (2, (7, 3, 1)), (2, (8, 4, 2)), (2, (9, 5, 3)), (2, (17, 9, 5)),
                                      (3, (1, 1, 1)), (3, (4, 4, 2)), (3, (5, 5, 3)), (3, (3, 9, 5)),
                                      (4, (1, 1, 1)), (4, (4, 3, 2)), (4, (5, 4, 3)), (4, (3, 2, 5))])
def test_reinit_apply_tile_edges(k, ncells):
    m = W.Mesh(ncells=ncells, degree=k, bc=(0,) * 6, extent=(1.0, 0.9, 1.2))
    normal = W.normal_field(m, (0.47, 0.52, 0.5))
    x = W.uniform_vectors(6, 1, m.ndofs)[0]
    ref = oracle.reinit_matrix(m, normal, 0.08, 0.05) @ x
    p = vpp.Problem.from_mesh(m)
    say("reinit apply", k, ncells)
    assert rel(host(p.reinit_apply(dev(x), [dev(c) for c in normal], 0.08, 0.05)), ref) < 1e-12


def test_reinit_apply_large_k3_tile():
    """The k = 3 tile of meshes above 50,000 cells: sampled rows."""
    m = W.Mesh(ncells=(41, 37, 34), degree=3, bc=(0,) * 6)
    normal = W.normal_field(m, (0.47, 0.52, 0.5))
    x = W.uniform_vectors(7, 1, m.ndofs)[0]
    rows = np.random.default_rng(3).choice(m.ndofs, 60, replace=False)
    ax, _, _ = oracle.reinit_rows(m, normal, 0.05, 0.04, x, x, rows)
    p = vpp.Problem.from_mesh(m)
    say("reinit apply 41x37x34 Q3")
    y = host(p.reinit_apply(dev(x), [dev(c) for c in normal], 0.05, 0.04))
    assert np.abs(y[rows] - ax).max() < 1e-12 * np.abs(ax).max()


@pytest.mark.parametrize("k,ncells", [(2, (28, 27, 26)), (2, (28, 27, 27)), (3, (25, 26, 24)), (3, (26, 25, 25)),
                                      (4, (20, 20, 20)), (4, (20, 21, 20))])
def test_default_configuration_rule(k, ncells):
    """Both sides of the rule's lines: the default gives the tuner's candidates' result."""
    m = W.Mesh(ncells=ncells, degree=k, bc=(0, 1, 1, 0, 0, 1), rho_l=1000.0, rho_g=1.0)
    phi = W.droplet_phi(m, 0.3, 0.1)
    x = dev(W.uniform_vectors(8, 1, m.ndofs)[0])
    p = vpp.Problem.from_mesh(m)
    p.set_phi(dev(phi))
    say("default", k, ncells, p.config_for("fp64"), p.config_for("fp32"))
    y, y32 = host(p.apply(x)), host(p.apply(x.float()).double())
    other = [c for c in vpp.config_candidates(k) if c["variant"] == 1 and c != p.config_for("fp64")]
    other = other or [c for c in vpp.config_candidates(k) if c != p.config_for("fp64")]
    p.set_config(other[0]["variant"], other[0]["tile"])
    ref = host(p.apply(x))
    assert rel(y, ref) < 1e-12 and rel(y32, ref) < 2e-6


@pytest.mark.parametrize("k,ncells", [(2, (34, 34, 34)), (2, (35, 35, 33)), (3, (21, 14, 9)),
                                      (4, (20, 20, 20)), (4, (21, 20, 20))])
def test_default_configuration_with_the_mass_shift(k, ncells):
    """The configuration chosen by mesh size once the mass shift is set, on both
    sides of the line, against every other one with the shift (1e-12: FP64
    rounding of sums of at most 8 (k+1)^3 terms, with room)."""
    m = W.Mesh(ncells=ncells, degree=k, bc=(1,) * 6, rho_l=1000.0, rho_g=1.0, mass=1.5)
    m.eps = 0.1
    prob = vpp.Problem.from_mesh(m)
    prob.set_phi(dev(W.droplet_phi(m, 0.3, m.eps, centre=(0.45, 0.5, 0.55))))
    prob.set_mass(1.5)
    x = dev(W.uniform_vectors(5, 1, m.ndofs)[0])
    y, y32 = prob.apply(x), prob.apply(x.float())
    count = 0
    for cfg in vpp.config_candidates(k):
        try:
            prob.set_config(cfg["variant"], cfg["tile"])
        except vpp.VppError:
            continue
        count += 1
        z, z32 = prob.apply(x), prob.apply(x.float())
        assert float((z - y).norm() / y.norm()) < 1e-12, cfg
        assert float((z32 - y32).norm() / y32.norm()) < 2e-6, cfg
    assert count >= 2


def _thin(k, ncells):
    h = 1.0 / max(ncells)
    return W.Mesh(ncells=ncells, degree=k, bc=(0, 1, 1, 0, 0, 1), extent=tuple(h * n for n in ncells), rho_l=1000.0,
                  rho_g=1.0)


# thin boxes, whose defaults go by the extent: in FP64 4x4x2, 4x2x2, 2x2x2 and 4x4x1,
# in FP32 8x8x4 (k = 2) and 4x3x2 (k = 4)
@pytest.mark.parametrize("k,ncells,tile", [(2, (1, 231, 230), (8, 8, 4)), (3, (141, 139, 1), (4, 4, 2)),
                                           (3, (151, 1, 149), (4, 2, 2)), (4, (1, 101, 99), (2, 2, 2)),
                                           (4, (101, 99, 1), (4, 4, 1))])
def test_default_config_of_thin_boxes(k, ncells, tile):
    m = _thin(k, ncells)
    phi = W.uniform_vectors(3, 1, m.ndofs)[0]
    x = W.uniform_vectors(5, 1, m.ndofs)[0]
    rows = np.random.default_rng(1).choice(m.ndofs, 2000, replace=False)
    ref = oracle.apply_rows(m, phi, x, rows)
    p = vpp.Problem.from_mesh(m)
    p.set_phi(dev(phi))
    say("thin box", k, ncells, p.config_for("fp64"), p.config_for("fp32"))
    assert p.config_for("fp64")["tile"] == tile
    assert rel(host(p.apply(dev(x)))[rows], ref) < 1e-12
    assert rel(host(p.apply(dev(x).float()).double())[rows], ref) < 2e-6


# thin boxes on which the reinitialization operator runs one cell per thread
@pytest.mark.parametrize("k,ncells", [(2, (1, 201, 199)), (3, (1, 1, 20001))])
def test_reinit_of_thin_boxes(k, ncells):
    m = _thin(k, ncells)
    normal = W.normal_field(m, (0.3 * m.extent[0], 0.47 * m.extent[1], 0.52 * m.extent[2]))
    h = m.extent[2] / ncells[2]
    x = W.uniform_vectors(7, 1, m.ndofs)[0]
    rows = np.random.default_rng(2).choice(m.ndofs, 2000, replace=False)
    ax, _, rb = oracle.reinit_rows(m, normal, 2 * h, 2 * h, x, x, rows)
    p = vpp.Problem.from_mesh(m)
    nd = [dev(c) for c in normal]
    say("thin reinit", k, ncells)
    assert rel(host(p.reinit_apply(dev(x), nd, 2 * h, 2 * h))[rows], ax) < 1e-12
    new, info = p.reinit_step(dev(x), nd, 2 * h, 2 * h)
    say("thin reinit step", info)
    assert info["status"] == 0 and info["true_rel_residual"] < 1.01e-12
    assert rel(host(p.reinit_apply(new, nd, 2 * h, 2 * h))[rows], rb) < 1e-9


# k = 2 defaults change from the plane to the cell kernels with the mesh's size: in
# FP32 the planes' error relative to FP64 is, over meshes and laws, no larger than
# the cells' (both round each factor once, so single meshes differ by chance only)
def test_plane_f32_error_not_above_the_cell_kernels():
    ratio = []
    for nc in [(8, 8, 8), (13, 11, 9), (16, 12, 10), (20, 20, 20), (24, 24, 24), (32, 32, 32)]:
        for law in (0, 1):
            for rho_l in (1000.0, 10.0):
                m = W.Mesh(ncells=nc, degree=2, bc=(0, 0, 0, 0, 0, 0), extent=tuple(n / max(nc) for n in nc), rho_l=rho_l,
                           rho_g=1.0, heaviside=law)
                p = vpp.Problem.from_mesh(m)
                p.set_phi(dev(W.droplet_phi(m, 0.3, 4.0 / max(nc))))
                x = [dev(W.uniform_vectors(s, 1, m.ndofs)[0]).float() for s in (11, 12, 13)]
                err = []
                for cfg in [(1, (8, 4, 2)), (4, (8, 8, 4))]:
                    p.set_config(*cfg, "fp32")
                    err.append(np.mean([rel(host(p.apply(v).double()), host(p.apply(v.double()))) for v in x]))
                ratio.append(err[0] / err[1])
    say("FP32 error, planes over cells", float(np.mean(ratio)), max(ratio))
    assert np.mean(ratio) <= 1.0


# Q3 boxes that 8x4x4 would leave CUs idle on: 4x4x2, 4x4x4 and 4x2x2
@pytest.mark.parametrize("ncells,tile", [((24, 88, 8), (4, 4, 2)), ((33, 30, 28), (4, 4, 4)), ((33, 26, 34), (4, 2, 2))])
def test_default_config_by_rounds(ncells, tile):
    m = _thin(3, ncells)
    phi = W.uniform_vectors(3, 1, m.ndofs)[0]
    x = W.uniform_vectors(5, 1, m.ndofs)[0]
    rows = np.random.default_rng(1).choice(m.ndofs, 2000, replace=False)
    ref = oracle.apply_rows(m, phi, x, rows)
    p = vpp.Problem.from_mesh(m)
    p.set_phi(dev(phi))
    say("rounds", ncells, p.config_for("fp64"), p.config_for("fp32"))
    assert p.config_for("fp64")["tile"] == p.config_for("fp32")["tile"] == tile
    assert rel(host(p.apply(dev(x)))[rows], ref) < 1e-12
    assert rel(host(p.apply(dev(x).float()).double())[rows], ref) < 2e-6
