"""Refined-mesh solver on its packed vector: residuals on identity rows, initial
guesses, faces without Dirichlet conditions, and cell counts around the groups
of its cells kernel (84 cells a workgroup at k = 2, 64 at k = 3, 48 at k = 4).
Bars: apply 1e-12 against the oracle's matrix; solves against the sparse direct
solution to 1e-8, and the iteration count of the oracle's PCG on the whole
system (identity rows included) +- 2."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla

import oracle.amr as amr
import workloads as W
from gpu_util import dev, host, rel, say

pytestmark = pytest.mark.gpu

vpp = pytest.importorskip("paper_2401_07805_amd")


def problem(nc, k, mask, bc):
    m = W.Mesh(ncells=nc, degree=k, bc=bc, rho_l=1000.0, rho_g=1.0)
    m.eps = 0.1
    x, y, z = amr.node_coords(m)
    phi = np.tanh((0.3 - np.sqrt((x - .5) ** 2 + (y - .5) ** 2 + (z - .5) ** 2)) / (2 * m.eps))
    p = vpp.AmrProblem(m.ncells, m.degree, mask, m.origin, m.extent, m.bc, m.rho_l, m.rho_g)
    p.set_phi(dev(phi))
    return p, amr.operator(m, mask, phi)[0]


# active cells: below, at and above a workgroup's, single cells, all refined, none refined
@pytest.mark.parametrize("k,nc,nref", [(2, (1, 1, 1), 0), (2, (1, 1, 1), 1), (2, (7, 4, 3), 0), (2, (7, 3, 2), 6),
                                       (2, (7, 4, 3), 1), (3, (4, 4, 4), 0), (3, (4, 2, 1), 8), (3, (5, 4, 3), 1),
                                       (4, (4, 4, 3), 0), (4, (3, 2, 1), 6), (4, (4, 3, 3), 2)])
def test_apply_cell_groups(k, nc, nref):
    mask = np.zeros(int(np.prod(nc)), dtype=np.uint8)
    mask[np.random.default_rng(3).permutation(mask.size)[:nref]] = 1
    p, A = problem(nc, k, mask, (0, 1, 1, 0, 1, 1))
    x = np.random.default_rng(4).uniform(-1, 1, p.n)
    say("amr groups", k, nc, nref)
    assert rel(host(p.apply(dev(x))), A @ x) < 1e-12


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("identity", [0.0, 1.0, 30.0])
def test_solve_with_identity_rows(k, identity):
    nc = (4, 3, 3)
    mask = np.zeros(36, dtype=np.uint8)
    mask[[0, 13, 14, 22]] = 1
    p, A = problem(nc, k, mask, (0, 0, 0, 1, 0, 0))
    rng = np.random.default_rng(5)
    d = A.diagonal()
    ident = (abs(A).sum(axis=1).A1 == 1.0) & (d == 1.0) if hasattr(abs(A).sum(axis=1), "A1") else \
        (np.asarray(abs(A).sum(axis=1)).ravel() == 1.0) & (d == 1.0)
    assert ident.sum() == p.n - p.nfree
    b = np.where(ident, identity, 1.0) * rng.uniform(-1, 1, p.n)
    x0 = rng.uniform(-1, 1, p.n)
    if identity == 0.0:
        x0[ident] = 0.0
    ref = spla.spsolve(A.tocsc(), b)
    say("amr identity rows", k, identity)
    x, info = p.cg_solve(dev(b), x0=dev(x0), rtol=1e-12)
    x = host(x)
    r0 = np.linalg.norm(b - A @ x0)
    assert info["status"] == 0 and rel(x, ref) < 1e-8
    assert np.linalg.norm(b - A @ x) < 1e-11 * r0
    assert abs(info["true_rel_residual"] - np.linalg.norm(b - A @ x) / r0) < 1e-13
    assert np.abs(x[ident] - b[ident]).max() <= 1e-11 * r0
    # the recurrence of the whole system: zero initial guess, the oracle's count
    _, it = amr.pcg(A, b, rtol=1e-10)
    _, i0 = p.cg_solve(dev(b), rtol=1e-10)
    assert abs(i0["iterations"] - it) <= 2


@pytest.mark.parametrize("k,nc,most", [(2, (16, 14, 15), 1000), (3, (9, 8, 10), 1200)])
def test_attained_residual(k, nc, most):
    """The constrained values of the search direction follow their own recurrence for
    the whole solve.  Run far past convergence, it leaves no more than rounding: the
    residual of the returned solution within 64 units of 2^-53 (a row's products)
    and the known solution within 1e-13."""
    mask = np.zeros(int(np.prod(nc)), dtype=np.uint8)
    c = [(np.arange(n) + 0.5) / n for n in nc]
    z, y, x = np.meshgrid(c[2], c[1], c[0], indexing="ij")
    mask[np.abs(np.sqrt((x - .5) ** 2 + (y - .5) ** 2 + (z - .5) ** 2) - 0.3).ravel() < 0.15] = 1
    m = W.Mesh(ncells=nc, degree=k, bc=(0,) * 6, rho_l=1000.0, rho_g=1.0)
    m.eps = 0.1
    g = amr.node_coords(m)
    p = vpp.AmrProblem(m.ncells, m.degree, mask, m.origin, m.extent, m.bc, m.rho_l, m.rho_g)
    p.set_phi(dev(np.tanh((0.3 - np.sqrt(sum((a - .5) ** 2 for a in g))) / (2 * m.eps))))
    xs = np.random.default_rng(6).uniform(-1, 1, p.n)
    b = p.apply(dev(xs))
    say("amr attained", k, nc, p.n, p.nfree)
    u, info = p.cg_solve(b, rtol=1e-200, max_iter=most, raise_on_failure=False)
    say("amr attained", info)
    assert info["true_rel_residual"] < 64 * 2.0 ** -53
    assert rel(host(u), xs) < 1e-13
