"""Dirichlet values on the levels of an FMG solve: with f = 0 and the boundary
values of a linear divergence-free velocity the discrete solution of every
level is that velocity with zero pressure, so the solve reproduces it to
rounding, and a boundary value from a wrong node of the finest level on any
level shows as an error of the order of h.  Hierarchies whose intermediate
levels interpolate by sites and (65 nodes per edge and more) by cubes, one
and several refinements below the finest level."""
import numpy as np
import pytest

from paper_2010_13513_amd import hhg
from tests.gpu_util import Lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("disc,lmin,lmax", [(hhg.HHG_P1P1, 0, 1), (hhg.HHG_P1P1, 0, 4), (hhg.HHG_P1P1, 0, 7),
                                            (hhg.HHG_P2P1, 1, 2), (hhg.HHG_P2P1, 1, 4), (hhg.HHG_P2P1, 1, 7)])
def test_linear_velocity_is_reproduced(disc, lmin, lmax):
    N = 2 ** lmax
    m = (N if disc == hhg.HHG_P1P1 else 2 * N) + 1
    lib = Lib(disc, lmin, lmax)
    try:
        k, j, i = np.meshgrid(*(np.arange(m) / (m - 1),) * 3, indexing="ij")
        u = np.stack([j - 0.5 * k, k + 0.25 * i, i - j])     # divergence 0
        inner = np.zeros((m, m, m), bool)
        inner[1:-1, 1:-1, 1:-1] = True
        want = np.concatenate([u.reshape(-1), np.zeros((N + 1) ** 3)])
        start = np.concatenate([np.where(inner, 7.0, u).reshape(-1), np.full((N + 1) ** 3, 3.0)])
        x = lib.from_lattice(lmax, start)
        bs = [lib.empty(l) for l in range(lmin, lmax + 1)]
        xi = 1 if disc == hhg.HHG_P1P1 else 3
        hhg.hhg_fmg_solve(lib.h, x, bs, hhg.solver_params(1, 2, 0, 1, hhg.HHG_GS_FWD, xi, 2.34))
        got = lib.to_lattice(lmax, x)
        # residuals of eps |A| |u| summed over N levels of nodes: eps N^2, with room for the constants
        tol = 50 * 2.0 ** -52 * max(N, 16) ** 2
        nv = 3 * m ** 3
        assert np.abs(got[:nv] - want[:nv]).max() <= tol
        edge = ~np.broadcast_to(inner, (3, m, m, m)).reshape(-1)
        assert np.array_equal(got[:nv][edge], start[:nv][edge])
        assert np.abs(got[nv:]).max() <= tol * N
    finally:
        lib.close()
