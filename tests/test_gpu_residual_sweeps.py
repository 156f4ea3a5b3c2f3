"""Sweeps of several colours per launch on lattices that the oracle does not
reach in the time of a test: P1 with a varying viscosity on 16 x 8 x 8 boxes at
N = 64 (against the oracle's pointwise sweeps; runs of two to four colours in
float32, of one and two in float64), and from there on against the same sweeps
done colour by colour from residuals of the whole level and the operator's
diagonal (the apply kernels have their own parity tests)."""
import pytest

from paper_2010_13513_amd import hhg
from tests.gpu_util import Lib
from tests.test_gpu_boxes import FWD, NU, P1, P2, SYM, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gs,xi,iters", [(FWD, 3, 1), (FWD, 2, 1), (FWD, 1, 2), (SYM, 1, 1), (SYM, 2, 2)])
def test_viscosity_on_boxes_matches_oracle(gs, xi, iters):
    _check(P1, 6, gs, xi, iters, True)


def _diagonal(lib, L, G, n1, ijk, varnu):
    """A's diagonal per group and node.  Rows couple nodes one step apart per
    axis, so a class of nodes mod 3 shows its own diagonal; with constant
    coefficients one node of a group does."""
    torch, vw = lib.torch, lib.layout(L)[2]
    e, y = (torch.zeros(vw, dtype=torch.float64, device=lib.dev) for _ in range(2))
    diag = torch.ones(G, n1, n1, n1, dtype=torch.float64, device=lib.dev)
    u, Au = (v[:G * n1 ** 3].view(G, n1, n1, n1) for v in (e, y))
    if not varnu:
        mid = (n1 // 2,) * 3
        for g in range(G):
            u.zero_()
            u[(g, *mid)] = 1.0
            hhg.hhg_apply(lib.h, L, hhg.HHG_OP_A, e, y)
            diag[g] = Au[(g, *mid)]
        return diag
    for c in range(27):
        at = (ijk[0] % 3 == c % 3) & (ijk[1] % 3 == c // 3 % 3) & (ijk[2] % 3 == c // 9)
        u[0] = at
        hhg.hhg_apply(lib.h, L, hhg.HHG_OP_A, e, y)
        diag[0] = torch.where(at & (Au[0] != 0), Au[0], diag[0])         # Dirichlet rows are zero
    return diag


@pytest.mark.parametrize("gs,xi", [(FWD, 3), (FWD, 2), (FWD, 1), (SYM, 2)])
@pytest.mark.parametrize("disc,L,varnu", [(P1, 7, True), (P1, 7, False), (P2, 6, False), (P2, 7, False)])
def test_matches_residual_sweeps(disc, L, varnu, gs, xi):
    n1, G = 2 ** L + 1, 1 if disc == P1 else 8
    lib = Lib(disc, L - 1, L)
    torch = lib.torch
    try:
        k, j, i = torch.meshgrid(*(torch.arange(n1, device=lib.dev),) * 3, indexing="ij")
        if varnu:
            pts = [(c.double() / (n1 - 1)).reshape(-1).cpu().numpy() for c in (i, j, k)]
            hhg.hhg_set_viscosity(lib.h, L, torch.from_numpy(NU(*pts)).to(lib.dev))
        diag = _diagonal(lib, L, G, n1, (i, j, k), varnu)
        lw, nv = lib.layout(L)[3], 3 * G * n1 ** 3
        gen = torch.Generator(device=lib.dev).manual_seed(13513 + xi)
        x, b = (lib.empty(L) for _ in range(2))
        for v in (x, b):
            hhg.hhg_vec_from_lattice(lib.h, L, torch.randn(lw, generator=gen, dtype=torch.float64, device=lib.dev), v)
        want, r = x.clone(), torch.empty_like(x)
        u, ru = (v[:nv].view(3, G, n1, n1, n1) for v in (want, r))
        odd = (i + j + k) % 2
        forward = list(range(2 if G == 1 else 9))
        for c in (forward if gs == FWD else forward + forward[::-1]) * xi:
            hhg.hhg_residual(lib.h, L, want, b, r)
            g = max(c - 1, 0)
            step = ru[:, g] / diag[g]
            u[:, g] += torch.where(odd == c, step, 0.0) if c < 2 else step
        for prec, dt, tol in ((hhg.HHG_F64, torch.float64, 1e-12), (hhg.HHG_F32, torch.float32, 500 * 2.0 ** -24)):
            got = x.to(dt, copy=True)
            hhg.hhg_smooth(lib.h, L, got, b.to(dt), 1, gs, xi, 2.3, prec)
            err = float((got[:nv].double() - want[:nv]).abs().max() / want[:nv].abs().max())
            print(f"[parity] disc {disc} level {L} {gs} xi {xi} {dt}: velocity {err:.2e} (tol {tol:.0e})", flush=True)
            assert err <= tol
    finally:
        lib.close()
