"""The one-workgroup V-cycle kernels specialised on the top level's lattice
size against the launch-per-phase form (same arithmetic, sums in another
order): every top size, every depth of the coarsest level, both precisions,
a viscosity on no, every
or only the finest level, forward and symmetric sweeps, no pre-smoothing,
more smoothing below."""
import numpy as np
import pytest

from oracle import mesh
from paper_2010_13513_amd import hhg, workloads as W
from tests.gpu_util import Lib, block_errors

pytestmark = pytest.mark.gpu

P1, P2 = hhg.HHG_P1P1, hhg.HHG_P2P1
NU = W.gaussian_bump_viscosity(W.SEED_BASE + 4000, N_ref=32)


@pytest.mark.parametrize("gs,xi,pre,post,inc", [(hhg.HHG_GS_FWD, 3, 0, 2, 1), (hhg.HHG_GS_SYM, 1, 2, 0, 0)])
@pytest.mark.parametrize("disc,lmin,L", [(P1, 0, 1), (P1, 0, 2), (P1, 0, 3), (P1, 1, 2), (P1, 1, 3), (P1, 2, 3),
                                         (P2, 1, 2)])
@pytest.mark.parametrize("nu_levels", ["none", "all", "finest"])
def test_small_cycle_matches_phases(disc, lmin, L, gs, xi, pre, post, inc, nu_levels):
    rng = np.random.default_rng(13513 + 10 * L + lmin)
    lib = Lib(disc, lmin, L)
    try:
        for l in {"none": [], "all": range(lmin, L + 1), "finest": [L]}[nu_levels]:
            c = mesh.p1_coords(2 ** l) / float(2 ** l)
            hhg.hhg_set_viscosity(lib.h, l, lib.torch.from_numpy(NU(c[:, 0], c[:, 1], c[:, 2])).to(lib.dev))
        _, _, _, lw = lib.layout(L)
        x, b = rng.standard_normal(lw), rng.standard_normal(lw)
        prm = hhg.solver_params(pre, post, inc, 1, gs, xi, 2.3)
        for prec, tol in ((hhg.HHG_F64, 1e-11), (hhg.HHG_F32, 1000 * 2.0 ** -24)):
            out = []
            for sites in (0, 800):
                hhg.hhg_hier_set_fused_sites(lib.h, sites)
                xd, bd = lib.from_lattice(L, x, prec), lib.from_lattice(L, b, prec)
                hhg.hhg_vcycle(lib.h, L, xd, bd, prm, prec)
                out.append(lib.to_lattice(L, xd, prec))
            eu, ep = block_errors(lib, L, out[1], out[0])
            assert eu <= tol and ep <= tol, (prec, eu, ep)
    finally:
        lib.close()
