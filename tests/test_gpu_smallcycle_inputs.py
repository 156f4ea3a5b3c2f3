"""Right-hand-side words that no row uses (Dirichlet velocity sites) in the
one-workgroup V-cycle kernels: whatever a caller left there, not-a-number
included, the result is bit for bit that of zeros.  Every top size, both
precisions, with and without a viscosity, in a V-cycle and in an FMG solve."""
import numpy as np
import pytest

from oracle import mesh
from paper_2010_13513_amd import hhg, workloads as W
from tests.gpu_util import Lib

pytestmark = pytest.mark.gpu

P1, P2 = hhg.HHG_P1P1, hhg.HHG_P2P1
NU = W.gaussian_bump_viscosity(W.SEED_BASE + 4000, N_ref=32)


def _dirichlet(disc, L):
    """Mask of the Dirichlet velocity words in lattice order."""
    m = (2 ** L if disc == P1 else 2 ** (L + 1)) + 1
    edge = np.ones((m, m, m), bool)
    edge[1:-1, 1:-1, 1:-1] = False
    return np.concatenate([np.broadcast_to(edge, (3, m, m, m)).reshape(-1), np.zeros((2 ** L + 1) ** 3, bool)])


@pytest.mark.parametrize("varnu", [False, True])
@pytest.mark.parametrize("disc,lmin,L", [(P1, 0, 1), (P1, 0, 2), (P1, 0, 3), (P1, 1, 3), (P2, 1, 2)])
def test_dirichlet_right_hand_side_is_not_used(disc, lmin, L, varnu):
    rng = np.random.default_rng(13513 + 10 * L + lmin)
    lib = Lib(disc, lmin, L)
    try:
        if varnu:
            for l in range(lmin, L + 1):
                c = mesh.p1_coords(2 ** l) / float(2 ** l)
                hhg.hhg_set_viscosity(lib.h, l, lib.torch.from_numpy(NU(c[:, 0], c[:, 1], c[:, 2])).to(lib.dev))
        prm = hhg.solver_params(1, 2, 1, 1, hhg.HHG_GS_FWD, 2, 2.3)
        lw = {l: lib.layout(l)[3] for l in range(lmin, L + 1)}
        x, bs = rng.standard_normal(lw[L]), {l: rng.standard_normal(lw[l]) for l in lw}
        for solve, prec in (("cycle", hhg.HHG_F64), ("cycle", hhg.HHG_F32), ("fmg", hhg.HHG_F64)):
            out = []
            for word in (0.0, np.nan, -np.inf):
                bd = [lib.from_lattice(l, np.where(_dirichlet(disc, l), word, bs[l]), prec) for l in sorted(bs)]
                xd = lib.from_lattice(L, x, prec)
                if solve == "fmg":
                    hhg.hhg_fmg_solve(lib.h, xd, bd, prm, want_stats=False)
                else:
                    hhg.hhg_vcycle(lib.h, L, xd, bd[-1], prm, prec)
                out.append(lib.to_lattice(L, xd, prec))
            assert np.isfinite(out[0]).all()
            differ = [int((o != out[0]).sum()) for o in out[1:]]
            assert differ == [0, 0], (solve, prec, differ)
    finally:
        lib.close()
