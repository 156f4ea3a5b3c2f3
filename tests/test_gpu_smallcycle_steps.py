"""Smoothing steps below zero in the one-workgroup V-cycle kernels: a level
with a negative count (fewer steps on the coarser levels, a negative
increment) takes none, as in the launch-per-phase form, and its residual is
still formed."""
import numpy as np
import pytest

from paper_2010_13513_amd import hhg
from tests.gpu_util import Lib, block_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pre,post,inc", [(-1, 2, 0), (1, 2, -1), (2, 1, -3)])
@pytest.mark.parametrize("disc,lmin,L", [(hhg.HHG_P1P1, 0, 3), (hhg.HHG_P2P1, 1, 2)])
def test_negative_steps_are_none(disc, lmin, L, pre, post, inc):
    rng = np.random.default_rng(13513 + L)
    lib = Lib(disc, lmin, L)
    try:
        lw = lib.layout(L)[3]
        x, b = rng.standard_normal(lw), rng.standard_normal(lw)
        prm = hhg.solver_params(pre, post, inc, 1, hhg.HHG_GS_FWD, 2, 2.3)
        out = []
        for sites in (0, 800):
            hhg.hhg_hier_set_fused_sites(lib.h, sites)
            xd, bd = lib.from_lattice(L, x), lib.from_lattice(L, b)
            hhg.hhg_vcycle(lib.h, L, xd, bd, prm, hhg.HHG_F64)
            out.append(lib.to_lattice(L, xd))
        # the bound of the same kernels' comparison with any other number of steps
        eu, ep = block_errors(lib, L, out[1], out[0])
        assert eu <= 1e-11 and ep <= 1e-11, (eu, ep)
    finally:
        lib.close()
