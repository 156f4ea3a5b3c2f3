"""Smoothing calls of unstructured meshes on node tables (one workgroup, or
one per velocity component) against the launch-per-colour form: same updates
in the same order, row sums in another order.  Meshes with few and many
cells, outflow faces, one level per kernel form, colours of one and of
several passes; forward and symmetric, one and several sweeps."""
import numpy as np
import pytest

from paper_2010_13513_amd import hhg, workloads as W
from tests.gpu_util import Lib, block_errors

pytestmark = pytest.mark.gpu

MESHES = {"cube24": lambda: W.cube24(), "jittered": lambda: W.jittered_cube(W.SEED_BASE + 7),
          "box": lambda: W.box_cube24(2, 1, 1)}


@pytest.mark.parametrize("gs,xi,iters", [(hhg.HHG_GS_FWD, 2, 3), (hhg.HHG_GS_SYM, 1, 2)])
@pytest.mark.parametrize("name,L,outflow", [("cube24", 1, 0), ("cube24", 2, 2), ("cube24", 3, 0), ("cube24", 4, 0),
                                            ("jittered", 3, 0), ("box", 2, 0), ("box", 3, 0)])
def test_node_smoothing_matches_colour_launches(name, L, outflow, gs, xi, iters):
    lib = Lib(hhg.HHG_P1P1, L - 1, L, mesh=MESHES[name](), outflow=outflow)
    try:
        lw = lib.layout(L)[3]
        rng = np.random.default_rng(13513 + L)
        x, b = rng.standard_normal(lw), lib.from_lattice(L, rng.standard_normal(lw))
        out = []
        for slots in (0, 30000):
            hhg.hhg_hier_set_fused_sites(lib.h, slots)
            xd = lib.from_lattice(L, x)
            hhg.hhg_smooth(lib.h, L, xd, b, iters, gs, xi, 2.69)
            out.append(xd)
        # rows of at most about 64 entries, sums of products of order one
        # carried over at most 8 sweeps: a few hundred roundings
        eu, ep = block_errors(lib, L, lib.to_lattice(L, out[1]), lib.to_lattice(L, out[0]))
        assert eu <= 1e-12 and ep <= 1e-12, (eu, ep)
        # every copy of an interface node holds the node's value
        back = lib.from_lattice(L, lib.to_lattice(L, out[1]))
        assert bool((back == out[1]).all())
    finally:
        lib.close()
