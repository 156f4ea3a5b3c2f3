"""Smoothing calls of unstructured meshes on node tables (one workgroup, or
one per velocity component) against the launch-per-colour form: same updates
in the same order, row sums in another order.  Meshes with few and many
cells, outflow faces, one level per kernel form, colours of one and of
several passes; forward and symmetric, one and several sweeps."""
import numpy as np
import pytest

from oracle import smoother as osm, umesh
from oracle.stokes import Stokes
from paper_2010_13513_amd import hhg, workloads as W
from tests.gpu_util import Lib, assert_blocks, block_errors

pytestmark = pytest.mark.gpu

ORACLE = {}
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


TET = np.array([[0.0, 0.0, 0.0], [1.0, 0.1, 0.0], [0.9, 1.1, 0.05], [1.05, 0.95, 1.2]])
CELLS = {"one": (TET, np.array([[0, 1, 2, 3]])),
         "two": (np.vstack([TET, [[0.1, 1.2, 1.1]]]), np.array([[0, 1, 2, 3], [0, 2, 3, 4]]))}


@pytest.mark.parametrize("gs,xi,iters", [("f", 2, 1), ("s", 1, 2), ("s", 3, 1)])
@pytest.mark.parametrize("name,L", [("one", 2), ("one", 3), ("two", 2), ("two", 3), ("two", 4), ("two", 5)])
def test_cell_interiors_match_oracle(name, L, gs, xi, iters):
    """The interior colours of a cell in one launch (cells of up to 32
    intervals), against the oracle's pointwise sweeps: the smallest cell with
    interior points to the largest, with no interface (three symmetric sweeps
    are more steps than a launch takes) and with one."""
    key = (name, L)
    if key not in ORACLE:
        ORACLE[key] = Stokes(umesh.ULevel(*CELLS[name], L))
    S = ORACLE[key]
    U = osm.Uzawa(S, "sd")
    lib = Lib(hhg.HHG_P1P1, L - 1, L, mesh=CELLS[name])
    try:
        hhg.hhg_hier_set_fused_sites(lib.h, 0)
        rng = np.random.default_rng(L)
        x, b = rng.standard_normal(S.n), rng.standard_normal(S.n)
        xd, bd = lib.from_lattice(L, x), lib.from_lattice(L, b)
        hhg.hhg_smooth(lib.h, L, xd, bd, iters, hhg.HHG_GS_FWD if gs == "f" else hhg.HHG_GS_SYM, xi, 2.0)
        want = x
        for _ in range(iters):
            want = U.iterate(want, b, gs, xi, 0.5)
        assert_blocks(lib, L, lib.to_lattice(L, xd), want, 1e-12, f"{name} {gs}{xi}")
    finally:
        lib.close()
