"""Node tables of unstructured levels on meshes far from a cube: a fan of
cells around one edge (rows of hundreds of entries at its nodes, 15 to 24
elsewhere) and levels without a free node."""
import numpy as np
import pytest

from paper_2010_13513_amd import hhg
from tests.gpu_util import Lib, block_errors, torch_cuda

pytestmark = pytest.mark.gpu


def fan(cells):
    """`cells` tetrahedra around the edge (0, 0, 0) - (0, 0, 1)."""
    a = 2 * np.pi * np.arange(cells) / cells
    xyz = np.vstack([[[0, 0, 0], [0, 0, 1]], np.stack([np.cos(a), np.sin(a), np.full(cells, 0.5)], 1)])
    ring = 2 + np.arange(cells)
    return xyz, np.stack([0 * ring, 0 * ring + 1, ring, np.roll(ring, -1)], 1)


def beam(cubes):
    """A row of unit cubes of six tetrahedra each."""
    xyz = np.array([[i, j, k] for i in range(cubes + 1) for j in (0, 1) for k in (0, 1)], float)
    steps = [(4, 2, 1), (4, 1, 2), (2, 4, 1), (2, 1, 4), (1, 4, 2), (1, 2, 4)]
    return xyz, np.array([np.cumsum((4 * c, *s)) for c in range(cubes) for s in steps])


def _smooth_both(lib, L, gs, xi, iters):
    rng = np.random.default_rng(13513 + L)
    x, b = (rng.standard_normal(lib.layout(L)[3]) for _ in range(2))
    bd, out = lib.from_lattice(L, b), []
    for slots in (0, 30000):
        hhg.hhg_hier_set_fused_sites(lib.h, slots)
        xd = lib.from_lattice(L, x)
        hhg.hhg_smooth(lib.h, L, xd, bd, iters, gs, xi, 2.69)
        out.append(lib.to_lattice(L, xd))
    return x, out


@pytest.mark.parametrize("gs,xi,iters", [(hhg.HHG_GS_FWD, 2, 2), (hhg.HHG_GS_SYM, 1, 2)])
@pytest.mark.parametrize("cells,L", [(5, 2), (40, 1), (40, 3), (200, 2)])
def test_smoothing_on_a_fan(cells, L, gs, xi, iters):
    lib = Lib(hhg.HHG_P1P1, L - 1, L, mesh=fan(cells))
    try:
        _, (want, got) = _smooth_both(lib, L, gs, xi, iters)
        # rows of up to about 800 entries, carried over at most 4 sweeps: under 4000 roundings
        eu, ep = block_errors(lib, L, got, want)
        assert eu <= 1e-12 and ep <= 1e-12, (eu, ep)
    finally:
        lib.close()


def test_tables_hold_the_rows_that_are_there():
    """150 cells around an edge at levels 2 and 3: 21014 nodes, all but the
    fourteen on the edge with 15 to 24 entries.  An entry takes 66 bytes, so
    the tables are below 21014 x 24 x 66 bytes = 34 MB; the other arrays of the
    hierarchy are below 26 MB, and each of at most 100 allocations may take 2 MB
    more than its size.  Rows of the longest one's length: 440 MB."""
    torch = torch_cuda()
    torch.cuda.synchronize()
    first = torch.cuda.mem_get_info()[0]
    lib = Lib(hhg.HHG_P1P1, 2, 3, mesh=fan(150))
    try:
        torch.cuda.synchronize()
        used = first - torch.cuda.mem_get_info()[0]
        print(f"[tables] {used / 1e6:.1f} MB", flush=True)
        assert used <= 260e6
    finally:
        lib.close()


def test_level_without_free_nodes():
    """A row of 190 cubes at level 0: 764 nodes, all of them on the boundary."""
    lib = Lib(hhg.HHG_P1P1, 0, 1, mesh=beam(190))
    try:
        x, (want, got) = _smooth_both(lib, 0, hhg.HHG_GS_SYM, 2, 2)
        nv = lib.layout(0)[3] * 3 // 4
        assert np.array_equal(want[:nv], x[:nv]) and np.array_equal(got[:nv], x[:nv])
        eu, ep = block_errors(lib, 0, got, want)
        assert eu == 0.0 and ep <= 1e-12, (eu, ep)
    finally:
        lib.close()
