"""Gauss-Seidel sweeps that run several colours per launch on boxes of the
lattice in LDS (whole small levels, overlapped tiles on the middle levels):
the smoother against the oracle's pointwise multicolour sweeps at every size
with its own tiling, in both precisions, constant and variable viscosity, forward and
symmetric, with an odd and an even number of sweeps (the tiles alternate
between two buffers)."""
import numpy as np
import pytest

from oracle import fe, mesh
from oracle.smoother import Uzawa
from oracle.stokes import Stokes
from paper_2010_13513_amd import hhg, workloads as W
from tests.gpu_util import Lib, assert_blocks

pytestmark = pytest.mark.gpu

P1, P2 = hhg.HHG_P1P1, hhg.HHG_P2P1
_ORACLE = {}


NU = W.gaussian_bump_viscosity(W.SEED_BASE + 4000, N_ref=32)


def _nu(N):
    c = mesh.p1_coords(N) / float(N)
    return NU(c[:, 0], c[:, 1], c[:, 2])


def _oracle(vorder, N, varnu):
    if (vorder, N, varnu) not in _ORACLE:
        _ORACLE[vorder, N, varnu] = Uzawa(Stokes(fe.Level(N, vorder, _nu(N) if varnu else None)), "sd")
    return _ORACLE[vorder, N, varnu]


FWD, SYM = hhg.HHG_GS_FWD, hhg.HHG_GS_SYM


@pytest.mark.parametrize("gs,xi,iters", [(FWD, 3, 1), (FWD, 1, 2), (SYM, 1, 1)])
@pytest.mark.parametrize("disc,L", [(P1, 3), (P1, 4), (P2, 2), (P2, 3), (P2, 4), (P2, 5)])
@pytest.mark.parametrize("varnu", [False, True])
def test_smooth_boxes(disc, L, gs, xi, iters, varnu):
    _check(disc, L, gs, xi, iters, varnu)


# the P1 lattices whose sweeps are cut into runs: every length of run and both
# first colours (the pressure alternates between two buffers as well)
@pytest.mark.parametrize("gs,xi,iters", [(FWD, 3, 1), (FWD, 2, 1), (FWD, 1, 2), (SYM, 1, 1), (SYM, 2, 2)])
@pytest.mark.parametrize("L,varnu", [(5, False), (5, True), (6, False)])
def test_smooth_runs_p1(L, gs, xi, iters, varnu):
    _check(P1, L, gs, xi, iters, varnu)


# the lattices whose runs march along k (constant coefficients), against the
# variable-viscosity kernels with a viscosity of one (a launch per colour for
# Taylor-Hood, boxes for P1: checked against the oracle on smaller lattices);
# every word, boundary values and padding included
@pytest.mark.parametrize("gs,xi,iters", [(FWD, 3, 1), (FWD, 1, 2), (SYM, 1, 1)])
@pytest.mark.parametrize("disc,L,prec", [(P2, 6, hhg.HHG_F64), (P2, 7, hhg.HHG_F64), (P2, 7, hhg.HHG_F32),
                                         (P1, 7, hhg.HHG_F64), (P1, 7, hhg.HHG_F32), (P1, 8, hhg.HHG_F64),
                                         (P1, 8, hhg.HHG_F32)])
def test_smooth_runs_along_k(disc, L, prec, gs, xi, iters):
    out = []
    for varnu in (False, True):
        lib = Lib(disc, L - 1, L)
        torch = lib.torch
        try:
            if varnu:
                hhg.hhg_set_viscosity(lib.h, L, torch.ones((2 ** L + 1) ** 3, dtype=torch.float64, device=lib.dev))
            dt = torch.float64 if prec == hhg.HHG_F64 else torch.float32
            gen = torch.Generator(device=lib.dev).manual_seed(13513 + 10 * L + xi)
            x = torch.randn(lib.empty(L, dt).shape, generator=gen, dtype=dt, device=lib.dev)
            b = torch.randn(x.shape, generator=gen, dtype=dt, device=lib.dev)
            hhg.hhg_smooth(lib.h, L, x, b, iters, gs, xi, 2.3, prec)
            torch.cuda.synchronize()
            out.append(x)
            nv, np_ = lib.layout(L)[:2]
        finally:
            lib.close()
    got, want = out
    tol = 1e-12 if prec == hhg.HHG_F64 else 500 * 2.0 ** -24
    split = got.numel() - np_
    for part in (slice(0, split), slice(split, None)):
        assert float((got[part] - want[part]).abs().max()) <= tol * float(want[part].abs().max())


def _check(disc, L, gs, xi, iters, varnu):
    vorder = 1 if disc == P1 else 2
    U = _oracle(vorder, 2 ** L, varnu)
    n = U.S.n
    rng = np.random.default_rng(13513 + 100 * L + vorder)
    lib = Lib(disc, L - 1, L)
    try:
        if varnu:
            hhg.hhg_set_viscosity(lib.h, L, lib.torch.from_numpy(_nu(2 ** L)).to(lib.dev))
        for prec, rnd, tol in ((hhg.HHG_F64, lambda a: a, 1e-12),
                               (hhg.HHG_F32, lambda a: a.astype(np.float32).astype(float), 500 * 2.0 ** -24)):
            x, b = rnd(rng.standard_normal(n)), rnd(rng.standard_normal(n))
            xd, bd = lib.from_lattice(L, x, prec), lib.from_lattice(L, b, prec)
            hhg.hhg_smooth(lib.h, L, xd, bd, iters, gs, xi, 2.3, prec)
            want = x
            for _ in range(iters):
                want = U.iterate(want, b, "s" if gs == hhg.HHG_GS_SYM else "f", xi, 1.0 / 2.3)
            got = lib.to_lattice(L, xd, prec)
            assert_blocks(lib, L, got, want, tol, f"smooth boxes xi {xi} iters {iters}")
            assert np.array_equal(lib.to_lattice(L, bd, prec), b)
    finally:
        lib.close()
