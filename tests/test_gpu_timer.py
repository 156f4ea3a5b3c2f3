"""The kernel timer's families and work units of smoothing calls: sites that
the call's launches update, a colour that a symmetric sweep takes once counted
once; P1 has vertex colours only.  One lattice per kernel form."""
import pytest

from paper_2010_13513_amd import hhg
from tests.gpu_util import Lib

pytestmark = pytest.mark.gpu

P1, P2 = hhg.HHG_P1P1, hhg.HHG_P2P1


def _units(disc, L, gs):
    lib = Lib(disc, L - 1, L)
    try:
        x, b = lib.empty(L), lib.empty(L)
        fams = (hhg.KF_GS_VERTEX, hhg.KF_GS_EDGE)
        hhg.hhg_timer_start(sum(1 << f for f in fams))
        hhg.hhg_smooth(lib.h, L, x, b, 2, gs, 1, 2.3)
        out = [hhg.hhg_timer_read(f) for f in fams]
        hhg.hhg_timer_start(0)
        return out
    finally:
        lib.close()


@pytest.mark.parametrize("L", [1, 3, 5, 6, 7])
def test_p1_sites(L):
    m = 2 ** L - 1                                        # odd: the colours hold (m^3 -+ 1) / 2 sites
    first, second = (m ** 3 - 1) // 2, (m ** 3 + 1) // 2
    for gs, want in ((hhg.HHG_GS_FWD, first + second), (hhg.HHG_GS_SYM, 2 * first + second)):
        (ms, launches, units), (_, none, _) = _units(P1, L, gs)
        assert units == 2 * want and none == 0 and launches >= 2 and ms > 0.0


@pytest.mark.parametrize("L", [2, 3, 4, 5, 6, 7])
def test_p2_sites(L):
    m = 2 ** (L + 1) - 1
    N = 2 ** L
    for gs in (hhg.HHG_GS_FWD, hhg.HHG_GS_SYM):
        per = _units(P2, L, gs)
        # the last colour is the edges of direction (1, 1, 1), N^3 of them;
        # the runs take it twice at a turn, the other forms once
        once = m ** 3 if gs == hhg.HHG_GS_FWD else 2 * m ** 3 - N ** 3
        twice = m ** 3 if gs == hhg.HHG_GS_FWD else 2 * m ** 3
        runs = L >= 4
        assert sum(u for _, _, u in per) == 2 * (twice if runs else once)
        assert all(ms > 0.0 for ms, n, _ in per if n)
