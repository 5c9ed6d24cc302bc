"""The step rule and the overlap over more levels than the weights kept in LDS,
and the overlap of one point around the number of levels that a wave holds;
against the oracle."""
import numpy as np
import pytest

from oracle import schedule as S
from tests.paritylib import rel_ok

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,levels", [(64, 1023), (64, 1025), (64, 4096), (128, 4097), (128, 9000), (128, 16385)])
def test_wide_populations(L, levels):
    from paper_2401_07965_amd import pa
    R, N = 700, L * L
    rng = np.random.default_rng(levels)
    h = rng.integers(0, levels, R)
    h[0], h[-1] = 0, levels - 1
    E = (4 * h - 4 * (levels // 2)).astype(np.int32)
    g = pa.PARun(2, L, R, seed=1)
    g.import_state(R=R, step=1, sweeps=0, beta=0.1, lnZ=0.0, spins=np.zeros(((R + 63) // 64, N), np.uint64), energy=E,
                   magnetization=np.zeros(R, np.int32), label=np.arange(R, dtype=np.uint32))
    for db in (0.0, 0.001, 0.2):
        assert rel_ok(g.step_alpha(db), S.alpha(E, db), 1e-12)
    for astar, dmax, it in ((0.7, 0.2, 60), (0.9, 0.01, 20)):
        assert g.step_rule(astar, dmax, it) == S.step_rule(E, astar, dmax, it), (astar, dmax, it)
    g.close()
