"""The step rule's search where its division of work changes: populations
over one level up to more levels than the waves share (imported energies),
few and many halvings, targets near both ends; bit for bit against the
oracle's bisection."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import schedule as S
from tests.paritylib import rel_ok

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [1, 2, 64, 65, 1023, 1024, 1025, 2048, 2049, 3500])
def test_rule_over_levels(levels):
    from paper_2401_07965_amd import pa
    L, R = 64, 700
    N = L * L
    rng = np.random.default_rng(levels)
    h = rng.integers(0, levels, R)
    h[0], h[-1] = 0, levels - 1
    E = (4 * h - 4 * (levels // 2)).astype(np.int32)
    print(f"[rule] levels={levels}", flush=True)
    g = pa.PARun(2, L, R, seed=1)
    g.import_state(R=R, step=1, sweeps=0, beta=0.1, lnZ=0.0, spins=np.zeros(((R + 63) // 64, N), np.uint64), energy=E,
                   magnetization=np.zeros(R, np.int32), label=np.arange(R, dtype=np.uint32))
    for db in (0.0, 0.001, 0.2):
        assert rel_ok(g.step_alpha(db), S.alpha(E, db), 1e-12)
    for astar, dmax, it in ((0.7, 0.2, 60), (0.7, 0.2, 1), (0.7, 0.2, 3), (0.7, 0.2, 10), (0.999, 0.5, 200),
                            (0.01, 3.0, 61), (0.7, 1e-9, 20)):
        assert g.step_rule(astar, dmax, it) == S.step_rule(E, astar, dmax, it), (astar, dmax, it)
    g.close()
