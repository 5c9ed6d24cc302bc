"""The ancestor map where few replicas take most of the copies: steps far wider
than the energy distribution, so that one replica's copies span several
windows of a tile, and populations at the edges of the scans' tiles (1024,
4096 and 8192 slots) and of the switch between tile sizes, all four schemes,
against the oracle: sizes, labels and spins bit for bit."""
import pytest

from oracle import oracle as O
from tests.paritylib import run_pair

pytestmark = pytest.mark.gpu

WIDE = 1 << 18  # capacity from which the tiles hold 4096 slots


@pytest.mark.parametrize("scheme", [O.MULTINOMIAL, O.POISSON, O.NEAREST_INT, O.SYSTEMATIC])
@pytest.mark.parametrize("R,capacity", [(1, 64), (1023, None), (1025, None), (4096, None), (8193, None),
                                        (6000, WIDE), (WIDE + 1, None)])
def test_degenerate_steps(scheme, R, capacity):
    from paper_2401_07965_amd import pa
    L = 2 if R > 10000 else 4
    betas = [0.0, 0.05, 2.0, 5.0]
    try:
        g, _ = run_pair(2, L, R, scheme, betas, 1, seed=9, capacity=capacity)
        g.close()
    except pa.ExtinctError:  # the smallest populations can die out: the oracle's does too
        o = O.OracleRun(2, L, R, seed=9, capacity=capacity if capacity else O.default_capacity(R))
        with pytest.raises(O.ExtinctError):
            for b in betas[1:]:
                o.reweight(b)
                o.resample(scheme)
                o.sweep(1)
