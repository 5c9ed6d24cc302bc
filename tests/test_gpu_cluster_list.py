"""Cluster updates at temperatures where the clusters grow from a list of their
sites, and on either side of the change; a list that overflows leaves the rest
of the call to the other kernel; populations of one column, of part of one and
of more columns than CUs; several updates in a call; against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.paritylib import compare_state, ea_couplings, rel_ok

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("glass", [False, True])
@pytest.mark.parametrize("d,L,R", [(2, 2, 65), (2, 24, 70), (2, 30, 66), (2, 32, 130), (2, 64, 3), (3, 2, 70),
                                   (3, 6, 65), (3, 12, 66), (3, 16, 65)])
def test_cold_to_hot(d, L, R, glass):
    """(2 d - 1) (1 - exp(-2 beta)) = 0, then up to and across 1.2."""
    from paper_2401_07965_amd import pa
    J = ea_couplings(d, L, 5) if glass else None
    print(f"[cluster] d={d} L={L} R={R} glass={glass}", flush=True)
    g = pa.PARun(d, L, R, seed=3, run_id=7, couplings=J)
    o = O.OracleRun(d, L, R, seed=3, run_id=7, J=J)
    for r in (g, o):
        r.cluster(2)
    compare_state(g, o, "beta 0")
    for x in (0.06, 0.6, 1.19, 1.21, 1.5):
        b = -0.5 * float(np.log1p(-x / (2 * d - 1)))
        assert rel_ok(g.reweight(b), o.reweight(b))
        assert g.resample(O.SYSTEMATIC) == o.resample(O.SYSTEMATIC)
        for n in (1, 3):
            g.cluster(n)
            o.cluster(n)
        g.sweep(1)
        o.sweep(1)
        compare_state(g, o, f"x {x}")
    g.close()


def test_a_full_list():
    """Aligned spins (imported) with p just below the percolation threshold of
    the cubic lattice's bonds: lists overflow, in the first update or a later
    one of the call."""
    from paper_2401_07965_amd import pa
    d, L, R = 3, 16, 70
    N = L ** d
    b = -0.5 * float(np.log1p(-1.19 / 5))
    g, o = pa.PARun(d, L, R, seed=4), O.OracleRun(d, L, R, seed=4)
    for r in (g, o):
        r.reweight(b)
        r.resample(O.SYSTEMATIC)
    st = g.export()
    E = np.full(R, -3 * N, np.int32)
    g.import_state(R=R, step=st["step"], sweeps=0, beta=b, lnZ=st["lnZ"], spins=np.zeros_like(st["spins"]), energy=E,
                   magnetization=np.full(R, N, np.int32), label=st["label"])
    o.import_state(np.ones((R, N), np.int8), E, st["label"])
    largest = 0
    for n in (1, 4):
        before = o.spins.copy()
        g.cluster(n)
        o.cluster(n)
        largest = max(largest, int((o.spins != before)[:64].sum()))
        compare_state(g, o, f"{n} updates")
    print(f"[cluster] sites flipped in a column: {largest}", flush=True)
    assert largest > 1024
    g.close()


def test_more_columns_than_cus():
    from paper_2401_07965_amd import pa
    R = 64 * 270 + 5
    g = pa.PARun(2, 24, R, seed=6)
    o = O.OracleRun(2, 24, R, seed=6)
    for b in (0.05, 0.2):
        assert rel_ok(g.reweight(b), o.reweight(b))
        assert g.resample(O.SYSTEMATIC) == o.resample(O.SYSTEMATIC)
        g.cluster(2)
        o.cluster(2)
        compare_state(g, o, f"beta {b}")
    g.close()


@pytest.mark.parametrize("d,L,glass,taken", [(2, 64, True, True), (2, 66, False, False), (2, 68, False, False),
                                             (3, 16, True, True), (3, 18, False, False), (3, 20, False, False)])
def test_largest_lattices(d, L, glass, taken):
    """4096 sites are taken, more refused, with the bound in the message."""
    from paper_2401_07965_amd import pa
    g = pa.PARun(d, L, 10, seed=1, couplings=ea_couplings(d, L, 1) if glass else None)
    if taken:
        g.cluster(1)
        g.export()
    else:
        with pytest.raises(pa.PAError, match="4096"):
            g.cluster(1)
    g.close()
