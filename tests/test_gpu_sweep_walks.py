"""Every walk of the sweeps over a colour's sites (coordinates kept from pass
to pass, the site table, coordinates computed at each site) at workgroup sizes
that select it, small populations, with and without couplings, above and below
the temperature where the coldest class stops drawing; against the oracle."""
import pytest

from oracle import oracle as O
from tests.paritylib import compare_state, ea_couplings, run_pair

pytestmark = pytest.mark.gpu

#        d, L, lanes     walk
SHAPES = [(2, 48, 64),   # index: the table would cost resident waves
          (2, 48, 192),  # fixed axis
          (2, 12, 64),   # table
          (2, 10, 320),  # fixed axis, lanes without a site
          (2, 22, 192),  # table
          (3, 14, 128),  # index
          (3, 10, 128),  # table
          (3, 6, 64),    # table
          (3, 12, 576),  # fixed axis
          (3, 8, 64),    # fixed axis
          (3, 16, 256)]  # fixed axis, wave-uniform z


@pytest.mark.parametrize("glass", [False, True])
@pytest.mark.parametrize("d,L,lanes", SHAPES)
def test_walks(d, L, lanes, glass):
    from paper_2401_07965_amd import pa
    betas, R = [0.0, 0.2, 1.0, 2.0, 3.0], 70
    J = ea_couplings(d, L, 4) if glass else None
    print(f"[walk] d={d} L={L} lanes={lanes} glass={glass}", flush=True)
    o = O.OracleRun(d, L, R, seed=8, run_id=2, J=J)
    for b in betas[1:]:
        o.reweight(b)
        o.resample(O.SYSTEMATIC)
        o.sweep(2)
    B = pa.PABatch([dict(dim=d, L=L, R=R, seed=8, run_id=2, couplings=J)], max_points=len(betas))
    B.set_threads(0, lanes)
    B.anneal(betas, 2, O.SYSTEMATIC, use_graph=False)

    class Exported:
        export = staticmethod(lambda: B.export_run(0))

    compare_state(Exported, o, "end")
    B.close()


def test_sweeps_at_infinite_temperature():
    """beta = 0: every move is accepted outright."""
    for d, L in ((2, 12), (3, 6)):
        g, o = run_pair(d, L, 100, O.SYSTEMATIC, [0.0, 0.0], 3, J=ea_couplings(d, L, 2))
        compare_state(g, o, "beta 0")
        g.close()
