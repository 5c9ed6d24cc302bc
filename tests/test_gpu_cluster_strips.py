"""Cluster updates at the sizes where the division of a column into strips
changes: strips of four or two sites, one or two per lane, rows of a single
strip, workgroups that the strips do not fill; against the oracle, several
updates in one call, with and without couplings, a ragged last column."""
import pytest

from oracle import oracle as O
from tests.paritylib import compare_state, ea_couplings, rel_ok

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("glass", [False, True])
@pytest.mark.parametrize("d,L,R", [(2, 2, 65), (2, 4, 70), (2, 10, 130), (2, 46, 66), (2, 62, 64), (2, 64, 3),
                                   (3, 2, 70), (3, 4, 64), (3, 10, 65), (3, 12, 66), (3, 14, 65)])
def test_cluster_strips(d, L, R, glass):
    from paper_2401_07965_amd import pa
    J = ea_couplings(d, L, 5) if glass else None
    beta = (0.6 if glass else 0.42) if d == 2 else (0.5 if glass else 0.21)
    print(f"[cluster] d={d} L={L} R={R} glass={glass}", flush=True)
    g = pa.PARun(d, L, R, seed=3, run_id=7, couplings=J)
    o = O.OracleRun(d, L, R, seed=3, run_id=7, J=J)
    for b, n in ((beta / 2, 1), (beta, 3)):
        assert rel_ok(g.reweight(b), o.reweight(b))
        assert g.resample(O.SYSTEMATIC) == o.resample(O.SYSTEMATIC)
        g.cluster(n)
        o.cluster(n)
        compare_state(g, o, f"beta {b}")
    g.close()
