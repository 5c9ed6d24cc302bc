"""Word-site updates and attempts of populations that do not fill their last
column and change size: their closed forms; Philox evaluations: at least the
oracle's, which counts live replicas alone (the library draws whole words), and
the same when read again; in one wave and in several per column."""
import pytest

from oracle import oracle as O
from tests.paritylib import ea_couplings

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,R", [(2, 4, 1), (2, 8, 130), (3, 6, 777), (2, 32, 300)])
def test_ragged(d, L, R):
    from paper_2401_07965_amd import pa
    J = ea_couplings(d, L, 3) if d == 3 else None
    g = pa.PARun(d, L, R, seed=8, couplings=J)
    o = O.OracleRun(d, L, R, seed=8, J=J)
    updates = attempts = 0
    for k, b in enumerate((0.1, 0.2, 0.3)):
        for r in (g, o):
            r.reweight(b)
            r.resample(O.SYSTEMATIC if k == 0 or R == 1 else O.POISSON)
            r.sweep(k + 1)
        assert g.export(arrays=False)["R"] == o.Rcur
        updates += (k + 1) * L ** d * ((o.Rcur + 63) // 64)
        attempts += (k + 1) * L ** d * o.Rcur
        c = g.counters()
        assert c["philox_calls"] >= o.philox_calls, (b, c)
        assert c["site_updates"] == updates and c["spin_attempts"] == attempts
        assert c == g.counters()
    g.close()
