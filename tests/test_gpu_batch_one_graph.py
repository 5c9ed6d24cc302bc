"""A batch of several groups keeps the graph of its first captured anneal: an
anneal with other sizes, sweeps or temperatures in between is launched
directly, and the first one's arguments replay it; all as a plain batch."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.paritylib import ea_couplings, schedule

pytestmark = pytest.mark.gpu


def test_other_anneals_between_replays():
    from paper_2401_07965_amd import pa
    cfgs = [dict(dim=2, L=8, R=300, seed=1, run_id=0), dict(dim=2, L=12, R=200, seed=1, run_id=1),
            dict(dim=3, L=6, R=5000, seed=1, run_id=2, couplings=ea_couplings(3, 6, 1))]
    a, b = schedule(0.6, 6), schedule(0.9, 5)
    B = pa.PABatch(cfgs, max_points=6)
    sizes = B.groups()
    P = pa.PABatch(cfgs, max_points=6)

    def check(betas, theta, scheme, graph):
        B.anneal(betas, theta, scheme, use_graph=graph)
        P.anneal(betas, theta, scheme, use_graph=False)
        x, y = B.records(), P.records()
        assert all(np.array_equal(x[f], y[f]) for f in x.dtype.names)
        for m in range(len(cfgs)):
            s, t = B.export_run(m), P.export_run(m)
            assert all(np.array_equal(s[f], t[f]) for f in ("spins", "energy", "label"))

    check(a, 3, O.SYSTEMATIC, True)   # captured
    check(b, 3, O.SYSTEMATIC, True)   # another schedule
    check(a, 3, O.SYSTEMATIC, True)   # replayed
    B.set_threads(2, 64 if sizes[2] != 64 else 128)
    check(a, 3, O.SYSTEMATIC, True)   # other sizes
    check(a, 2, O.POISSON, True)      # and another scheme
    check(b, 1, O.NEAREST_INT, False)
    B.set_threads(2, sizes[2])
    for _ in range(3):
        check(a, 3, O.SYSTEMATIC, True)  # replayed
    B.close()
    P.close()
