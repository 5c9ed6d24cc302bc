"""Observables of small runs (one workgroup) against those of large ones (three
passes): the same run with a capacity on either side of the switch gives the
same numbers bit for bit, uniform and weighted, and both match the oracle;
also with an energy range wider than the counts kept in LDS and in a batch
that mixes small and large runs."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.paritylib import compare_observables, ea_couplings, schedule

pytestmark = pytest.mark.gpu

SMALL = 4096


@pytest.mark.parametrize("R", [1, 63, 1000, 1025, 2049, 4000])
def test_either_side_of_the_switch(R):
    from paper_2401_07965_amd import pa
    J = ea_couplings(3, 4, 2)
    runs = [pa.PARun(3, 4, R, seed=6, capacity=c, couplings=J) for c in (SMALL, SMALL + 64)]
    o = O.OracleRun(3, 4, R, seed=6, capacity=SMALL, J=J)
    print(f"[obs] R={R}", flush=True)
    for b in (0.1, 0.2, 0.4, 0.45, 0.5):
        for r in runs + [o]:
            r.reweight(b)
            if b < 0.4:
                r.resample(O.SYSTEMATIC)
            else:
                r.resample_conditional(O.SYSTEMATIC, 0.2)
            r.sweep(2)
        a, c = (r.observables() for r in runs)
        assert a == c, (b, a, c)
        if b < 0.4:
            compare_observables(runs[0], o, f"beta {b}")
    for r in runs:
        r.close()


def test_wide_energy_range():
    """More levels than a workgroup counts in LDS (imported energies): the
    reweighting after it sees the whole histogram."""
    from paper_2401_07965_amd import pa
    L, R = 64, 900
    N = L * L
    E = (4 * np.random.default_rng(1).integers(-1800, 1800, R)).astype(np.int32)
    E[:2] = -4 * 1800, 4 * 1799
    g = [pa.PARun(2, L, R, seed=1, capacity=c) for c in (1024, SMALL + 64)]
    q = []
    for r in g:
        r.import_state(R=R, step=1, sweeps=0, beta=0.1, lnZ=0.0, spins=np.zeros(((R + 63) // 64, N), np.uint64),
                       energy=E, magnetization=np.full(R, 2, np.int32), label=np.arange(R, dtype=np.uint32) // 7)
        a = r.observables()
        assert a["sum_E"] == int(E.astype(np.int64).sum()) and a["families"] == (R + 6) // 7
        q.append((a, r.reweight(0.1005)))
        r.close()
    assert q[0] == q[1]


def test_mixed_batch():
    from paper_2401_07965_amd import pa
    betas = schedule(0.6, 5)
    cfgs = [dict(dim=2, L=4, R=r, seed=3, run_id=k) for k, r in enumerate((50, 40000, 3000, 1000, 5000))]
    B = pa.PABatch(cfgs, max_points=len(betas))
    B.anneal(betas, 2, O.POISSON)
    rec = B.records()
    for k, c in enumerate(cfgs):
        S = pa.PABatch([c], max_points=len(betas))
        S.anneal(betas, 2, O.POISSON, use_graph=False)
        assert np.array_equal(S.records()[0], rec[k]), k
        S.close()
    B.close()
