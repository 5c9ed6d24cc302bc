"""Batches of small runs, middle and tiny ones started apart where they are
many; against the same runs alone, bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

FIELDS = ("beta", "lnQ", "lnZ", "sv", "R", "sum_E", "sum_E2", "sum_M2", "sum_c2", "families", "e", "m2", "S_f", "status")


def alone(cfg, betas, theta, scheme):
    from paper_2401_07965_amd import pa
    B = pa.PABatch([cfg], max_points=len(betas))
    B.anneal(betas, theta, scheme, use_graph=False)
    rec = B.records()[0]
    B.close()
    return rec


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("scheme", [O.POISSON, O.NEAREST_INT, O.SYSTEMATIC])
def test_middle_and_tiny_runs_apart(scheme, large):
    """Sizes in no order: the middle ones' records are in their own rows."""
    from paper_2401_07965_amd import pa
    betas = [0.0, 0.2, 0.4, 0.6]
    cfgs = [dict(dim=2, L=4, R=1100 + k if k % 7 == 3 else 30 + k % 50, seed=5, run_id=k) for k in range(600)]
    if large:
        cfgs[100] = dict(dim=2, L=4, R=5000, seed=5, run_id=100)
    B = pa.PABatch(cfgs, max_points=len(betas))
    B.anneal(betas, 2, scheme, use_graph=False)
    rec = B.records()
    for k in (0, 3, 10, 99, 100, 101, 598, 599):
        one = alone(cfgs[k], betas, 2, scheme)
        for f in FIELDS:
            assert np.array_equal(rec[k][f], one[f]), (k, f)
    B.close()
