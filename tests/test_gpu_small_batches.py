"""Batches of small runs: middle and tiny ones started apart where they are
many, populations over more levels than the lanes of a workgroup, and the
records of a run that dies out; against the same runs alone, bit for bit."""
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


@pytest.mark.parametrize("scheme", [O.MULTINOMIAL, O.SYSTEMATIC])
def test_more_levels_than_lanes(scheme):
    """More than 256 runs, each over more than 256 energy levels (multinomial:
    the reweighting as a launch of its own)."""
    from paper_2401_07965_amd import pa
    betas = [0.0, 0.2, 0.35, 0.42, 0.44, 0.443]
    cfgs = [dict(dim=2, L=96, R=900, seed=5, run_id=k) for k in range(260)]
    B = pa.PABatch(cfgs, max_points=len(betas))
    B.anneal(betas[:-1], 3, scheme, use_graph=False)
    spans = [int(np.ptp(B.export_run(k)["energy"])) // 4 + 1 for k in (0, 259)]
    print(f"[levels] scheme {scheme}: {spans}", flush=True)
    assert min(spans) > 256
    B.anneal(betas, 3, scheme, use_graph=False)
    rec = B.records()
    for k in (0, 131, 259):
        g = pa.PARun(**cfgs[k])
        for i, b in enumerate(betas[1:], 1):
            q = g.reweight(b)
            g.resample(scheme)
            g.sweep(3)
            o = g.observables()
            assert (rec[k]["lnQ"][i], rec[k]["sum_E"][i], rec[k]["sum_c2"][i]) == (q, o["sum_E"], o["sum_c2"]), (k, i)
        g.close()
    B.close()


@pytest.mark.parametrize("graph", [False, True])
def test_records_of_a_run_that_dies_out(graph):
    """Poisson copy numbers leave a run of one replica extinct sooner or later:
    its status says so from that step on, and its rows repeat the last good
    step; the other runs of the batch go on."""
    from paper_2401_07965_amd import pa
    betas = [0.0, 0.15, 0.3, 0.32, 0.9]
    cfgs = [dict(dim=2, L=8, R=r, seed=5, run_id=k) for k, r in enumerate((1, 1, 1, 1, 1, 1, 1, 1, 63, 900))]
    B = pa.PABatch(cfgs, max_points=len(betas))
    B.anneal(betas, 2, O.POISSON, use_graph=graph)
    rec = B.records()
    died = 0
    for k, c in enumerate(cfgs):
        g = pa.PARun(**c)
        last = 0
        for i, b in enumerate(betas[1:], 1):
            g.reweight(b)
            try:
                g.resample(O.POISSON)
            except pa.ExtinctError:
                break
            g.sweep(2)
            last = i
        g.close()
        assert not rec[k]["status"][:last + 1].any()
        for i in range(last + 1, len(betas)):
            assert rec[k]["status"][i] != 0, (k, i)
            for f in ("beta", "lnZ", "R", "sum_E", "sum_M2", "sum_c2", "families", "e", "m2"):
                assert rec[k][f][i] == rec[k][f][last], (k, i, f)
        died += last + 1 < len(betas)
    assert 0 < died <= 8 and rec[9]["beta"][-1] == betas[-1]
    B.close()
