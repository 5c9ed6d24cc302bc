"""The resampling of small runs (one workgroup) against that of large ones
(passes over all runs): the same run with a capacity on either side of the
switch holds the same replicas and numbers bit for bit, uniform and weighted,
at the edges of its chunks, through wide steps; a resampling that does not fit
is refused on both sides of the chunk switch and can be repeated."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.paritylib import ea_couplings

pytestmark = pytest.mark.gpu

SMALL, CHUNK = 4096, 1024


@pytest.mark.parametrize("scheme", [O.POISSON, O.NEAREST_INT, O.SYSTEMATIC])
@pytest.mark.parametrize("R", [1, 63, 255, 900, 1000, 1025, 2049, 3700])
def test_either_side_of_the_switch(scheme, R):
    from paper_2401_07965_amd import pa
    J = ea_couplings(3, 4, 2)
    caps = ([CHUNK] if R <= 900 else []) + [SMALL, SMALL + 64]
    runs = [pa.PARun(3, 4, R, seed=6, capacity=c, couplings=J) for c in caps]
    print(f"[resample] scheme {scheme} R={R}", flush=True)
    for b, kappa in ((0.1, None), (0.2, None), (0.3, 0.2), (0.35, None), (1.2, None), (3.0, None)):
        out = []
        for r in runs:
            q = r.reweight(b)
            try:
                res = r.resample(scheme) if kappa is None else r.resample_conditional(scheme, kappa)
            except pa.ExtinctError:
                res = "extinct"
            r.sweep(1)
            obs = r.observables()
            st = r.export()
            out.append((q, res, obs, {k: np.asarray(v).tolist() for k, v in st.items()}))
        assert all(o == out[0] for o in out[1:]), b
    for r in runs:
        r.close()


@pytest.mark.parametrize("R,capacity", [(60, 64), (1000, 1024), (3000, 3008)])
def test_refused_and_repeated(R, capacity):
    """Poisson draws that overflow the capacity are refused (the oracle's are),
    the population stays, and the systematic scheme then resamples it."""
    from paper_2401_07965_amd import pa
    for seed in range(20):
        g = pa.PARun(2, 4, R, seed=seed, capacity=capacity)
        o = O.OracleRun(2, 4, R, seed=seed, capacity=capacity)
        g.reweight(0.3)
        o.reweight(0.3)
        try:
            o.resample(O.POISSON)
            g.resample(O.POISSON)
        except O.CapacityError:
            with pytest.raises(pa.CapacityError):
                g.resample(O.POISSON)
            o.resample(O.SYSTEMATIC)
            g.resample(O.SYSTEMATIC)
            a, b = g.export(), o.label[:o.R]
            assert a["R"] == o.R and np.array_equal(a["label"][:o.R], b)
            g.close()
            return
        g.close()
    pytest.fail("no seed overflowed the capacity")


@pytest.mark.parametrize("scheme", [O.MULTINOMIAL, O.POISSON, O.NEAREST_INT, O.SYSTEMATIC])
@pytest.mark.parametrize("sizes", [(1, 63, 900), (1000, 40, 2049, 3000)])
def test_anneal_against_steps(scheme, sizes):
    """A batch of small runs reweights and resamples in one launch; its runs are
    those of the step-by-step calls, also through a run that dies out."""
    from paper_2401_07965_amd import pa
    betas = [0.0, 0.15, 0.3, 0.32, 0.9]
    cfgs = [dict(dim=2, L=8, R=r, seed=5, run_id=k) for k, r in enumerate(sizes)]
    for graph in (False, True):
        print(f"[resample] batch {sizes} scheme {scheme} graph={graph}", flush=True)
        B = pa.PABatch(cfgs, max_points=len(betas))
        for _ in range(2):
            B.anneal(betas, 2, scheme, use_graph=graph)
        rec = B.records()
        for k, c in enumerate(cfgs):
            g = pa.PARun(**c)
            for i, b in enumerate(betas[1:], 1):
                q = g.reweight(b)
                try:
                    g.resample(scheme)
                except pa.ExtinctError:
                    break
                g.sweep(2)
                o = g.observables()
                assert (rec[k]["lnQ"][i], rec[k]["R"][i], rec[k]["sum_E"][i]) == (q, g.export(arrays=False)["R"], o["sum_E"])
            else:
                a, b = B.export_run(k), g.export()
                assert all(np.array_equal(a[f], b[f]) for f in ("spins", "energy", "magnetization", "label"))
            g.close()
        B.close()
