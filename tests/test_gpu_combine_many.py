"""The combination over more runs than a workgroup has lanes, in groups of all
sizes down to an empty one, against the oracle; and the final states of runs
read out of such a batch one by one."""
import math

import numpy as np
import pytest

from oracle import combine as OC
from oracle import oracle as O
from tests.paritylib import rel_ok, schedule

pytestmark = pytest.mark.gpu


def test_many_runs():
    from paper_2401_07965_amd import pa
    betas = schedule(0.5, 4)
    n = 601
    B = pa.PABatch([dict(dim=2, L=4, R=20 + k % 70, seed=5, run_id=k) for k in range(n)], max_points=len(betas))
    B.anneal(betas, 2, O.NEAREST_INT)
    rec = B.records()
    groups = [0 if k % 3 else (1 if k % 2 else -1) for k in range(n)]
    groups[600] = 3  # group 2 stays empty, group 3 has one run
    out = B.combine(groups, 4, 3)
    for g in (0, 1, 3):
        rs = [{k: (int if k == "R" else float)(rec[m, 3][k]) for k in ("R", "lnZ", "beta", "e", "e2", "abs_m", "m2")}
              for m in range(n) if groups[m] == g]
        ref = OC.combine(rs, 16)
        assert out[g]["runs"] == ref["runs"] == len(rs)
        # float64 sums of up to 400 terms; c and chi are differences of numbers about ten times as large
        for k in ("lnZ", "e", "e2", "abs_m", "m2", "c", "chi", "n_eff", "c_naive", "chi_naive", "e_plain", "c_plain",
                  "chi_plain"):
            assert rel_ok(out[g][k], ref[k], 1e-11), (g, k, out[g][k], ref[k])
    assert out[2]["runs"] == 0 and math.isnan(out[2]["lnZ"]) and out[2]["n_eff"] == 0.0
    for m in (0, 255, 256, 600):
        st = B.export_run(m)
        assert st["R"] == rec[m, 3]["R"] and rel_ok(st["lnZ"], rec[m, 3]["lnZ"], 0.0)
        assert int(st["energy"].astype(np.int64).sum()) == rec[m, 3]["sum_E"]
        assert int(np.abs(st["magnetization"].astype(np.int64)).sum()) == rec[m, 3]["sum_absM"]
    B.close()
