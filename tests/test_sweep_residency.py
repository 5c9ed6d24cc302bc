"""Sweep waves a CU holds: more than four to a SIMD only where LDS has room for
six, since between the two the SIMDs fill unevenly and a launch waits for the
fullest."""
import ctypes

import pytest

from tests.paritylib import compare_state, ea_couplings


def waves_cap(N, d, threads, J):
    from paper_2401_07965_amd import build, pa
    import os
    if not os.path.exists(pa.LIB_PATH):
        build.build()
    f = ctypes.CDLL(pa.LIB_PATH)["_Z18pa_sweep_waves_capiiib"]
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool], ctypes.c_int
    return f(N, d, threads, J)


#        d, L, lanes, glass: waves that fit the LDS
UNEVEN = [(2, 32, 128, False),  # 20
          (2, 32, 128, True),   # 18
          (2, 24, 64, True),    # 18
          (2, 24, 128, False),  # 22
          (2, 20, 64, False),   # 18
          (3, 8, 64, True),     # 18
          (3, 8, 64, False)]    # 20


@pytest.mark.parametrize("d,L,lanes,glass", UNEVEN)
def test_uneven_waves_keep_to_four_a_simd(d, L, lanes, glass):
    assert waves_cap(L ** d, d, lanes, glass) == 16


@pytest.mark.parametrize("d,L,lanes,glass,cap", [(2, 16, 64, False, 28), (2, 8, 128, False, 28), (3, 6, 64, True, 20),
                                                 (3, 8, 128, True, 20), (3, 16, 256, True, 16)])
def test_other_shapes_keep_their_waves(d, L, lanes, glass, cap):
    assert waves_cap(L ** d, d, lanes, glass) == cap


@pytest.mark.gpu
@pytest.mark.parametrize("d,L,lanes,glass", UNEVEN)
def test_their_sweeps_against_the_oracle(d, L, lanes, glass):
    from oracle import oracle as O
    from paper_2401_07965_amd import pa
    R, betas = 70, [0.0, 0.3, 1.0]
    J = ea_couplings(d, L, 4) if glass else None
    o = O.OracleRun(d, L, R, seed=8, run_id=2, J=J)
    for b in betas[1:]:
        o.reweight(b)
        o.resample(O.SYSTEMATIC)
        o.sweep(3)
    B = pa.PABatch([dict(dim=d, L=L, R=R, seed=8, run_id=2, couplings=J)], max_points=len(betas))
    B.set_threads(0, lanes)
    B.anneal(betas, 3, O.SYSTEMATIC, use_graph=False)

    class Exported:
        export = staticmethod(lambda: B.export_run(0))

    compare_state(Exported, o, "end")
    B.close()
