"""The level histogram that a reweighting builds by itself against the one the
observables leave: the same ln Q and resampled population bit for bit, for
populations of part of a tile, several tiles and both tile sizes, narrow and
as wide as the lattice's levels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,R,span", [(4, 1, 1), (8, 1023, 20), (8, 1025, 65), (128, 5000, 16385), (16, 4097, 100),
                                      (8, 262144, 65), (64, 300001, 4097)])
def test_either_build(L, R, span):
    from paper_2401_07965_amd import pa
    N = L * L
    rng = np.random.default_rng(R)
    lo = (N + 1 - span) // 2
    E = (-2 * N + 4 * (lo + rng.integers(0, span, R))).astype(np.int32)
    E[:2] = [-2 * N + 4 * (lo + k) for k in (span - 1, 0)][:min(R, 2)]
    out = []
    for observe in (False, True):
        g = pa.PARun(2, L, R, seed=2)
        g.import_state(R=R, step=1, sweeps=0, beta=0.1, lnZ=0.0, spins=np.zeros(((R + 63) // 64, N), np.uint64),
                       energy=E, magnetization=np.full(R, N, np.int32), label=np.arange(R, dtype=np.uint32))
        if observe:
            g.observables()
        lnq = g.reweight(0.1 + 1.0 / N)
        g.resample("systematic")
        s = g.export()
        out.append((lnq, s["energy"], s["label"]))
        g.close()
    assert out[0][0] == out[1][0]
    np.testing.assert_array_equal(out[0][1], out[1][1])
    np.testing.assert_array_equal(out[0][2], out[1][2])
