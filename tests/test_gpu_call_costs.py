"""Calls that only read a run's state cost a record's copy, whatever the run's
size."""
import statistics
import time

import pytest

pytestmark = pytest.mark.gpu


def median_us(f, n=60):
    f()
    t = []
    for _ in range(n):
        t0 = time.perf_counter()
        f()
        t.append((time.perf_counter() - t0) * 1e6)
    return statistics.median(t)


def test_counters_cost_a_record():
    """62500 columns: adding up a count per column took three times a record's copy."""
    from paper_2401_07965_amd import pa
    g = pa.PARun(2, 4, 4000000)
    g.sweep(1)
    record = median_us(lambda: g.free_energy())
    counters = median_us(lambda: g.counters())
    print(f"record {record:.1f} us, counters {counters:.1f} us", flush=True)
    assert counters < 1.6 * record
    g.close()


def test_counters_of_more_columns_than_slots():
    """Every column's evaluations are counted: equal runs of 300 columns count
    alike, and 300 columns in proportion to 150 of the same spins' statistics."""
    from paper_2401_07965_amd import pa
    c = []
    for R in (64 * 150, 64 * 300, 64 * 300):
        g = pa.PARun(2, 8, R, seed=3)
        for b in (0.2, 0.4):
            g.reweight(b)
            g.resample("systematic")
            g.sweep(4)
        c.append(g.counters())
        g.close()
    assert c[1] == c[2]
    # 8 sweeps of 64 sites a word, between one plane pair each and sixteen
    for k, W in ((0, 150), (1, 300)):
        assert c[k]["site_updates"] == 8 * 64 * W
        assert c[k]["site_updates"] <= c[k]["philox_calls"] <= 16 * c[k]["site_updates"]
    ratio = c[1]["philox_calls"] / c[0]["philox_calls"]
    assert abs(ratio - 2.0) < 0.02  # 76800 and more independent word updates each
