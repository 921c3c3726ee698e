"""The load-balance report, on records made by hand (no GPU)."""
import numpy as np
import pytest

from paper_2505_19609_amd import balance


@pytest.mark.parametrize("per_unit", [1, 2, 3])
def test_places_of_a_unit_are_those_that_were_taken(per_unit):
    """Units with `per_unit` workgroups at a time, eight items after another in each: a greedy schedule of the same
    durations on as many places takes exactly as long, whichever shape the kernel had."""
    units, rows = 6, []
    for u in range(units):
        for p in range(per_unit):
            for i in range(8):
                t0 = 1000 + 100 * i
                rows.append((t0, t0 + 100, u << 8, 0, (i * per_unit + p) * units + u, 1))
    r = balance.analyse(np.array(rows, dtype=balance.REC))
    assert r["places_per_unit"] == per_unit
    assert r["span_over_greedy"] == 1.0 and r["busy"] == 1.0 and r["sum_wg_time_over_units_x_span"] == 1.0
    assert r["ideal_span_us"] == r["span_us"] == 8.0
    assert balance.analyse(np.array(rows, dtype=balance.REC), per_unit) == r
