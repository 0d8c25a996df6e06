"""The time step of many tracks, whose reference density looks at all pairs:
parallel and tilted tracks, several arrival times, periodic and absorbing
cells, separate radii, and offsets of many cell widths, against the oracle."""
import itertools

import numpy as np
import pytest

import workloads as W

FORMS = list(itertools.product((1, 2, 37), (0.0, 0.6), (0, 3), (0, 1), (False, True), (0.0, 1e3, 1e9)))


@pytest.mark.parametrize("n,tilt,late,absorbing,radii,offset", FORMS)
def test_dt_of_many_tracks(orc, n, tilt, late, absorbing, radii, offset):
    import paper_1610_06749_amd as it
    r = np.random.default_rng(n)
    L = 48 * 5e-4
    cols = [np.exp(r.uniform(0, 5, n)), r.uniform(5e-4, 2.5e-3, n), r.uniform(0, L, n) + offset, r.uniform(0, L, n),
            r.uniform(0, tilt, n), r.uniform(0, 6, n), np.floor(r.uniform(0, late, n)) * 1e-6]
    if radii:
        cols.append(r.uniform(5e-4, 2e-3, n))
    tr = np.stack(cols, axis=1)
    ch = W.chamber(48, 40, 20, 5e-4, 0.01, 200.0, lateral_bc=absorbing, uniform_n0=1e5)
    assert it.it_dt(ch, tr) == pytest.approx(orc.dt(ch, tr), rel=1e-14)
