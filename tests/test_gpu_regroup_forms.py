"""GPU: the two sides of the benchmark's regrouping comparison are the same form, passes with and without the sort."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench
from paper_1101_1245_amd import gpumcd as G, inputs as I

pytestmark = pytest.mark.gpu


def test_both_sides_run_as_passes():
    ph = I.homogeneous(16, 0.5)
    beams = [I.centred(ph, I.Source(p, e=6.0, wx=2.0, wy=2.0, beam_id=p)) for p in (I.PHOTON, I.ELECTRON)]
    with G.Context(0) as c:
        pid, tid = c.load_phantom(ph), c.load_tables((I.WATER,), I.Physics(ecut=0.7, pcut=0.05))
        got = [c.run_beams(pid, tid, beams, [20_000, 5_000], 3, tuning=dict(bench.REGROUP_TUNING, energy_sort=s))
               for s in (0, 1)]
    for r in got:
        assert r[4]["n_electron_launches"] > 0 and r[4]["n_photon_launches"] > 0 and r[4]["n_round_launches"] == 0
    assert np.array_equal(got[0][2], got[1][2])
