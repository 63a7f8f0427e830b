"""A history follows one path, bit for bit, in the transport, in its replay and
in the adjoint's replay.  The detector's pixels are as fine as the FP32
rounding of an arrival point (0.6 um; a direction one ulp off moves the arrival
by about 0.02 um per cm flown), so a kernel that rounds a scattered direction
in another way puts a few percent of the scattered arrivals in another bin."""
import math

import numpy as np
import pytest

import phantoms
from parity import ids_of_work

pytestmark = pytest.mark.gpu


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _run(options):
    mc = _mc()
    p = phantoms.thorax_problem("paths", 24, 0.8, 5, 1, 180.0, 8192, 0.8, 200_000_000)
    dp = mc.to_device(p.with_(pixel_cm=0.5 / 8192, accept_half_angle_rad=math.radians(80.0), e_lo_kev=20.0,
                              e_cut_kev=20.0))
    sim = mc.simulate(dp, event_capacity=1 << 17, want_sq=False, options=options)
    ev = sim.events_numpy()
    assert 2000 < len(ev) < 1 << 17
    return mc, p, dp, sim, ev


@pytest.mark.parametrize("options", [{}, {"variance_reduction": 2},
                                     {"variance_reduction": 3, "forced_direction_half_angle": 2.0}])
def test_replay_follows_the_transport(options):
    mc, p, dp, sim, ev = _run(options)
    views, hists = ids_of_work(p, ev["work"])
    r = mc.replay(dp, views, hists, options=options)
    nu = dp.nu
    scattered = r["n_scatter"] > 0
    assert scattered.sum() > 1000
    np.testing.assert_array_equal(r["fate"], 5)
    np.testing.assert_array_equal(((views.astype(np.int64) * 2 + r["cls"]) * dp.nv + r["iv"]) * nu + r["iu"], ev["bin"])


def test_adjoint_follows_the_transport():
    """Every listed event replays to its bin: the adjoint raises otherwise."""
    import torch
    mc, _, dp, sim, ev = _run({})
    g = mc.adjoint(dp, torch.ones(dp.tally_shape, dtype=torch.float64, device="cuda"), sim)
    assert float(g.abs().sum()) > 0.0
