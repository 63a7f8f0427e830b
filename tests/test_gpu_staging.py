"""Input staging at the sizes where its passes can go wrong: the threshold
palette around its capacity, with the distinct values together or spread over
the workgroups."""
import numpy as np
import pytest

import phantoms

pytestmark = pytest.mark.gpu


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _same(a, b):
    for x, y in ((a.tally, b.tally), (a.fates, b.fates), (a.energy, b.energy), (a.counters, b.counters)):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())


@pytest.mark.parametrize("spread", ["rows", "shuffled"])
@pytest.mark.parametrize("brick", [0, 2])
@pytest.mark.parametrize("n_distinct", [1, 255, 256, 257, 300, 20_000])
def test_palette_around_its_capacity(n_distinct, brick, spread):
    """n_distinct attenuation values, in ascending order along the grid (each
    workgroup meets a few of them, the overflow shows only between
    workgroups) or shuffled (a workgroup meets them all): the palette is used
    iff they fit, and the run equals the 32-bit table's bit for bit."""
    mc = _mc()
    n = 48
    levels = (phantoms.MU_WATER_140 * (0.7 + 0.6 * np.arange(n_distinct) / max(1, n_distinct - 1))).astype(np.float32)
    mu = levels[np.arange(n ** 3) * n_distinct // n ** 3]
    if spread == "shuffled":
        np.random.Generator(np.random.PCG64(n_distinct)).shuffle(mu)
    p = phantoms.point_source_cube("palette", n, 0.4, 100_000, seed=9).with_(mu=mu.reshape(n, n, n))
    dp = mc.to_device(p)
    a = mc.simulate(dp, options={"brick_log2": brick})
    b = mc.simulate(dp, options={"brick_log2": brick, "threshold_bytes": 4})
    assert int(a.check_status()[2]) == (1 if n_distinct <= 256 else 0)
    _same(a, b)
