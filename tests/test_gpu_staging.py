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


@pytest.mark.parametrize("n", [8, 16, 17, 48, 101])
def test_small_problem_alone_and_beside_a_large_one(n):
    """A call of problems of at most 256 stretches of 4096 voxels has its maxima
    and prefixes taken by each workgroup; beside a problem of more, a launch of
    its own takes them: the same bits, for one stretch and less up to 252."""
    mc = _mc()
    p = mc.to_device(phantoms.thorax_problem("small", n, 38.4 / n, 3, 3, 180.0, 16, 2.4, 40_000))
    big = mc.to_device(phantoms.thorax_problem("big", 104, 0.36, 4, 3, 180.0, 16, 2.4, 10_000, problem_id=1))
    a, b = mc.simulate([p]), mc.simulate([p, big])
    m = a.tally.numel()
    for x, y in ((a.tally, b.tally[:m]), (a.tally_sq, b.tally_sq[:m]), (a.fates[0], b.fates[0]),
                 (a.energy[0], b.energy[0]), (a.counters[0], b.counters[0])):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
    assert int(a.fates[0].sum().item()) == 40_000
