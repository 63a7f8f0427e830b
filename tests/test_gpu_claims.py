"""The transport's work claims and totals: every history runs exactly once,
whatever the number of chunks, queues, waves and problems."""
import numpy as np
import pytest

import phantoms

pytestmark = pytest.mark.gpu


def _mc():
    import paper_2105_13324_amd as mc
    return mc


@pytest.mark.parametrize("n_problems", [1, 3, 67])
@pytest.mark.parametrize("options", [{}, {"hist_per_lane": 1, "block_size": 64, "blocks_per_cu": 1},
                                     {"hist_per_lane": 1}, {"hist_per_lane": 3, "block_size": 192},
                                     {"forced_detection": 1}])
def test_every_history_once(n_problems, options):
    """Problems of 1 to about 40,000 histories: fewer chunks than queues, as
    many, and more than the waves take without a claim.  Histories, fates,
    energies and tallies per problem equal those of the problem run alone
    with one-history-per-lane claims on one small grid."""
    mc = _mc()
    base = phantoms.thorax_problem("claims", 16, 2.4, 3, 3, 180.0, 16, 2.4, 1)
    rng = np.random.Generator(np.random.PCG64(n_problems))
    counts = [40_000] if n_problems == 1 else [1, 63, 64, 2048][:n_problems] + \
        [int(x) for x in rng.integers(1, 4000, size=max(0, n_problems - 4))]
    probs = [mc.to_device(base.with_(n_histories=n, problem_id=k)) for k, n in enumerate(counts)]
    opt = dict(options)
    s = mc.simulate(probs, options=opt)
    assert [int(x) for x in s.fates.sum(dim=1).cpu()] == counts
    assert [int(x) for x in s.counters[:, 3].cpu()] == counts
    few = {"hist_per_lane": 1, "block_size": 128, "blocks_per_cu": 1}
    if "forced_detection" in opt:
        few["forced_detection"] = 1
    for k in range(0, n_problems, max(1, n_problems // 6)):
        one = mc.simulate(probs[k], options=few)
        np.testing.assert_array_equal(s.fates[k].cpu(), one.fates[0].cpu())
        np.testing.assert_array_equal(s.energy[k].cpu(), one.energy[0].cpu())
        np.testing.assert_array_equal(s.counters[k].cpu(), one.counters[0].cpu())
        np.testing.assert_array_equal(s.tallies()[k].cpu(), one.tallies()[0].cpu())


@pytest.mark.parametrize("n_hist", [64 * 32, 64 * 3072, 64 * 3072 + 1, 64 * 3072 * 2 - 5])
def test_chunks_around_the_number_of_waves(n_hist):
    """One chunk per queue, per wave, and just more: nothing lost or repeated
    when the last chunks are taken from other queues."""
    mc = _mc()
    p = phantoms.point_source_cube("claims", 16, 0.8, n_hist, nu=16, pixel_cm=1.6)
    dp = mc.to_device(p)
    a = mc.simulate(dp, options={"hist_per_lane": 1})
    b = mc.simulate(dp, options={"hist_per_lane": 16, "blocks_per_cu": 1, "block_size": 64})
    assert int(a.fates.sum()) == n_hist
    for x, y in ((a.tally, b.tally), (a.fates, b.fates), (a.energy, b.energy), (a.counters, b.counters)):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
