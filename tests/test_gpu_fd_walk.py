"""The forced copies' walk over the brick table of codes against the walk over
the FP32 map (taken when the palette is switched off): the same bits."""
import math

import numpy as np
import pytest

import phantoms

pytestmark = pytest.mark.gpu


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _problem(shape, fill, half_angle, n_hist):
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(nx * 1000 + ny * 10 + nz))
    # three materials in blocks, or water to every face of the grid
    mu = np.full(shape, phantoms.MU_WATER_140, dtype=np.float32)
    if fill == "blocks":
        b = rng.integers(0, 4, size=[(n + 4) // 5 for n in shape])
        b = np.kron(b, np.ones((5, 5, 5), dtype=np.int64))[:nz, :ny, :nx]
        mu = np.array([0.0, 0.045, 0.151, 0.28], dtype=np.float32)[b]
        mu[0, 0, 0] = 0.28
        if min(shape) > 8:                 # a box inside the grid on some faces
            mu[:, :, :3] = 0.0
            mu[:, -2:, :] = 0.0
    vox = 20.0 / max(shape)
    # axis-parallel, diagonal and general directions
    ang = np.array([0.0, math.pi / 2, math.pi / 4, math.pi, 0.3, 2.2, 4.4, 5.9])
    return phantoms.Problem(
        name="walk", nx=nx, ny=ny, nz=nz, voxel_cm=vox, mu=mu,
        activity=rng.integers(0, 5, size=shape).astype(np.uint32) + (np.arange(nx) == nx // 2).astype(np.uint32),
        angles=ang, nu=24, nv=20, pixel_cm=1.1, radius_cm=phantoms.detector_radius(nx, ny, vox),
        accept_half_angle_rad=half_angle, e_lo_kev=100.0, e_hi_kev=154.0, e_cut_kev=90.0, n_histories=n_hist, seed=3)


SHAPES = [(1, 1, 1), (1, 8, 16), (2, 9, 17), (5, 15, 31), (29, 31, 33), (32, 32, 32), (64, 24, 40), (7, 100, 65),
          (100, 3, 130)]


@pytest.mark.parametrize("fill", ["water", "blocks"])
@pytest.mark.parametrize("shape", SHAPES)
def test_code_walk_equals_map_walk(shape, fill):
    mc = _mc()
    for mode, half_angle in ((1, 0.035), (1, 0.5), (2, 0.035)):
        dp = mc.to_device(_problem(shape, fill, half_angle, 150_000))
        runs = []
        for opt in ({}, {"threshold_bytes": 4}, {"brick_log2": 2}):
            cap = 1 << 20 if mode == 1 else 0
            s = mc.simulate(dp, event_capacity=cap, options={"forced_detection": mode, **opt})
            assert int(s.status[2]) == (0 if "threshold_bytes" in opt else 1)
            ev = s.events_numpy()
            runs.append((s.tally.cpu().numpy(), s.tally_sq.cpu().numpy(), s.fates.cpu().numpy(),
                         s.counters.cpu().numpy(), np.sort(ev, order=["work", "bin", "weight"])))
        assert runs[0][0].sum() > 0 and runs[0][3][0, 5] > 0
        for other in runs[1:]:
            for a, b in zip(runs[0], other):
                np.testing.assert_array_equal(a, b)


def test_values_sharing_a_threshold_use_the_map():
    """Two attenuation values closer than a threshold step: one palette code
    for both, so the walk reads the map itself."""
    mc = _mc()
    p = _problem((24, 24, 24), "water", 0.035, 200_000)
    mu = p.mu.copy()
    mu[::2] = np.float32(0.30)
    mu[1::4] = np.nextafter(np.float32(0.02), np.float32(1.0))
    mu[3::4] = np.float32(0.02)
    dp = mc.to_device(p.with_(mu=mu))
    a = mc.simulate(dp, options={"forced_detection": 1})
    b = mc.simulate(dp, options={"forced_detection": 1, "threshold_bytes": 4})
    assert int(a.status[2]) == 1
    np.testing.assert_array_equal(a.tally.cpu().numpy(), b.tally.cpu().numpy())
    np.testing.assert_array_equal(a.tally_sq.cpu().numpy(), b.tally_sq.cpu().numpy())


@pytest.mark.parametrize("angle", [math.pi / 4, 0.6])
def test_rays_past_a_corner_near_the_exit(angle):
    """Rays from the corner voxel that leave the grid within rounding of another
    plane, a fraction of a voxel away: the last planes (multiples of the rounded
    voxel size) lie before the exits (the rounded grid size), so such a walk
    takes a step outside the grid before its last piece.  1.004 cm is a size where 17 voxels differ most from the grid.
    The attenuation is chosen so that the table's padding there, leftover
    bytes of the thresholds, would be taken for the code of a high value."""
    mc = _mc()
    n, vox, v = 17, 1.004, 0x40A8A8          # two bytes of v equal its palette slot
    assert (v * 2654435761 & 0xFFFFFFFF) >> 24 == v & 255 == v >> 8 & 255
    assert float(np.float32(n * vox)) - n * float(np.float32(vox)) > 1.5e-6
    mu = np.zeros((n, n, n), dtype=np.float32)
    mu[:n - 1] = v * 2.0**-10
    mu[0, 0, 0] = 2.0**24 * 2.0**-10
    act = np.zeros((n, n, n), dtype=np.uint32)
    act[-1, -1, -1] = 1
    p = phantoms.Problem(
        name="corner", nx=n, ny=n, nz=n, voxel_cm=vox, mu=mu, activity=act, angles=np.array([angle]), nu=4, nv=32,
        pixel_cm=1.0, radius_cm=phantoms.detector_radius(n, n, vox), accept_half_angle_rad=0.035, e_lo_kev=100.0,
        e_hi_kev=154.0, e_cut_kev=90.0, n_histories=1_000_000_000, seed=5, max_steps=1)
    dp = mc.to_device(p)
    a = mc.simulate(dp, options={"forced_detection": 1})
    b = mc.simulate(dp, options={"forced_detection": 1, "threshold_bytes": 4})
    assert int(a.status[2]) == 1 and int(b.status[2]) == 0 and int(b.tally.sum()) > 0
    np.testing.assert_array_equal(a.tally.cpu().numpy(), b.tally.cpu().numpy())
