"""Response-matrix build from a written event list, at the sizes where its tiles
can go wrong (2048 events merged and 4096 sorted per workgroup), against the
counts added up in integers: lists shorter than a tile, around one and two,
runs of one (bin, voxel) and rows of one bin across tiles, filtered classes,
empty and overflowing lists, image factors from single voxels to the whole map."""
import numpy as np
import pytest

import phantoms

pytestmark = pytest.mark.gpu


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _keys(kind, n, n_bins, n_vox, rng):
    """Tally bins (view, class, v, u) and emission voxels of n events."""
    if kind == "one entry":
        return np.full(n, n_bins // 3), np.full(n, n_vox // 2)
    if kind == "one bin":
        return np.full(n, n_bins - 1), rng.integers(0, n_vox, size=n)
    if kind == "runs":
        pick = np.repeat(np.arange(n), rng.integers(1, 900, size=n))[:n]
        return rng.integers(0, n_bins, size=n)[pick], rng.integers(0, n_vox, size=n)[pick]
    return rng.integers(0, n_bins, size=n), rng.integers(0, n_vox, size=n)


@pytest.mark.parametrize("kind,n,cap,f", [
    ("random", 0, 1, 2), ("random", 1, 1, 2), ("random", 2047, 2047, 1), ("random", 2048, 9000, 4),
    ("random", 2049, 4096, 24), ("random", 4095, 4097, 2), ("random", 4097, 4097, 8), ("random", 50_000, 60_000, 3),
    ("one entry", 2048, 5000, 2), ("one entry", 9001, 9001, 2), ("one bin", 8193, 10_000, 2),
    ("runs", 30_000, 30_000, 6), ("random", 3000, 2999, 2)])
def test_matrix_build(kind, n, cap, f):
    import torch
    mc = _mc()
    rng = np.random.Generator(np.random.PCG64(n + 7 * f))
    prob = phantoms.thorax_problem("mb", 24, 1.2, 2, 5, 180.0, 13, 1.2, 100_003, image_factor=f)
    dp = mc.to_device(prob)
    act = rng.integers(1, 2**31, size=24**3)
    dp = dp.with_(activity=torch.as_tensor(act.astype(np.int32).reshape(24, 24, 24), device="cuda"))
    V, _, nv, nu = dp.tally_shape
    sim = mc.Simulator(dp, event_capacity=cap, want_sq=False)
    bins, vox = _keys(kind, n, V * 2 * nv * nu, 24**3, rng)
    w = rng.integers(1, 2**40, size=n)
    order = rng.permutation(n)
    bins, vox, w = bins[order], vox[order], w[order]
    raw = np.zeros((n, 3), dtype=np.int64)
    raw[:, 1] = bins | vox << 32
    raw[:, 2] = w
    sim.events[:min(n, cap)] = torch.as_tensor(raw[:cap], device="cuda")
    sim.n_events.fill_(n)
    if n > cap:
        with pytest.raises(mc.McError):
            mc.system_matrix(dp, sim)
        return

    m_ = 24 // f
    z, y, x = vox // 576, vox // 24 % 24, vox % 24
    img = x // f + m_ * (y // f + m_ * (z // f))
    A = act.reshape(m_, f, m_, f, m_, f).sum(axis=(1, 3, 5)).ravel().astype(np.float64)
    view, cls = bins // (2 * nv * nu), bins // (nv * nu) % 2
    row = view * nv * nu + bins % (nv * nu)
    n_view = 100_003 // V + (np.arange(V) < 100_003 % V)
    for classes, keep in (("all", cls >= 0), ("primary", cls == 0), ("scatter", cls == 1)):
        m = mc.system_matrix(dp, sim, classes)
        key, inv = np.unique(row[keep] * m.n_img + img[keep], return_inverse=True)
        c = np.zeros(len(key), dtype=np.int64)
        np.add.at(c, inv, w[keep])
        r, i = key // m.n_img, key % m.n_img
        val = (c.astype(np.float64) * 2.0**-32 / (n_view[r // (nv * nu)] * A[i] / float(act.sum()))).astype(np.float32)
        P = np.zeros(m.n_bins, dtype=np.int64)
        np.add.at(P, row[keep], w[keep])
        k = m.nnz
        assert k == len(key)
        np.testing.assert_array_equal(m.T_rowptr.cpu().numpy(), np.searchsorted(r, np.arange(m.n_bins + 1)))
        np.testing.assert_array_equal(m.T_col[:k].cpu().numpy(), i)
        np.testing.assert_array_equal(m.T_val[:k].cpu().numpy(), val)
        t = np.argsort(i, kind="stable")
        np.testing.assert_array_equal(m.Tt_rowptr.cpu().numpy(), np.searchsorted(i[t], np.arange(m.n_img + 1)))
        np.testing.assert_array_equal(m.Tt_col[:k].cpu().numpy(), r[t])
        np.testing.assert_array_equal(m.Tt_val[:k].cpu().numpy(), val[t])
        np.testing.assert_array_equal(m.proj.cpu().numpy(), (P.astype(np.float64) * 2.0**-32).astype(np.float32))
