"""Row sweeps of dense matrices (MLEM and OSEM) where their tiles can go wrong:
rows around one tile of 2048 entries, several tiles long, empty, and counts of
rows around a workgroup's 256, against the updates written out in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP64 sums in another order, then one rounding to float32 per image value
RTOL = 4e-7


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _matrix(lengths, n_cols, seed):
    import scipy.sparse as sp
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = np.repeat(np.arange(len(lengths)), lengths)
    cols = np.concatenate([rng.choice(n_cols, size=n, replace=False) for n in lengths] + [np.zeros(0, int)])
    vals = rng.uniform(0.1, 1.0, size=len(rows)).astype(np.float32)
    return sp.csr_matrix((vals, (rows, cols)), shape=(len(lengths), n_cols))


def _rows(kind):
    rng = np.random.Generator(np.random.PCG64(7))
    if kind == "tile edges":
        return [2047, 2048, 2049, 0, 1, 4096, 4097, 0, 0, 6000, 3, 2045]
    if kind == "255":
        return list(rng.integers(0, 30, size=255))
    if kind == "256":
        return list(rng.integers(0, 30, size=256))
    if kind == "257":
        return list(rng.integers(0, 30, size=257))
    if kind == "uneven":
        return list((rng.pareto(0.7, size=900) * 4).astype(int).clip(0, 5000))
    if kind == "one row":
        return [5000]
    return [0] * 700 + [3000, 2500] + [0] * 300 + [40] * 130


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("kind", ["tile edges", "255", "256", "257", "uneven", "one row", "gaps"])
def test_sweeps(kind, transpose):
    import torch
    mc = _mc()
    T = _matrix(_rows(kind), 6100 if kind != "255" else 37, 3)
    T = (T.T if transpose else T).tocsr()
    rng = np.random.Generator(np.random.PCG64(11))
    P = rng.uniform(0.0, 5.0, size=T.shape[0]).astype(np.float32)
    m = mc.csr_from_scipy(T)
    m.proj = torch.as_tensor(P, device="cuda")
    T = T.astype(np.float64)
    # MLEM: the dense layout is taken above n_bins + n_vox entries; empty rows
    # and columns pad a matrix that is below it, so both layouts run here
    img = torch.ones(m.n_img, dtype=torch.float32, device="cuda")
    mc.Mlem(m).run(img, 3)
    sens = np.asarray(T.sum(axis=0)).ravel()
    S = np.where(sens > 0, 1.0, 0.0)
    for _ in range(3):
        y = T @ S
        S = np.where(sens > 0, S * (T.T @ np.divide(P, y, out=np.zeros_like(y), where=y > 0)) / np.maximum(sens, 1e-300), 0)
    np.testing.assert_allclose(img.cpu().numpy(), S, rtol=RTOL, atol=0)
    # OSEM on the same rows, as views of one bin each, with a scatter term
    for n_sub, bpv in ((1, 1), (min(3, T.shape[0]), 1)):
        sc = rng.uniform(0.0, 1.0, size=T.shape[0]).astype(np.float32)
        img = torch.ones(m.n_img, dtype=torch.float32, device="cuda")
        mc.osem(m, img, 2, n_sub, bpv, scatter=torch.as_tensor(sc, device="cuda"))
        S = np.where(sens > 0, 1.0, 0.0)
        sub = (np.arange(T.shape[0]) // bpv) % n_sub
        for _ in range(2):
            for k in range(n_sub):
                Tk = T[sub == k]
                y = Tk @ S + sc[sub == k]
                sk = np.asarray(Tk.sum(axis=0)).ravel()
                b = Tk.T @ np.divide(P[sub == k], y, out=np.zeros_like(y), where=y > 0)
                S = np.where(sk > 0, S * b / np.maximum(sk, 1e-300), S)
        np.testing.assert_allclose(img.cpu().numpy(), S, rtol=RTOL, atol=0)


@pytest.mark.parametrize("transpose", [False, True])
def test_sweeps_large(transpose):
    """Above the entry count from which MLEM sweeps tiles whatever the row
    lengths: several rows per tile, uneven, some empty, in thousands of groups."""
    import scipy.sparse as sp
    import torch
    mc = _mc()
    rng = np.random.Generator(np.random.PCG64(17))
    n_rows, n_cols = 300_000, 9973
    lengths = (rng.pareto(1.2, size=n_rows) * 10).astype(int).clip(0, 3000)
    lengths[rng.integers(0, n_rows, size=5000)] = 0
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    k = np.arange(ptr[-1]) - np.repeat(ptr[:-1], lengths)
    cols = (np.repeat(rng.integers(0, n_cols, size=n_rows), lengths) + 7 * k) % n_cols
    T = sp.csr_matrix((rng.uniform(0.1, 1.0, size=ptr[-1]).astype(np.float32), cols, ptr), shape=(n_rows, n_cols))
    T = (T.T if transpose else T).tocsr()
    T.sort_indices()
    assert T.nnz >= 1 << 23
    P = rng.uniform(0.0, 5.0, size=T.shape[0]).astype(np.float32)
    m = mc.csr_from_scipy(T)
    m.proj = torch.as_tensor(P, device="cuda")
    T = T.astype(np.float64)
    Tt = T.T.tocsr()
    img = torch.ones(m.n_img, dtype=torch.float32, device="cuda")
    mc.Mlem(m).run(img, 2)
    sens = np.asarray(T.sum(axis=0)).ravel()
    S = np.where(sens > 0, 1.0, 0.0)
    for _ in range(2):
        y = T @ S
        S = np.where(sens > 0, S * (Tt @ np.divide(P, y, out=np.zeros_like(y), where=y > 0)) / np.maximum(sens, 1e-300), 0)
    np.testing.assert_allclose(img.cpu().numpy(), S, rtol=RTOL, atol=0)
    img = torch.ones(m.n_img, dtype=torch.float32, device="cuda")
    mc.osem(m, img, 1, 2, 1)
    S = np.where(sens > 0, 1.0, 0.0)
    for s in range(2):
        Tk = T[s::2]
        y = Tk @ S
        sk = np.asarray(Tk.sum(axis=0)).ravel()
        b = Tk.T @ np.divide(P[s::2], y, out=np.zeros_like(y), where=y > 0)
        S = np.where(sk > 0, S * b / np.maximum(sk, 1e-300), S)
    np.testing.assert_allclose(img.cpu().numpy(), S, rtol=RTOL, atol=0)
