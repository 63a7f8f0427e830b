"""OSEM's sweeps where the shape of their work can go wrong, against the update
written out in float64: a dual matrix whose two parts ask for other numbers of
lanes per row (each pair of 1, 4, 16 and 64, and tiles), and tiles of several
rows of a view with a short last chunk, empty bins beside full ones and
subsets that do not divide the views."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP64 sums in another order, then one rounding to float32 per image value
RTOL = 4e-7


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _matrix(n_rows, n_cols, mean, seed):
    """Rows of 0 to about 4 mean entries, a tenth of them empty."""
    import scipy.sparse as sp
    rng = np.random.Generator(np.random.PCG64(seed))
    lengths = np.minimum(rng.exponential(mean, size=n_rows).astype(int) + 1, min(n_cols, 4 * mean + 2))
    lengths[rng.random(n_rows) < 0.1] = 0
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    k = np.arange(ptr[-1]) - np.repeat(ptr[:-1], lengths)
    cols = (np.repeat(rng.integers(0, n_cols, size=n_rows), lengths) + 7 * k) % n_cols
    T = sp.csr_matrix((rng.uniform(0.1, 1.0, size=ptr[-1]).astype(np.float32), cols, ptr), shape=(n_rows, n_cols))
    T.sort_indices()
    return T


def _osem(C, B, P, sc, n_iter, n_sub, bpv):
    C, B = C.astype(np.float64), B.astype(np.float64)
    sub = (np.arange(C.shape[0]) // bpv) % n_sub
    sens = [np.asarray(B[sub == k].sum(axis=0)).ravel() for k in range(n_sub)]
    S = np.where(sum(sens) > 0, 1.0, 0.0)
    for _ in range(n_iter):
        for k in range(n_sub):
            y = C[sub == k] @ S + sc[sub == k]
            r = np.divide(P[sub == k], y, out=np.zeros_like(y), where=y > 0)
            S = np.where(sens[k] > 0, S * (B[sub == k].T @ r) / np.maximum(sens[k], 1e-300), S)
    return S


def _check(C, B, n_iter, n_sub, bpv):
    import torch
    mc = _mc()
    rng = np.random.Generator(np.random.PCG64(11))
    P = rng.uniform(0.0, 5.0, size=C.shape[0]).astype(np.float32)
    sc = rng.uniform(0.0, 1.0, size=C.shape[0]).astype(np.float32)
    c = mc.csr_from_scipy(C)
    b = c if B is C else mc.csr_from_scipy(B)
    img = torch.ones(c.n_img, dtype=torch.float32, device="cuda")
    mc.osem(c, img, n_iter, n_sub, bpv, b=b, proj=torch.as_tensor(P, device="cuda"),
            scatter=torch.as_tensor(sc, device="cuda"))
    np.testing.assert_allclose(img.cpu().numpy(), _osem(C, B, P, sc, n_iter, n_sub, bpv), rtol=RTOL, atol=0)


@pytest.mark.parametrize("mean_b", [1, 8, 40, 150, 600])
@pytest.mark.parametrize("mean_c", [1, 8, 40, 150, 600])
def test_dual_densities(mean_c, mean_b):
    views, bpv, n_vox = 7, 131, 1900
    C = _matrix(views * bpv, n_vox, mean_c, 3 + mean_c)
    B = _matrix(views * bpv, n_vox, mean_b, 5 + mean_b)
    _check(C, B, 2, 3, bpv)


@pytest.mark.parametrize("n_sub", [1, 6])
def test_tiles_of_a_view(n_sub):
    views, bpv, n_vox = 23, 13_001, 9973
    C = _matrix(views * bpv, n_vox, 34, 2)
    assert C.nnz >= 1 << 23 and bpv % (8 * 256 * 3 // 4 // (C.nnz // (views * bpv))) != 0
    _check(C, C, 1, n_sub, bpv)
