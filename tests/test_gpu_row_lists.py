"""The lists of non-empty rows that MLEM sweeps on dense matrices, where they
can go wrong: rows around one and two chunks of 4096, whole chunks empty, rows
only at the ends, lists longer than one pass scans (8.4e6 rows), and each
number of lanes per row, against the update written out in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP64 sums in another order, then one rounding to float32 per image value
RTOL = 4e-7


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _matrix(n_rows, n_cols, live, mean, seed):
    """Rows `live` of n_rows with 1 to 2 mean - 1 entries (mean on average)."""
    import scipy.sparse as sp
    rng = np.random.Generator(np.random.PCG64(seed))
    lengths = np.zeros(n_rows, dtype=np.int64)
    lengths[live] = rng.integers(1, 2 * mean, size=len(live))
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    k = np.arange(ptr[-1]) - np.repeat(ptr[:-1], lengths)
    cols = (np.repeat(rng.integers(0, n_cols, size=n_rows), lengths) + 7 * k) % n_cols
    T = sp.csr_matrix((rng.uniform(0.1, 1.0, size=ptr[-1]).astype(np.float32), cols, ptr), shape=(n_rows, n_cols))
    T.sort_indices()
    return T


def _live(kind, n):
    if kind == "all":
        return np.arange(n)
    if kind == "ends":
        return np.r_[:40, n - 60:n]
    if kind == "one chunk of three":
        return np.arange(5000, 6000)
    return np.flatnonzero(np.random.Generator(np.random.PCG64(5)).random(n) < 0.3)


CASES = [(4095, "all", 3, 700), (4096, "all", 6, 700), (4097, "all", 30, 1000), (8193, "third", 20, 3000),
         (9000, "ends", 150, 1500), (12288, "one chunk of three", 40, 2000), (70_000, "third", 200, 5000),
         (8_400_000, "all", 2, 33_000)]


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("n_rows,kind,mean,n_cols", CASES)
def test_lists(n_rows, kind, mean, n_cols, transpose):
    import torch
    mc = _mc()
    T = _matrix(n_rows, n_cols, _live(kind, n_rows), mean, n_rows + mean)
    assert T.nnz > n_rows + n_cols                    # not the compact layout
    T = (T.T if transpose else T).tocsr()
    T.sort_indices()
    P = np.random.Generator(np.random.PCG64(11)).uniform(0.0, 5.0, size=T.shape[0]).astype(np.float32)
    m = mc.csr_from_scipy(T)
    m.proj = torch.as_tensor(P, device="cuda")
    T = T.astype(np.float64)
    Tt = T.T.tocsr()
    sens = np.asarray(T.sum(axis=0)).ravel()
    S = np.where(sens > 0, 1.0, 0.0)
    for _ in range(2):
        y = T @ S
        S = np.where(sens > 0, S * (Tt @ np.divide(P, y, out=np.zeros_like(y), where=y > 0)) / np.maximum(sens, 1e-300), 0)
    solver = mc.Mlem(m)
    for _ in range(2):                                # the lists serve every call
        img = torch.ones(m.n_img, dtype=torch.float32, device="cuda")
        solver.run(img, 2)
        np.testing.assert_allclose(img.cpu().numpy(), S, rtol=RTOL, atol=0)
