"""Products with a grouped matrix whose two-row groups have 1 to 70 entries (every remainder of the
8-lane kernel's pairs of entries), with stretches of single rows and one-entry rows among them, against
scipy.

Tolerance: a row's sum of m products in any order is within (m + 2) eps sum |a x| of the exact one; scipy's
own sum is held to the same bound."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


def _matrix(seed, n_pairs, mixed):
    """Rows 2 i and 2 i + 1 share their columns up to shifts by one; mixed: of 11 pairs the rows
    of one differ (single rows) and two times two have the same columns (groups of four)."""
    rng = np.random.default_rng(seed)
    n = 2 * n_pairs
    rows, cols = [], []
    for i in range(n_pairs):
        m = 2 + i % 69 if not mixed else 1 + i % 70
        # even columns in ascending order, the rows' own one among them
        lo = 2 * min(max(i - 3 * m, 0), n_pairs - 8 * m) if n_pairs > 8 * m else 0
        c = lo + 2 * np.sort(rng.choice(min(8 * m, n_pairs), m, replace=False))
        c[min(np.searchsorted(c, 2 * i), m - 1)] = 2 * i
        c = np.unique(c)
        if len(c) < 2 and not mixed:
            c = np.unique(np.append(c, (2 * i + 2) % n))
        d = rng.integers(0, 2, len(c))
        d[c == 2 * i] = 1
        c1 = c + d
        if mixed and i % 11 == 0:
            c1 = np.append(c1[:-1], 2 * i + 1) if len(c1) > 1 else c1
            c1 = np.unique(c1)
        if mixed and i % 11 in (2, 3, 6, 7):  # four rows with the same columns
            c = c1 = quad if i % 11 in (3, 7) else c
            quad = c
        rows += [np.full(len(c), 2 * i), np.full(len(c1), 2 * i + 1)]
        cols += [c, c1]
    r, c = np.concatenate(rows), np.concatenate(cols)
    return sp.csr_matrix((rng.standard_normal(len(r)), (r, c)), shape=(n, n))


@pytest.mark.parametrize("mixed", [False, True])
def test_grouped_pairs(mixed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    J = _matrix(3 + mixed, 66000, mixed)
    n = J.shape[0]
    assert J.nnz >= 4 << 20
    print(f"mixed {mixed}: {n} rows, {J.nnz} entries", flush=True)
    rng = np.random.default_rng(5)
    diag = np.abs(J.diagonal())
    dofs = np.argsort(-diag)[:4].reshape(4, 1).astype(np.int32)
    P = sp.csr_matrix((np.ones(n), (np.arange(n), np.arange(n) % 3)), shape=(n, 3))
    levels = [dict(J=vk.upload_csr(sp.identity(3, format="csr"), DEV), n_cells=0, n_K=0, cell_dofs=None,
                   colour_cells=None, colour_ptr=np.zeros(1, dtype=np.int32), n_colours=0),
              dict(J=vk.upload_csr(J, DEV), P=vk.upload_csr(P, DEV), R=vk.upload_csr(sp.csr_matrix(P.T), DEV),
                   n_cells=4, n_K=1, cell_dofs=torch.from_numpy(dofs).to(DEV),
                   colour_cells=torch.arange(4, dtype=torch.int32, device=DEV),
                   colour_ptr=np.arange(5, dtype=np.int32), n_colours=4)]
    S = vk.Solver(levels)
    S.vk_set_workspace("f64", 5, device=DEV)
    S.vanka_setup(0.7, "additive")
    assert S.vk_spmv_format(1) > 0
    x, z = rng.standard_normal(n), rng.standard_normal(n)
    xt, zt = torch.from_numpy(x).to(DEV), torch.from_numpy(z).to(DEV)
    y = torch.empty_like(xt)
    bound = 2 * (np.diff(J.indptr) + 4) * np.finfo(float).eps * (abs(J) @ abs(x) + abs(z))
    for lanes in (8, 16):
        S.vk_set_spmv_format(lanes)
        assert S.vk_spmv_format(1) == lanes
        S.vk_spmv(1, xt, y)
        assert (np.abs(y.cpu().numpy() - J @ x) <= bound).all(), lanes
        S.vk_spmv(1, xt, y, alpha=-1.0, beta=1.0, z=zt)
        assert (np.abs(y.cpu().numpy() - (z - J @ x)) <= bound).all(), lanes
    S.close()
