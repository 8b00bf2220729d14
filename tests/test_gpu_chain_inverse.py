"""Dense inverses of directly solved blocks through a chain of small blocks, against numpy.

Tolerance: both eliminations are backward stable up to their growth factors; with chain blocks of random
diagonally weighted matrices (growth a few units) the error relative to the inverse's largest entry is
below 1e3 eps cond(J).  The fallback's matrices are inverted by Gauss-Jordan with partial pivoting over
all rows and get the same bound."""
import types

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


def _banded(n, band, seed, weight=2.0, zero=0):
    """A randomly permuted banded matrix; zero: the leading principal submatrix of that size is stored as
    zeros."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), 2 * band + 1)
    j = (np.arange(n)[:, None] + np.arange(-band, band + 1)[None, :]).ravel()
    k = (j >= 0) & (j < n)
    i, j = i[k], j[k]
    v = rng.standard_normal(len(i)) + weight * np.sqrt(band) * (i == j)
    v[(i < zero) & (j < zero)] = 0.0
    p = rng.permutation(n)
    return sp.csr_matrix((v, (p[i], p[j])), shape=(n, n))


def _solver(vk, J):
    lv = types.SimpleNamespace(J=J, P=None, R=None, cell_dofs=np.zeros((1, 1), np.int32), colours=np.zeros(1, np.int32))
    S = vk.Solver([vk.upload_level(lv, DEV)])
    S.vk_set_workspace("f64", 5, device=DEV)
    return S


def _inverse(S, n):
    out = torch.empty((n, n), dtype=torch.float64, device=DEV)
    S.vk_get_coarse_inverse(out)
    return out.cpu().numpy()


def _vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    return vk


# chain blocks of 64 to 176 rows (matrix-core kernel of several tile counts), and beyond 176 (two and more
# pieces); 384: the narrowest block that is chained
@pytest.mark.parametrize("n,band", [(384, 9), (500, 17), (889, 33), (1000, 47), (1301, 85), (2000, 88), (2000, 150), (2000, 190), (2600, 310)])
def test_chain_inverse(n, band):
    vk = _vk()
    print(f"chain inverse n {n} band {band}", flush=True)
    J = _banded(n, band, n + band)
    A = J.toarray()
    want = np.linalg.inv(A)
    bound = 1e3 * np.finfo(float).eps * np.linalg.cond(A) * np.abs(want).max()
    S = _solver(vk, J)
    b = np.random.default_rng(2).standard_normal(n)
    x = torch.empty(n, dtype=torch.float64, device=DEV)
    for solver in (0, 1, 0):
        S.vk_set_coarse_solver(solver)
        for rep in range(2):
            S.vanka_setup(0.7, "additive")
            nb, flops = S.vk_coarse_plan(0)
            assert nb == 0 and ((flops < 2.0 * n ** 3) if solver == 0 else (flops == 2.0 * n ** 3))
            S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
            assert np.abs(x.cpu().numpy() - want @ b).max() <= bound * np.abs(b).sum()
            assert np.abs(_inverse(S, n) - want).max() <= bound
    S.close()


def test_chain_falls_back_to_the_dense_inverse():
    """A regular matrix whose first and last chain blocks are singular (40 x 40 zeros in blocks of 64 to 100
    rows) is inverted densely, and stays so; values with a good chain afterwards stay right too."""
    vk = _vk()
    n, band = 700, 60
    J = _banded(n, band, 7, zero=60)
    A = J.toarray()
    want = np.linalg.inv(A)
    bound = 1e3 * np.finfo(float).eps * np.linalg.cond(A) * np.abs(want).max()
    S = _solver(vk, J)
    b = np.random.default_rng(2).standard_normal(n)
    for rep in range(2):
        S.vanka_setup(0.7, "additive")
        x = torch.empty(n, dtype=torch.float64, device=DEV)
        S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
        assert np.abs(x.cpu().numpy() - want @ b).max() <= bound * np.abs(b).sum()
        assert S.vk_coarse_plan(0)[1] == 2.0 * n ** 3
        assert np.abs(_inverse(S, n) - want).max() <= bound
    S.close()


def test_chain_singular_matrix_reported():
    vk = _vk()
    J = _banded(600, 30, 9)
    J.data[J.indptr[123]:J.indptr[124]] = 0.0
    S = _solver(vk, J)
    S.vanka_setup(0.7, "additive")
    x = torch.zeros(600, dtype=torch.float64, device=DEV)
    with pytest.raises(vk.VkError, match="singular"):
        S.vcycle(torch.ones(600, dtype=torch.float64, device=DEV), x, 0, 0)
    S.close()


# 1 025 to 1 536 rows: three panel rows a thread (dense solver)
@pytest.mark.parametrize("n", [1025, 1100, 1536])
def test_dense_inverse_three_rows_a_thread(n):
    vk = _vk()
    A = np.random.default_rng(n).standard_normal((n, n)) + np.sqrt(n) * np.eye(n)
    want = np.linalg.inv(A)
    S = _solver(vk, sp.csr_matrix(A))
    S.vanka_setup(0.7, "additive")
    assert S.vk_coarse_plan(0) == (0, 2.0 * n ** 3)
    assert np.abs(_inverse(S, n) - want).max() <= 1e3 * np.finfo(float).eps * np.linalg.cond(A) * np.abs(want).max()
    S.close()


def test_chain_blocks_of_one_level():
    """Chained and dense blocks of different widths on one level, solved together."""
    vk = _vk()
    parts = [_banded(700, 20, 1), _banded(300, 20, 2), sp.csr_matrix(np.random.default_rng(3).standard_normal((450, 450)) +
                                                                     20 * np.eye(450)),
             _banded(1300, 40, 4), _banded(50, 5, 5)]
    J = sp.block_diag(parts, format="csr")
    n = J.shape[0]
    rows = np.concatenate([[0], np.cumsum([p.shape[0] for p in parts])])
    S = vk.Solver([dict(J=vk.upload_csr(J, DEV), P=None, R=None, groups=[], blocks=rows)])
    S.vk_set_workspace("f64", 5, device=DEV)
    S.vanka_setup(0.7, "additive")
    assert S.vk_coarse_plan(0)[1] < 2.0 * (np.diff(rows).astype(float) ** 3).sum()
    b = np.random.default_rng(6).standard_normal(n)
    x = torch.empty(n, dtype=torch.float64, device=DEV)
    S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
    got = x.cpu().numpy()
    for p, r0, r1 in zip(parts, rows[:-1], rows[1:]):
        A = p.toarray()
        want = np.linalg.solve(A, b[r0:r1])
        bound = 1e3 * np.finfo(float).eps * np.linalg.cond(A) * np.linalg.norm(np.linalg.inv(A), 2) * np.linalg.norm(b[r0:r1])
        assert np.linalg.norm(got[r0:r1] - want) <= bound
    S.close()
