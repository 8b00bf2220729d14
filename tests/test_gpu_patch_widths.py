"""Patch inverses of every tile remainder of the one-wavefront matrix-core kernel (widths 1 .. 64) and of the
blocked kernels (200 .. 512), on random sparse matrices whose pivots lie off the diagonal, against numpy.

Tolerance: Gauss-Jordan with partial pivoting is backward stable up to the growth factor, so the error
relative to the inverse's largest entry is below c eps cond with c = 1e3 (n <= 64, growth of random
matrices ~ n^(2/3)); the vector kernels (setup variant 2) get the same bound."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


def _levels(vk, n_K, cells):
    rng = np.random.default_rng(n_K)
    n = 3 * n_K + 5
    J = np.where(rng.random((n, n)) < 0.7, rng.standard_normal((n, n)), 0.0)
    J[np.arange(n), (np.arange(n) + 1) % n] += 1.0
    J[np.arange(n), np.arange(n)] += 0.5 * (rng.random(n) < 0.3)
    dofs = np.stack([rng.permutation(n)[:n_K] for _ in range(cells)]).astype(np.int32)
    for c in range(cells):  # a nonsingular patch whose pivots are off its diagonal
        J[dofs[c], np.roll(dofs[c], 1)] += 2.0 * np.sqrt(n_K)
    P = sp.csr_matrix(rng.standard_normal((n, 3)))
    levels = [dict(J=vk.upload_csr(sp.identity(3, format="csr"), DEV), n_cells=0, n_K=0, cell_dofs=None,
                   colour_cells=None, colour_ptr=np.zeros(1, dtype=np.int32), n_colours=0),
              dict(J=vk.upload_csr(sp.csr_matrix(J), DEV), P=vk.upload_csr(P, DEV), R=vk.upload_csr(P.T, DEV),
                   n_cells=cells, n_K=n_K, cell_dofs=torch.from_numpy(dofs).to(DEV),
                   colour_cells=torch.arange(cells, dtype=torch.int32, device=DEV),
                   colour_ptr=np.arange(cells + 1, dtype=np.int32), n_colours=cells)]
    return levels, np.stack([J[np.ix_(d, d)] for d in dofs])


@pytest.mark.parametrize("n_K", [1, 2, 4, 12, 13, 15, 16, 17, 29, 32, 33, 47, 48, 49, 60, 61, 64])
def test_narrow_patch_inverses(n_K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"patch width {n_K}", flush=True)
    cells = 7
    levels, blocks = _levels(vk, n_K, cells)
    want = np.linalg.inv(blocks)
    tol = 1e3 * np.finfo(float).eps * np.array([np.linalg.cond(b) for b in blocks])
    S = vk.Solver(levels)
    for prec, unit in (("f64", 0.0), ("f32", 2.0 ** -24), ("bf16", 2.0 ** -8)):
        for variant in (0, 2):
            S.vk_set_workspace(prec, 5, device=DEV)
            S.vk_set_setup_variant(variant)
            S.vanka_setup(0.7)
            out = torch.empty((cells, n_K, n_K), dtype=torch.float64, device=DEV)
            S.vk_get_patch_inverses(1, 0, cells, out)
            err = np.abs(out.cpu().numpy() - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
            assert (err <= tol + unit).all(), (prec, variant, err.max())


# the gather of the dense patches takes 16 rows a pass while they fit 64 KB of LDS, 8 beyond
@pytest.mark.parametrize("n_K", [200, 255, 256, 467, 468, 469, 512])
def test_blocked_patch_inverses(n_K):
    """Growth of partial pivoting ~ n^(2/3) <= 64 for n <= 512, an order of magnitude above the narrow
    patches': 1e4 eps cond."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"patch width {n_K}", flush=True)
    cells = 3
    levels, blocks = _levels(vk, n_K, cells)
    want = np.linalg.inv(blocks)
    tol = 1e4 * np.finfo(float).eps * np.array([np.linalg.cond(b) for b in blocks])
    S = vk.Solver(levels)
    for prec, unit in (("f64", 0.0), ("f32", 2.0 ** -24)):
        S.vk_set_workspace(prec, 5, device=DEV)
        S.vanka_setup(0.7)
        out = torch.empty((cells, n_K, n_K), dtype=torch.float64, device=DEV)
        S.vk_get_patch_inverses(1, 0, cells, out)
        err = np.abs(out.cpu().numpy() - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
        assert (err <= tol + unit).all(), (prec, err.max())
    S.close()


# one and the last width of every tile count of the workgroup's matrix-core kernel, 177 the first beyond it
@pytest.mark.parametrize("n_K", [65, 80, 81, 96, 97, 112, 113, 126, 128, 129, 144, 145, 160, 161, 169, 171, 176, 177])
def test_workgroup_patch_inverses(n_K):
    """Growth of partial pivoting ~ n^(2/3) <= 32: twice the narrow patches', 2e3 eps cond."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"patch width {n_K}", flush=True)
    cells = 5
    levels, blocks = _levels(vk, n_K, cells)
    want = np.linalg.inv(blocks)
    tol = 2e3 * np.finfo(float).eps * np.array([np.linalg.cond(b) for b in blocks])
    S = vk.Solver(levels)
    for prec, unit in (("f64", 0.0), ("f32", 2.0 ** -24), ("bf16", 2.0 ** -8)):
        S.vk_set_workspace(prec, 5, device=DEV)
        for rep in range(2):
            S.vanka_setup(0.7)
            out = torch.empty((cells, n_K, n_K), dtype=torch.float64, device=DEV)
            S.vk_get_patch_inverses(1, 0, cells, out)
            err = np.abs(out.cpu().numpy() - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
            assert (err <= tol + unit).all(), (prec, err.max())
    S.close()
