"""Pivot choice of the patch inversions: the first row of largest |pivot|, compared in full.

The widths take the one-wavefront kernel (2 .. 64; 17 .. 32, 33 .. 48 and 49 .. 64 rows its tile counts) and
the workgroup kernel (84 .. 120: two rows a lane); setup variant 2 the vector kernels where they exist."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


def _inverses(blocks, variant=0):
    """The FP64 patch inverses of disjoint cells with these matrices."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    cells, n_K = blocks.shape[:2]
    n = cells * n_K
    print(f"patch width {n_K}, variant {variant}", flush=True)
    J = sp.block_diag([sp.csr_matrix(b) for b in blocks], format="csr")
    P = sp.csr_matrix(np.ones((n, 3)))
    levels = [dict(J=vk.upload_csr(sp.identity(3, format="csr"), DEV), n_cells=0, n_K=0, cell_dofs=None,
                   colour_cells=None, colour_ptr=np.zeros(1, dtype=np.int32), n_colours=0),
              dict(J=vk.upload_csr(J, DEV), P=vk.upload_csr(P, DEV), R=vk.upload_csr(P.T, DEV), n_cells=cells, n_K=n_K,
                   cell_dofs=torch.arange(n, dtype=torch.int32, device=DEV).reshape(cells, n_K),
                   colour_cells=torch.arange(cells, dtype=torch.int32, device=DEV),
                   colour_ptr=np.array([0, cells], dtype=np.int32), n_colours=1)]
    S = vk.Solver(levels)
    S.vk_set_workspace("f64", 5, device=DEV)
    S.vk_set_setup_variant(variant)
    out = torch.empty((cells, n_K, n_K), dtype=torch.float64, device=DEV)
    try:
        S.vanka_setup(0.7)
        S.vk_get_patch_inverses(1, 0, cells, out)
    finally:
        S.close()
    return out.cpu().numpy()


@pytest.mark.parametrize("n_K", [2, 16, 42, 63, 64, 84, 85, 105, 120])
@pytest.mark.parametrize("at", [0, 1])
def test_largest_pivot_near_the_top_of_the_range(n_K, at):
    """A column with 1 and 1 + 2^-14 beside an entry close to the largest number: eliminating with the larger
    one leaves that entry alone, with the smaller one it overflows.  The inverse's other entries are 0, 1
    or exact to two roundings."""
    b, c = np.ldexp(1.9999, 1023), 1.0 + 2.0 ** -14
    i, j = (0, 1) if at == 0 else (n_K - 2, n_K - 1)
    A = np.eye(n_K)
    A[[i, i, j, j], [i, j, i, j]] = 1.0, b, c, 0.0
    want = np.eye(n_K)
    want[[i, i, j, j], [i, j, i, j]] = 0.0, 1.0 / c, 1.0 / b, -1.0 / c / b
    for variant in (0, 2):
        got = _inverses(A[None], variant)[0]
        assert np.isfinite(got).all()
        assert np.abs(got - want).max() <= 4 * 2.0 ** -53


@pytest.mark.parametrize("n_K", [3, 15, 31, 48, 63, 64, 84, 105, 120])
def test_pivots_tied_in_their_leading_digits(n_K):
    """Columns whose candidates agree in the leading 20 bits and differ in the last ones, some of them exactly
    tied: the error stays that of partial pivoting, 1e3 eps cond (growth of sign matrices ~ n^(2/3))."""
    rng = np.random.default_rng(n_K)
    blocks = []
    while len(blocks) < 5:
        A = np.where(rng.random((n_K, n_K)) < 0.5, -1.0, 1.0) * (1.0 + rng.integers(0, 3, (n_K, n_K)) * 2.0 ** -50)
        if np.linalg.cond(A) < 1e6:
            blocks.append(A)
    blocks = np.stack(blocks)
    want = np.linalg.inv(blocks)
    for variant in (0, 2):
        got = _inverses(blocks, variant)
        err = np.abs(got - want).max(axis=(1, 2)) / np.abs(want).max(axis=(1, 2))
        assert (err <= 1e3 * np.finfo(float).eps * np.array([np.linalg.cond(x) for x in blocks])).all()


@pytest.mark.parametrize("n_K", [3, 48, 64, 85, 120])
@pytest.mark.parametrize("value", [0.0, np.inf, np.nan])
def test_columns_without_a_pivot_are_reported(n_K, value):
    import paper_2210_02690_amd as vk
    rng = np.random.default_rng(n_K)
    A = np.stack([rng.standard_normal((n_K, n_K)) for _ in range(3)])
    if value == 0.0:
        A[1, :, n_K // 2] = 0.0
    else:
        A[1, n_K // 3, n_K // 2] = value
    with pytest.raises(vk.VkError, match="cell 1 on level 1 is singular"):
        _inverses(A)
