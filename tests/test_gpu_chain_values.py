"""Which values of J, and which inverse, a level with chain inverses answers with: values that change between
setups, chain blocks that are singular or badly conditioned although J is not.

The matrices are banded and randomly permuted.  `mates`: unknowns i and i + 50 of every 100 are coupled by
entries of 1 to 2, everything else in the band by noise of size eps.  J then has a condition number below 5,
but the level sets cut through the pairs, so the chain's first blocks have the noise for pivots: singular
for eps = 0, inverses of size 1 / eps otherwise.

Tolerance: Gauss-Jordan with partial pivoting over all rows leaves an error of n u cond(J) relative to the
inverse's largest entry up to its growth factor, here at most 10 (u = 2^-53)."""
import types

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"
N, BAND, U = 700, 60, 2.0 ** -53


def _matrix(kind, eps=0.0, n=N, seed=7):
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), 2 * BAND + 1)
    j = (np.arange(n)[:, None] + np.arange(-BAND, BAND + 1)[None, :]).ravel()
    i, j = i[(j >= 0) & (j < n)], j[(j >= 0) & (j < n)]
    p = rng.permutation(n)
    v = rng.standard_normal(len(i))
    if kind == "plain":
        v += 2.0 * np.sqrt(BAND) * (i == j)
    else:
        v *= eps
        other = np.where(i % 100 < 50, i + 50, i - 50)
        mate = j == np.where(other < n, other, i)
        v[mate] += 1.0 + rng.random(mate.sum())
    J = sp.csr_matrix((v, (p[i], p[j])), shape=(n, n))
    J.sort_indices()
    return J


def _vk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    return vk


def _solver(vk, J):
    lv = types.SimpleNamespace(J=J, P=None, R=None, cell_dofs=np.zeros((1, 1), np.int32), colours=np.zeros(1, np.int32))
    S = vk.Solver([vk.upload_level(lv, DEV)])
    S.vk_set_workspace("f64", 5, device=DEV)
    return S


def _put(S, J):
    S.levels[0]["J"]["val"].copy_(torch.from_numpy(J.data))
    torch.cuda.synchronize()


def _check(S, J):
    """The V-cycle (its coarse solve alone) and the exported inverse against numpy."""
    A = J.toarray()
    n = len(A)
    want = np.linalg.inv(A)
    bound = 10 * n * U * np.linalg.cond(A) * np.abs(want).max()
    b = np.random.default_rng(2).standard_normal(n)
    x = torch.empty(n, dtype=torch.float64, device=DEV)
    S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
    assert np.abs(x.cpu().numpy() - want @ b).max() <= bound * np.abs(b).sum()
    got = torch.empty((n, n), dtype=torch.float64, device=DEV)
    S.vk_get_coarse_inverse(got)
    assert np.abs(got.cpu().numpy() - want).max() <= bound


def _check_known_solution(S, J, units=64):
    """|x - v| <= units u max |G| |J| |v| for J x = J v (64: what a refined inverse is accepted with)."""
    n = J.shape[0]
    v = 1.0 + np.random.default_rng(5).random(n)
    x = torch.empty(n, dtype=torch.float64, device=DEV)
    S.vcycle(torch.from_numpy(J @ v).to(DEV), x, 0, 0)
    G = torch.empty((n, n), dtype=torch.float64, device=DEV)
    S.vk_get_coarse_inverse(G)
    assert np.abs(x.cpu().numpy() - v).max() <= units * U * (np.abs(G.cpu().numpy()) @ (np.abs(J) @ v)).max()


def _chained(S):
    n = S.levels[0]["J"]["n_rows"]
    return S.vk_coarse_plan(0)[1] < 2.0 * n ** 3


@pytest.mark.parametrize("kind", ["plain", "mates"])
def test_solves_use_the_values_of_the_setup(kind):
    """J overwritten after the setup (and the device synchronised), before the first solve: the setup's
    inverse answers, whether its chain holds or a dense inverse takes its place."""
    vk = _vk()
    J = _matrix(kind)
    S = _solver(vk, J)
    S.vanka_setup(0.7, "additive")
    torch.cuda.synchronize()
    other = J.copy()
    other.data = 3.0 * np.random.default_rng(11).standard_normal(len(J.data))
    _put(S, other)
    _check(S, J)
    S.close()


def test_an_unused_setup_leaves_nothing_behind():
    """A setup whose chain failed and that no solve used does not decide how the next one inverts."""
    vk = _vk()
    S = _solver(vk, _matrix("mates"))
    S.vanka_setup(0.7, "additive")
    torch.cuda.synchronize()
    _put(S, _matrix("plain"))
    S.vanka_setup(0.7, "additive")
    assert _chained(S)
    _check(S, _matrix("plain"))
    assert _chained(S)
    S.close()


@pytest.mark.parametrize("graphs", [False, True])
def test_a_failed_chain_decides_for_its_own_setup_only(graphs):
    """Values whose chain fails are inverted densely; the next values get the chain again, eagerly and
    where V-cycles replay a graph recorded under the other inverse."""
    vk = _vk()
    S = _solver(vk, _matrix("plain"))
    S.vk_set_graphs(graphs)
    for kind in ("plain", "mates", "plain", "plain", "mates", "mates", "plain"):
        J = _matrix(kind)
        _put(S, J)
        S.vanka_setup(0.7, "additive")
        for rep in range(3):
            _check(S, J)
            assert _chained(S) == (kind == "plain")
    S.close()


def test_a_failed_chain_among_other_blocks():
    """One block of a level fails its check beside a chained and a dense one: all three answer right, and
    the level is chained again once its values allow it."""
    vk = _vk()
    rng = np.random.default_rng(3)
    small = sp.csr_matrix(rng.standard_normal((150, 150)) + 20 * np.eye(150))
    rows = np.array([0, N, N + 150, N + 150 + 900])
    kinds = ("plain", "mates", "plain")
    Js = [sp.block_diag([_matrix(k), small, _matrix("plain", n=900, seed=8)], format="csr") for k in kinds]
    S = vk.Solver([dict(J=vk.upload_csr(Js[0], DEV), P=None, R=None, groups=[], blocks=rows)])
    S.vk_set_workspace("f64", 5, device=DEV)
    b = rng.standard_normal(rows[-1])
    x = torch.empty(rows[-1], dtype=torch.float64, device=DEV)
    for kind, J in zip(kinds, Js):
        _put(S, J)
        S.vanka_setup(0.7, "additive")
        S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
        assert (S.vk_coarse_plan(0)[1] < 2.0 * (np.diff(rows).astype(float) ** 3).sum()) == (kind == "plain")
        got = x.cpu().numpy()
        for r0, r1 in zip(rows[:-1], rows[1:]):
            A = J[r0:r1, r0:r1].toarray()
            want = np.linalg.inv(A)
            bound = 10 * (r1 - r0) * U * np.linalg.cond(A) * np.abs(want).max()
            assert np.abs(got[r0:r1] - want @ b[r0:r1]).max() <= bound * np.abs(b[r0:r1]).sum()
    S.close()


@pytest.mark.parametrize("eps,chained", [(0.05, True), (1e-2, True), (1e-4, True), (1e-6, True), (1e-9, False)])
def test_badly_conditioned_chain_blocks(eps, chained):
    """Noise for pivots costs a chain log10(1 / eps) and more digits: one refinement gives them back (up to
    eps = 1e-6), or the dense inverse takes its place.  Either way the result is as accurate as
    pivoting over all rows makes it."""
    vk = _vk()
    S = _solver(vk, _matrix("mates", eps))
    J = _matrix("mates", eps)
    for seed in (7, 8):
        _put(S, J)
        S.vanka_setup(0.7, "additive")
        _check(S, J)
        _check_known_solution(S, J)
        assert _chained(S) == chained
        J.data = J.data * (1.0 + 0.25 * np.random.default_rng(seed).random(len(J.data)))  # others of their kind
    S.close()


def test_refined_blocks_of_several_sizes():
    """A refinement beside ordinary chains and beyond 1 024 unknowns (odd sizes: uneven halves)."""
    vk = _vk()
    sizes = (700, 1301, 501)
    rows = np.concatenate([[0], np.cumsum(sizes)])
    J = sp.block_diag([_matrix("mates", 1e-3, n=sizes[0]), _matrix("mates", 1e-2, n=sizes[1], seed=9),
                       _matrix("plain", n=sizes[2], seed=8)], format="csr")
    S = vk.Solver([dict(J=vk.upload_csr(J, DEV), P=None, R=None, groups=[], blocks=rows)])
    S.vk_set_workspace("f64", 5, device=DEV)
    S.vanka_setup(0.7, "additive")
    b = np.random.default_rng(4).standard_normal(rows[-1])
    x = torch.empty(rows[-1], dtype=torch.float64, device=DEV)
    S.vcycle(torch.from_numpy(b).to(DEV), x, 0, 0)
    assert S.vk_coarse_plan(0)[1] < 2.0 * (np.diff(rows).astype(float) ** 3).sum()
    for r0, r1 in zip(rows[:-1], rows[1:]):
        A = J[r0:r1, r0:r1].toarray()
        want = np.linalg.inv(A)
        bound = 10 * (r1 - r0) * U * np.linalg.cond(A) * np.abs(want).max()
        assert np.abs(x.cpu().numpy()[r0:r1] - want @ b[r0:r1]).max() <= bound * np.abs(b[r0:r1]).sum()
    S.close()


def _channel(shape, length, k, nu=1e-3, tau=0.01, seed=1):
    from synth.assemble import assemble_jacobian
    from synth.mesh import StructuredMesh
    from synth.problems import inflow_state
    m = StructuredMesh(shape, (length, 0.41), k, 2)
    J = assemble_jacobian(m, inflow_state(m, 0.3, np.random.default_rng(seed)), nu, tau).tocsr()
    J.sort_indices()
    return J


@pytest.mark.parametrize("shape,length,k,nu", [((8, 2), 3.28, 3, 1.9e-3), ((10, 2), 4.1, 2, 1.2e-3),
                                               ((11, 2), 4.51, 3, 1.3e-3), ((11, 2), 2.255, 2, 1e-3)])
def test_chain_solutions_of_flow_matrices(shape, length, k, nu):
    """Elimination by rows (G J close to I) leaves 1 to 4 u max |G| |J| |v| in a solve with known solution v on
    these matrices, over all rows and in a chain alike; the transposed elimination (J G close to I) up to 27."""
    vk = _vk()
    for seed in range(1, 6):
        J = _channel(shape, length, k, nu, seed=seed)
        S = _solver(vk, J)
        S.vanka_setup(0.7, "additive")
        _check_known_solution(S, J, units=10)
        assert _chained(S)
        S.close()


@pytest.mark.parametrize("tau", [1e-5, 1e-2, 1e2])
def test_chain_of_flow_matrices_whatever_the_time_step(tau):
    """Coarse channel matrices keep their chain at every condition number (1e11 at tau = 1e-5, where any
    inverse in 64 bits leaves |b - J x| of 1e-9 and more), and solve as accurately."""
    vk = _vk()
    J = _channel((11, 2), 2.255, 1, tau=tau)
    S = _solver(vk, J)
    S.vanka_setup(0.7, "additive")
    _check_known_solution(S, J)
    assert _chained(S)
    S.close()
