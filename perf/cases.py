"""The work that users of this solver have it do, as timed cases.

Sizes are those of the repository's own workloads (the 44 x 8 ... 176 x 32 channels and the 100 x 16 x 16
box of `synth.problems`, the 88 x 16 and 48 x 8 x 8 meshes of the robustness study, the 64-channel batch, the
88 x 16 learned guess) and, for drawn cases, other meshes of the same family.  Every system is a Newton
linearisation of a channel or box flow about a parabolic inflow profile with 5 % noise, as `synth.problems`
builds it; the matrices are assembled on the GPU here, from element matrices of `synth.assemble`, so that new
inputs are quick to make.  The mesh (patterns, transfers, cell maps) does not depend on the seed; the states,
hence every matrix value, and the right-hand sides do.

Kinds of cases:
  sweep    vanka_smooth on the finest level: the smoother alone, as a caller's own multigrid uses it
  vcycle   one V-cycle: the preconditioner alone, as a caller's own Krylov method uses it
  newton   one Newton step: vanka_setup on new matrices, then gmres_solve to 1e-8 (bench.py's step)
  batch    the same for many independent systems in one context (gmres_solve_batched)
  train    one optimiser step of the learned guess's network (a minibatch of 512 cells)
  predict  the learned guess of one slab: extrapolations, patch features, network, DoF averages
"""
import functools

import numpy as np
import torch

import paper_2210_02690_amd as vk
from synth.assemble import element_matrices, local_pattern
from synth.batch import batch_shapes, draw_systems
from synth.learned import N_HIDDEN, WIDTH, init_mlp_params
from synth.mesh import StructuredMesh, hierarchy_shapes
from synth.problems import H_CHANNEL, inflow_state
from synth.radau import dg_time_matrices
from synth.transfer import inject_nodes, prolongation

DEV = "cuda:0"
OMEGA, TAU, NU, NU_SWEEPS, RESTART = 0.7, 0.01, 1e-3, (2, 2), 30
PREC_BYTES = {"f64": 8, "f32": 4, "bf16": 2}


def listed():
    two = dict(r=2, mode="additive", tuned=False)
    return [
        # the smallest smoother call: everything fits a cache, only latency and launches count
        dict(name="sweep_44x8_k1", kind="sweep", shape="44x8", levels=3, k=1, prec="f64", sweeps=2, **two),
        # the multiplicative smoother on an odd mesh, dG(3): one launch pair per colour
        dict(name="sweep_mult_60x12_k3", kind="sweep", shape="60x12", levels=3, k=3, prec="f64", sweeps=2, r=2,
             mode="multiplicative", tuned=False),
        # a 3D smoother call on matrices well beyond the caches
        dict(name="sweep_48x16x16_k1", kind="sweep", shape="48x16x16", levels=4, k=1, prec="f64", sweeps=2, **two),
        # the preconditioner of an ordinary 2D system, and of a 3D one with dG(0)
        dict(name="vcycle_88x16_k1", kind="vcycle", shape="88x16", levels=4, k=1, prec="f64", **two),
        dict(name="vcycle_48x8x8_k0", kind="vcycle", shape="48x8x8", levels=4, k=0, prec="f64", **two),
        # Newton steps: the marching workload's mesh with the smallest storage, the 2D headline, the
        # (Q4)^2/P3disc element of the 2D study, the widest 3D patches of the study, the 3D headline
        dict(name="newton_88x16_k1_bf16", kind="newton", shape="88x16", levels=4, k=1, prec="bf16", **two),
        dict(name="newton_176x32_k2_f32", kind="newton", shape="176x32", levels=5, k=2, prec="f32", r=2,
             mode="additive", tuned=True),
        dict(name="newton_88x16_q4_k1_f64", kind="newton", shape="88x16", levels=4, k=1, prec="f64", r=4,
             mode="additive", tuned=False),
        dict(name="newton_48x8x8_k2_f32", kind="newton", shape="48x8x8", levels=4, k=2, prec="f32", **two),
        dict(name="newton_100x16x16_k1_f32", kind="newton", shape="100x16x16", levels=4, k=1, prec="f32", r=2,
             mode="additive", tuned=True),
        # the batch of independent channels, graph replay on
        dict(name="batch_64_f32", kind="batch", systems=64, draw=0, prec="f32"),
        # training of the learned guess (its prediction is among the drawn cases)
        dict(name="train_88x16_k1", kind="train", cells=1408, n_K=42, batch=512),
    ]


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "vcycle", "vcycle", "newton", "newton", "newton", "batch", "train", "predict"])
    if kind == "batch":
        return dict(kind=kind, systems=int(round(2 ** rng.uniform(2, 5))), draw=rng.randrange(1, 1000),
                    prec=rng.choice(["f32", "f64"]))
    if kind == "train":
        return dict(kind=kind, cells=rng.randrange(300, 3000), n_K=rng.choice([21, 42, 63, 84]),
                    batch=int(round(2 ** rng.uniform(6, 11))))
    if kind == "predict":
        return dict(kind=kind, shape="%dx%d" % (rng.randrange(20, 180), rng.randrange(7, 33)), k=rng.choice([0, 1, 2, 3]))
    prec = "f64" if kind != "newton" else rng.choice(["f64", "f32", "f32", "bf16"])
    mode = "multiplicative" if kind == "sweep" and rng.random() < 0.25 else "additive"
    if rng.random() < 0.3:   # a box: odd coarse counts, two or three levels
        levels = rng.choice([2, 3])
        c = (rng.randrange(3, 8 if levels == 3 else 13), rng.choice([2, 2, 3]), 2)
        k, r = rng.choice([0, 1, 1, 2]) if levels == 2 else rng.choice([0, 1]), 2
    else:
        levels = rng.choice([2, 3, 4])
        c = (rng.randrange(5, 14), rng.choice([2, 2, 3]))
        k, r = rng.choice([0, 1, 1, 2, 2, 3, 4]), 2
        if rng.random() < 0.15 and levels < 4:
            k, r = rng.choice([0, 1]), 4
    case = dict(kind=kind, shape="x".join(str(v << (levels - 1)) for v in c), levels=levels, k=k, prec=prec, r=r,
                mode=mode, tuned=False)
    if kind == "sweep":
        case["sweeps"] = rng.choice([1, 2, 4])
    return case


# ---- inputs ---------------------------------------------------------------------------------------------------


class MeshLevel:
    """What one mesh level holds on the GPU whatever the state: the CSR pattern of J, the position in it of
    every element entry, the element matrices of a zero state (per boundary class of cells) and their linear
    dependence on the state's values at the cell's nodes."""

    def __init__(self, shape, lengths, k, r, nu, coarse):
        m = self.mesh = StructuredMesh(shape, lengths, k, r)
        n, nv, ns = m.n, m.d * m.n_loc_nodes, m.n_loc_space
        li, lj = np.nonzero(local_pattern(m))
        dofs = torch.from_numpy(m.cell_dofs().astype(np.int64)).to(DEV)
        keys = dofs[:, torch.from_numpy(li).to(DEV)] * n + dofs[:, torch.from_numpy(lj).to(DEV)]
        uniq, pos = torch.unique(keys, return_inverse=True)
        del keys
        self.pos = pos
        self.col = (uniq % n).to(torch.int32)
        self.row_ptr = torch.searchsorted(uniq, torch.arange(n + 1, device=DEV) * n)
        self.nnz = uniq.numel()
        # constant part: one cell of each boundary class, on a mesh of at most three cells a side
        small = tuple(min(s, 3) for s in m.shape)
        t = StructuredMesh(small, [h * s for h, s in zip(m.h, small)], k, r)
        zero = np.zeros((m.n_time, t.n_nodes, m.d))
        E0 = element_matrices(t, zero, nu, TAU)
        ci = m.cell_index()
        cls = [np.where(ci[:, i] == 0, 0, np.where(ci[:, i] == m.shape[i] - 1, small[i] - 1, 1)) for i in range(m.d)]
        self.cls = torch.from_numpy(np.ravel_multi_index(cls, small, order="F")).to(DEV)
        self.const = torch.from_numpy(E0[:, li, lj]).to(DEV)
        # the state's part, the same for every cell: unit states on a mesh of one cell
        one = StructuredMesh((1,) * m.d, m.h, k, r)
        base = element_matrices(one, np.zeros((m.n_time, one.n_nodes, m.d)), nu, TAU)[0][:nv, :nv]
        unit = np.zeros((nv, nv * nv))
        for i in range(nv):
            V = np.zeros((m.n_time, one.n_nodes, m.d))
            V[0, one.cell_nodes()[0, i // m.d], i % m.d] = 1.0
            unit[i] = (element_matrices(one, V, nu, TAU)[0][:nv, :nv] - base).ravel()
        self.unit = torch.from_numpy(unit).to(DEV)
        at = {(i, j): e for e, (i, j) in enumerate(zip(li, lj))}
        self.entries = [torch.tensor([at[a * ns + i, a * ns + j] for i in range(nv) for j in range(nv)], device=DEV)
                        for a in range(m.n_time)]
        w = dg_time_matrices(k)[1]
        self.weight = w / w[0]
        self.nodes = torch.from_numpy(m.cell_nodes()).to(DEV)
        # cells by colour, for the solver and for the assembly (cells of one colour share no entry)
        colours = m.colours()
        order = np.argsort(colours, kind="stable")
        self.ptr = np.concatenate([[0], np.cumsum(np.bincount(colours, minlength=m.n_colours))]).astype(np.int32)
        self.order = torch.from_numpy(order).to(DEV)
        self.fixed = dict(n_cells=m.n_cells, n_K=m.n_K, cell_dofs=dofs.to(torch.int32), P=None, R=None,
                          colour_cells=self.order.to(torch.int32), colour_ptr=self.ptr, n_colours=m.n_colours)
        self.inject = None
        if coarse is not None:
            P = prolongation(coarse.mesh, m)
            self.fixed.update(P=vk.upload_csr(P, DEV), R=vk.upload_csr(P.T.tocsr(), DEV))
            self.inject = torch.from_numpy(inject_nodes(coarse.mesh, m)).to(DEV)

    def values(self, V):
        """CSR values of J at the state V (n_time x n_nodes x d, on the GPU)."""
        data = self.const[self.cls]
        for a in range(self.mesh.n_time):
            Va = V[a][self.nodes].reshape(self.mesh.n_cells, -1)
            data[:, self.entries[a]] += (Va @ self.unit) * float(self.weight[a])
        val = torch.zeros(self.nnz, dtype=torch.float64, device=DEV)
        for c in range(self.mesh.n_colours):
            cells = self.order[int(self.ptr[c]):int(self.ptr[c + 1])]
            val[self.pos[cells]] += data[cells]
        return val

    def csr(self, val):
        n = self.mesh.n
        return dict(n_rows=n, n_cols=n, row_ptr=self.row_ptr, col=self.col, val=val)


@functools.lru_cache(maxsize=None)
def _meshes(shapes, lengths, k, r, nu):
    out = []
    for s in shapes:
        out.append(MeshLevel(s, lengths, k, r, nu, out[-1] if out else None))
    return out


def _levels(shapes, k, r, nu, seed):
    """(meshes, level dicts) of one system, coarsest first: cells are squares or cubes."""
    fine = shapes[-1]
    lengths = (H_CHANNEL * fine[0] / fine[1],) + tuple(H_CHANNEL * s / fine[1] for s in fine[1:])
    meshes = _meshes(tuple(shapes), lengths, k, r, nu)
    U = 0.3 if len(fine) == 2 else 0.45
    V = torch.from_numpy(inflow_state(meshes[-1].mesh, U, np.random.default_rng(1000 + seed))).to(DEV)
    out = []
    for m in reversed(meshes):
        out.insert(0, dict(m.fixed, J=m.csr(m.values(V))))
        if m.inject is not None:
            V = V[:, m.inject]
    return meshes, out


def _system(case, seed):
    shape = tuple(int(v) for v in case["shape"].split("x"))
    return _levels([tuple(s) for s in hierarchy_shapes(shape, case["levels"])], case["k"], case["r"], NU, seed)


def _normal(n, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device=DEV, generator=g)


def _solver(levels, case, segments=None):
    stream = torch.cuda.Stream(device=DEV)
    S = vk.Solver(levels, stream=stream)
    if segments is not None:
        S.vk_set_segments(segments)
    S.vk_set_workspace(case["prec"], RESTART, device=DEV)
    torch.cuda.synchronize()
    S.vanka_setup(OMEGA, case.get("mode", "additive"))
    return S, stream


@functools.lru_cache(maxsize=None)
def _batch_meshes(n_systems, draw_seed):
    """Hierarchies of the batch's systems and, per packed level, its pattern: the systems of a depth side by
    side, the ones solved directly there first (synth.batch's packing, on the GPU)."""
    hier = []
    for s in draw_systems(n_systems, draw_seed):
        shapes = batch_shapes(s["shape"], 1500, s["k"])
        hier.append((tuple(tuple(x) for x in shapes), s["k"], s["nu"], s["seed"]))
    return hier


def _csr_blocks(parts, n_rows, n_cols):
    """CSR with the blocks (row offset, column offset, csr dict) in ascending, disjoint row ranges."""
    counts = torch.zeros(n_rows, dtype=torch.int64, device=DEV)
    for r0, _, A in parts:
        counts[r0:r0 + A["n_rows"]] = A["row_ptr"][1:] - A["row_ptr"][:-1]
    ptr = torch.zeros(n_rows + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(counts, 0)
    col = torch.cat([A["col"] + c0 for _, c0, A in parts]).to(torch.int32)
    return dict(n_rows=n_rows, n_cols=n_cols, row_ptr=ptr, col=col, val=torch.cat([A["val"] for _, _, A in parts]))


def _batch_levels(case, seed):
    systems = [_levels(sh, k, 2, nu, 17 * seed + s) for sh, k, nu, s in _batch_meshes(case["systems"], case["draw"])]
    depth = max(len(lv) for _, lv in systems)
    packed, rows_of = [], []
    for pl in range(depth):
        at = {si: len(lv) - depth + pl for si, (_, lv) in enumerate(systems) if len(lv) - depth + pl >= 0}
        present = sorted(at, key=lambda si: (at[si] != 0, si))
        rows, blocks, off, groups = {}, [0], 0, {}
        for si in present:
            lv = systems[si][1][at[si]]
            rows[si] = off
            if at[si] == 0:
                blocks.append(off + lv["J"]["n_rows"])
            else:
                g = groups.setdefault(lv["n_K"], ([], []))
                g[0].append(lv["cell_dofs"] + off)
                g[1].append(systems[si][0][at[si]].mesh.colours())
            off += lv["J"]["n_rows"]
        J = _csr_blocks([(rows[si], rows[si], systems[si][1][at[si]]["J"]) for si in present], off, off)
        out = dict(J=J, P=None, R=None, groups=[], blocks=np.array(blocks if len(blocks) > 1 else [], dtype=np.int64))
        for n_K in sorted(groups):
            colours = np.concatenate(groups[n_K][1])
            ptr = np.concatenate([[0], np.cumsum(np.bincount(colours))]).astype(np.int32)
            cells = torch.cat(groups[n_K][0]).to(torch.int32)
            order = torch.from_numpy(np.argsort(colours, kind="stable").astype(np.int32)).to(DEV)
            out["groups"].append(dict(n_cells=cells.shape[0], n_K=n_K, cell_dofs=cells, colour_cells=order,
                                      colour_ptr=ptr, n_colours=len(ptr) - 1))
        if pl > 0:
            up = [si for si in present if at[si] > 0]
            prev = rows_of[-1]
            nc = packed[-1]["J"]["n_rows"]
            out["P"] = _csr_blocks([(rows[si], prev[si], systems[si][1][at[si]]["P"]) for si in up], off, nc)
            down = sorted(up, key=lambda si: prev[si])
            out["R"] = _csr_blocks([(prev[si], rows[si], systems[si][1][at[si]]["R"]) for si in down], nc, off)
        packed.append(out)
        rows_of.append(rows)
    seg = sorted(rows_of[-1].values()) + [packed[-1]["J"]["n_rows"]]
    return packed, np.array(seg, dtype=np.int64)


def _mlp_inputs(case, seed):
    """A dataset of patch features and targets, normalised as the trainer's, and the initial weights."""
    n_K = case["n_K"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn((8 * case["cells"], 2 * n_K), device=DEV, generator=g)
    mix = torch.randn((2 * n_K, n_K), device=DEV, generator=g) / (2 * n_K) ** 0.5
    target = torch.tanh(x @ mix) + 0.1 * torch.randn((x.shape[0], n_K), device=DEV, generator=g)
    rows = torch.randperm(x.shape[0], device=DEV, generator=g)[:case["batch"]].to(torch.int32)
    theta = torch.from_numpy(init_mlp_params(2 * n_K, WIDTH, N_HIDDEN, n_K, seed=seed)).to(DEV)
    return x.to(torch.bfloat16), target, rows, theta


def _predict_inputs(case, seed):
    nx, ny = (int(v) for v in case["shape"].split("x"))
    m = StructuredMesh((nx, ny), (H_CHANNEL * nx / ny, H_CHANNEL), case["k"])
    E = np.vander(dg_time_matrices(m.k)[0] + 1.0, m.n_time, increasing=True) @ np.linalg.inv(
        np.vander(dg_time_matrices(m.k)[0], m.n_time, increasing=True))
    slab = _normal(m.n, seed)
    slabs = [slab, slab + 0.01 * _normal(m.n, seed + 1)]      # two consecutive solutions
    cd = m.cell_dofs()
    g = torch.Generator(device=DEV).manual_seed(seed + 2)
    stats = [torch.rand(c, device=DEV, generator=g) * s + o for c, s, o in
             ((2 * m.n_K, 1e-3, 0.0), (2 * m.n_K, 10.0, 5.0), (m.n_K, 1e-3, 0.0), (m.n_K, 0.01, 0.005))]
    theta = torch.from_numpy(init_mlp_params(2 * m.n_K, WIDTH, N_HIDDEN, m.n_K, seed=seed)).to(DEV)
    return m, E, slabs, cd, stats, theta


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        levels, seg = _batch_levels(case, seed)
        S, stream = _solver(levels, case, seg)
        S.vk_autotune(10)
        S.vk_set_graphs(True)
        b = _normal(S.n, 2000 + seed)
        return dict(case=case, S=S, stream=stream, b=b, x=torch.zeros_like(b))
    if kind == "train":
        x, target, rows, theta = _mlp_inputs(case, seed)
        net = vk.MLP(2 * case["n_K"], WIDTH, N_HIDDEN, case["n_K"], max(4096, case["batch"]), device=DEV)
        net.set_params(theta)
        return dict(case=case, net=net, x=x, target=target, rows=rows)
    if kind == "predict":
        m, E, slabs, cd, stats, theta = _predict_inputs(case, seed)
        net = vk.MLP(2 * m.n_K, WIDTH, N_HIDDEN, m.n_K, max(4096, m.n_cells), device=DEV)
        net.set_params(theta)
        ptr, lst = vk.dof_entries(cd, m.n)
        like = [torch.zeros_like(slabs[0]) for _ in range(3)]
        return dict(case=case, net=net, E=E, slabs=slabs, stats=stats, n_K=m.n_K, base=like[0], prev_base=like[1],
                    out=like[2], cell_dofs=torch.from_numpy(cd).to(DEV), dof_ptr=torch.from_numpy(ptr).to(DEV),
                    dof_list=torch.from_numpy(lst).to(DEV),
                    feat=torch.zeros((m.n_cells, 2 * m.n_K), dtype=torch.bfloat16, device=DEV),
                    pred=torch.zeros((m.n_cells, m.n_K), dtype=torch.float32, device=DEV))
    _, levels = _system(case, seed)
    S, stream = _solver(levels, case)
    if case["tuned"]:
        S.vk_autotune(10)
    b = _normal(S.n, 2000 + seed)
    return dict(case=case, S=S, stream=stream, b=b, x=torch.zeros_like(b), d0=0.01 * _normal(S.n, 3000 + seed))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "train":
        loss, grad = state["net"].gradient(state["x"], state["target"], rows=state["rows"])
        state["net"].adam(1e-3)
        return dict(loss=loss, grad=grad, params=state["net"].get_params())
    if kind == "predict":
        net, (x1, x2) = state["net"], state["slabs"]
        in_mean, in_inv, out_mean, out_sd = state["stats"]
        net.slab_extrapolate(state["E"], x1, state["prev_base"])
        net.slab_extrapolate(state["E"], x2, state["base"])
        net.patch_features(state["cell_dofs"], x1, x2, state["prev_base"], in_mean, in_inv, state["feat"])
        net.forward(state["feat"], out=state["pred"])
        net.patch_average(state["dof_ptr"], state["dof_list"], state["n_K"], state["pred"], out_mean, out_sd,
                          state["base"], state["out"])
        return dict(pred=state["pred"], out=state["out"])
    S, b, x = state["S"], state["b"], state["x"]
    with torch.cuda.stream(state["stream"]):
        if kind == "sweep":
            x.copy_(state["d0"])
            S.vanka_smooth(case["levels"] - 1, b, x, case["sweeps"])
            return dict(d=x)
        if kind == "vcycle":
            S.vcycle(b, x, *NU_SWEEPS)
            return dict(x=x)
        S.vanka_setup(OMEGA, "additive")
        x.zero_()
        solve = S.gmres_solve_batched if kind == "batch" else S.gmres_solve
        out = solve(b, x, restart=RESTART, max_iter=300, rtol=1e-8, nu_pre=NU_SWEEPS[0], nu_post=NU_SWEEPS[1],
                    raise_on_noconv=False)
        return dict(its=out[0], x=x)


# ---- what a pass cannot do without ------------------------------------------------------------------------------


def _mesh_work(shapes, k, r, prec, nu, its, setup):
    """Bytes and flops of `its` V-cycles with nu sweeps in all on each level >= 1 (each sweep reads the stored
    inverses once and, but for the first, J once; one more J product for the residual) and of the setup (J read,
    inverses written, 2 n_K^3 flop per patch)."""
    total = dict(bytes=0.0, flops=0.0)
    for l, s in enumerate(shapes):
        m = StructuredMesh(s, (1.0,) * len(s), k, r)
        # nodes that share a cell with a node, and cells that hold it, summed over the nodes
        near = np.prod([(n - 1) * (2 * r + 1) + 2 * (r + 1) + n * (r - 1) * (r + 1) for n in m.shape])
        nnz = float(m.n_time * m.d * ((m.d + k) * near + 2 * m.n_pmodes * m.n_cells * m.n_loc_nodes))
        inv = m.n_cells * m.n_K ** 2 if l else 0
        products = its * (nu if l else 0)
        total["bytes"] += products * (12 * nnz + 24 * m.n) + its * nu * inv * PREC_BYTES[prec]
        total["flops"] += products * 2 * nnz + its * nu * 2 * inv
        if setup:
            total["bytes"] += 12 * nnz + inv * PREC_BYTES[prec]
            total["flops"] += 2.0 * inv * m.n_K if l else 2.0 * m.n ** 2
    return total


def work(case):
    kind = case["kind"]
    if kind == "batch":
        parts = [_mesh_work(sh, k, 2, case["prec"], sum(NU_SWEEPS), 9, True)
                 for sh, k, _, _ in _batch_meshes(case["systems"], case["draw"])]
        return {key: sum(p[key] for p in parts) for key in ("bytes", "flops")}
    if kind in ("train", "predict"):
        if kind == "predict":
            nx, ny = (int(v) for v in case["shape"].split("x"))
            m = StructuredMesh((nx, ny), (1.0, 1.0), case["k"])
            batch, n_K, passes = m.n_cells, m.n_K, 1
        else:
            batch, n_K, passes = case["batch"], case["n_K"], 3
        params = 2 * n_K * WIDTH + (N_HIDDEN - 1) * WIDTH ** 2 + n_K * WIDTH
        return dict(bytes=batch * n_K * 8.0 + params * (4 if passes == 1 else 32), flops=passes * 2.0 * batch * params)
    shape = tuple(int(v) for v in case["shape"].split("x"))
    shapes = hierarchy_shapes(shape, case["levels"])
    if kind == "sweep":
        w = _mesh_work(shapes, case["k"], case["r"], case["prec"], case["sweeps"], 1, False)
        c = _mesh_work(shapes[:-1], case["k"], case["r"], case["prec"], case["sweeps"], 1, False)
        return {key: w[key] - c[key] for key in w}
    its = 9 if kind == "newton" else 1
    return _mesh_work(shapes, case["k"], case["r"], case["prec"], sum(NU_SWEEPS), its, kind == "newton")


# ---- the same in 64 bits with plain torch -----------------------------------------------------------------------


class _Plain:
    """One level in plain torch: J as sparse CSR, the patch inverses by torch.linalg.inv."""

    def __init__(self, lv, patches=True):
        J = lv["J"]
        self.n = n = J["n_rows"]
        self.J = torch.sparse_csr_tensor(J["row_ptr"], J["col"].long(), J["val"], size=(n, n))
        self.dofs = lv["cell_dofs"].long()
        self.colours = [lv["colour_cells"].long()[lv["colour_ptr"][c]:lv["colour_ptr"][c + 1]]
                        for c in range(lv["n_colours"])]
        if not patches:
            return
        self.p = torch.bincount(self.dofs.ravel(), minlength=n).double()
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), J["row_ptr"][1:] - J["row_ptr"][:-1])
        keys = rows * n + J["col"]
        self.inv = []
        for d in self.dofs.split(1024):
            want = d[:, :, None] * n + d[:, None, :]
            at = torch.searchsorted(keys, want).clamp_(max=keys.numel() - 1)
            self.inv.append(torch.linalg.inv(torch.where(keys[at] == want, J["val"][at], 0.0)))
        self.inv = torch.cat(self.inv)

    def mul(self, x):
        return (self.J @ x[:, None])[:, 0]

    def local(self, cells, r):
        return (self.inv[cells] @ r[self.dofs[cells]][:, :, None])[:, :, 0]

    def sweep(self, b, d, mode):
        if mode == "additive":
            every = torch.arange(self.dofs.shape[0], device=DEV)
            z = torch.zeros_like(d).index_add_(0, self.dofs.ravel(), self.local(every, b - self.mul(d)).ravel())
            return d + OMEGA * z / self.p
        for cells in self.colours:
            y = self.local(cells, b - self.mul(d))
            d = d.clone()
            d[self.dofs[cells].ravel()] += OMEGA * y.ravel()
        return d


def _plain_vcycle(plain, levels, l, b):
    if l == 0:
        return torch.linalg.solve(plain[0].J.to_dense(), b)
    x = torch.zeros_like(b)
    for _ in range(NU_SWEEPS[0]):
        x = plain[l].sweep(b, x, "additive")
    P = levels[l]["P"]
    P = torch.sparse_csr_tensor(P["row_ptr"], P["col"].long(), P["val"], size=(P["n_rows"], P["n_cols"]))
    R = levels[l]["R"]
    R = torch.sparse_csr_tensor(R["row_ptr"], R["col"].long(), R["val"], size=(R["n_rows"], R["n_cols"]))
    c = _plain_vcycle(plain, levels, l - 1, (R @ (b - plain[l].mul(x))[:, None])[:, 0])
    x = x + (P @ c[:, None])[:, 0]
    for _ in range(NU_SWEEPS[1]):
        x = plain[l].sweep(b, x, "additive")
    return x


def _layers(theta, n_K):
    out, o = [], 0
    for fo, fi in [(WIDTH, 2 * n_K)] + [(WIDTH, WIDTH)] * (N_HIDDEN - 1) + [(n_K, WIDTH)]:
        out.append((theta[o:o + fo * fi].reshape(fo, fi), theta[o + fo * fi:o + fo * fi + fo]))
        o += fo * fi + fo
    return out


def _net(theta, x, n_K):
    layers = _layers(theta, n_K)
    for i, (W, b) in enumerate(layers):
        x = x @ W.T + b
        if i + 1 < len(layers):
            x = torch.tanh(x)
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, target, rows, theta = _mlp_inputs(case, seed)
        theta = theta.double().requires_grad_(True)
        loss = (_net(theta, x[rows.long()].double(), case["n_K"]) - target[rows.long()].double()).square().mean()
        grad, = torch.autograd.grad(loss, theta)
        step = 1e-3 * grad / (grad.abs() + 1e-8)        # Adam's first step
        return dict(loss=loss.detach().reshape(1), grad=grad, params=(theta - step).detach())
    if kind == "predict":
        m, E, (x1, x2), cd, (in_mean, in_inv, out_mean, out_sd), theta = _predict_inputs(case, seed)
        E, cd = torch.from_numpy(E).to(DEV), torch.from_numpy(cd).long().to(DEV)
        prev, base = ((E @ x.reshape(m.n_time, -1)).reshape(-1) for x in (x1, x2))
        feat = (torch.cat([(x2 - x1)[cd], (x2 - prev)[cd]], dim=1) - in_mean.double()) * in_inv.double()
        pred = _net(theta.double(), feat, m.n_K)
        z = torch.zeros_like(base).index_add_(0, cd.ravel(), (pred * out_sd.double() + out_mean.double()).ravel())
        return dict(pred=pred, out=base + z / torch.bincount(cd.ravel(), minlength=m.n).double())
    if kind == "batch":
        return None
    meshes, levels = _system(case, seed)
    n = meshes[-1].mesh.n
    b = _normal(n, 2000 + seed)
    if kind != "newton" and meshes[-1].mesh.n_cells * meshes[-1].mesh.n_K ** 2 > 1e8:
        return None  # the batched plain inverses take too long
    if kind == "newton":
        # the solution itself, which gmres_solve approaches to its tolerance; a dense solve while it is quick
        return dict(its=None, x=torch.linalg.solve(_Plain(levels[-1], False).J.to_dense(), b)) if n <= 33000 else None
    if kind == "vcycle":
        plain = [_Plain(lv, i > 0) for i, lv in enumerate(levels)]
        return dict(x=_plain_vcycle(plain, levels, len(levels) - 1, b))
    top, d = _Plain(levels[-1]), 0.01 * _normal(n, 3000 + seed)
    for _ in range(case["sweeps"]):
        d = top.sweep(b, d, case["mode"])
    return dict(d=d)
