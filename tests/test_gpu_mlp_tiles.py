"""The network kernels at the edges of their 16-wide tiles: layer widths and batches around multiples
of 16 (and 1, and 1 024), against the FP64 oracle with the same BF16 rounding points.

Tolerances as in test_gpu_learned.py for up to four layers (5e-3 forward, 2e-2 gradient: a rounding
decision that flips moves one entry by at most one BF16 unit, 2^-8 relative), in proportion to the
number of layers beyond that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import mlp as omlp  # noqa: E402
from oracle.precision import round_bf16  # noqa: E402
from synth.learned import init_mlp_params, mlp_layer_shapes  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n_in,width,n_hidden,n_out,batch", [
    (1, 1, 1, 1, 1), (15, 16, 1, 17, 15), (42, 128, 3, 21, 16), (17, 130, 2, 33, 17), (84, 64, 8, 42, 129),
    (1024, 1024, 1, 1024, 33), (84, 128, 3, 42, 1030)])
def test_tile_edges(n_in, width, n_hidden, n_out, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"mlp {n_in} {width} {n_hidden} {n_out} batch {batch}", flush=True)
    shapes = mlp_layer_shapes(n_in, width, n_hidden, n_out)
    rng = np.random.default_rng(n_in + batch)
    p = (init_mlp_params(n_in, width, n_hidden, n_out, seed=batch)
         + 0.02 * rng.standard_normal(omlp.n_params(shapes))).astype(np.float32)
    X = round_bf16(rng.standard_normal((batch + 3, n_in)))
    T = rng.standard_normal((batch + 3, n_out)).astype(np.float32)
    rows = rng.permutation(batch + 3)[:batch].astype(np.int32)
    net = vk.MLP(n_in, width, n_hidden, n_out, batch, device=DEV)
    net.set_params(torch.from_numpy(p).to(DEV))
    x = torch.from_numpy(X.astype(np.float32)).to(torch.bfloat16).to(DEV)
    r = torch.from_numpy(rows).to(DEV)
    rel = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))
    more = max(1.0, (n_hidden + 1) / 4)
    y = net.forward(x, rows=r).cpu().numpy().astype(np.float64)
    _, y_r = omlp.forward(p.astype(np.float64), shapes, X[rows], bf16_points=True)
    assert rel(y, y_r) <= 5e-3 * more
    loss, g = net.gradient(x, torch.from_numpy(T).to(DEV), rows=r)
    L_r, g_r = omlp.loss_and_grad(p.astype(np.float64), shapes, X[rows], T[rows].astype(np.float64), bf16_points=True)
    assert abs(float(loss.item()) - L_r) <= 5e-3 * more * L_r
    assert rel(g.cpu().numpy().astype(np.float64), g_r) <= 2e-2 * more


@pytest.mark.parametrize("batch", [512, 4099, 1 << 20])
def test_bias_gradients_of_large_batches(batch):
    """The last layer's bias gradient is the sum of dz = bf16(2 (y - t) / count) over the batch.  The terms have
    8 digits and are added exactly in pairs of pairs or in 64 bits, so its error is one rounding, 2^-24, plus
    what pairs more than 2^16 apart lose, another 2^-24 at most."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"mlp bias gradient, batch {batch}", flush=True)
    net = vk.MLP(4, 16, 1, 3, batch, device=DEV)
    net.set_params(torch.from_numpy(init_mlp_params(4, 16, 1, 3, seed=3)).to(DEV))
    g = torch.Generator(device=DEV).manual_seed(batch)
    x = torch.randn((batch, 4), device=DEV, generator=g).to(torch.bfloat16)
    target = 4.0 + torch.rand((batch, 3), device=DEV, generator=g)
    y = net.forward(x)
    _, grad = net.gradient(x, target)
    scale = torch.tensor(2.0, device=DEV) / (torch.tensor(float(batch), device=DEV) * 3.0)
    dz = (scale * (y - target)).to(torch.bfloat16).double()
    want = dz.sum(dim=0)
    assert ((grad[-3:].double() - want).abs() <= 2.0 ** -23 * dz.abs().sum(dim=0)).all()
    net.close()


@pytest.mark.parametrize("n_in,n_out,batch", [(32, 42, 4096), (84, 42, 5000), (200, 3, 3000), (1, 300, 1000)])
@pytest.mark.parametrize("indexed", [False, True])
def test_outputs_that_share_memory_with_the_inputs(n_in, n_out, batch, indexed):
    """y over x, over its end, and just behind and before it: the same bits as with an output of its own."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_02690_amd as vk
    print(f"mlp {n_in} -> {n_out}, batch {batch}, indexed {indexed}", flush=True)
    net = vk.MLP(n_in, 16, 1, n_out, batch, device=DEV)
    net.set_params(torch.from_numpy(init_mlp_params(n_in, 16, 1, n_out, seed=3)).to(DEV))
    g = torch.Generator(device=DEV).manual_seed(batch)
    xs = torch.randn((batch, n_in), device=DEV, generator=g).to(torch.bfloat16)
    rows = torch.randperm(batch, device=DEV, generator=g).to(torch.int32) if indexed else None
    want = net.forward(xs, rows=rows)
    nx, ny = 2 * xs.numel(), 4 * want.numel()
    pad = (ny + 255) // 256 * 256
    for off in (0, nx // 2 // 4 * 4, (nx + 3) // 4 * 4, -(ny // 2 // 4 * 4), -ny):  # of y, from the start of x
        buf = torch.zeros(2 * pad + nx + 256, dtype=torch.uint8, device=DEV)
        x = buf[pad:pad + nx].view(torch.bfloat16).reshape(batch, n_in)
        x.copy_(xs)
        y = buf[pad + off:pad + off + ny].view(torch.float32).reshape(batch, n_out)
        net.forward(x, rows=rows, out=y)
        assert torch.equal(y, want), off
    net.close()
