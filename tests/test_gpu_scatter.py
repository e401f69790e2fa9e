"""The chunked grid scatter at its edges: one vertex, a chunk short of full and
one past it (512 slots with a lane per slot, 1,024 with two), both orders, each
feature count; all vertices in one cell (every lane's sums merge) and a batch so
sparse that its lines overflow the block's table.  The gradient is held to the
FP32 tolerance (1e-5 of the oracle's condition scale).  A vertex whose gradient
is not finite marks the entries of its own corners and no others."""
import numpy as np
import pytest

from dataclasses import replace

from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import workload as W
from test_gpu_parity import F1_HASH, F4_HASH, check_backward, dev, oracle_net, randomize

pytestmark = pytest.mark.gpu

NETS = {"F1": F1_HASH, "F2": W.CFG5, "F4": F4_HASH, "F4dense": W.PAPER}


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


@pytest.mark.parametrize("order", [B.ORDER_NONE, B.ORDER_SPATIAL])
@pytest.mark.parametrize("name", list(NETS))
def test_gradient_at_chunk_edges(O, torch, name, order):
    net = replace(NETS[name], precision="fp32")
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=order,
                                scatter_mode=B.SCATTER_ATOMIC))
    on = oracle_net(O, net)
    params = randomize(model, on, np.random.default_rng(51), grid_sd=0.5)
    for n in (1, 511, 513, 65537 if name == "F4dense" else 1025):
        batch = W.make_batch("surface", n, seed=60 + n)
        print(name, order, n, flush=True)
        check_backward(O, torch, model, on, params, batch, f"{name} n={n}")
    batch = W.make_batch("surface", 1500, seed=61)
    batch.pos[:] = batch.pos[:, :1] + 1e-5 * batch.pos
    check_backward(O, torch, model, on, params, batch, f"{name} one cell")
    model.close()


def _grid_grad(torch, net, order, scatter, batch):
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=order,
                                scatter_mode=scatter))
    model.set_state(np.random.default_rng(52).normal(0, 0.3, model.layout.n_params).astype(np.float32))
    grad = torch.zeros(model.layout.n_params, dtype=torch.float32, device="cuda")
    model.backward(*[dev(torch, a) for a in (batch.pos, batch.dir, batch.radiance, batch.pdf)],
                   grad=grad)
    g = grad.cpu().numpy().astype(np.float64)[:model.layout.grid_params]
    model.close()
    return g


@pytest.mark.parametrize("n", [513, 70001])
@pytest.mark.parametrize("order", [B.ORDER_NONE, B.ORDER_SPATIAL])
def test_precision_form_sums(torch, order, n):
    """The fixed-point sums against the binned pass's (both exact but for the
    rounding of the FP32 adds into the gradient: 2^-24 of the entry's running
    sum each, at most one per chunk and one per corner that finds no line)."""
    net = replace(W.CFG5, precision="bf16")
    batch = W.make_batch("surface", n, seed=62)
    a = _grid_grad(torch, net, order, B.SCATTER_ATOMIC, batch)
    b = _grid_grad(torch, net, order, B.SCATTER_BINNED, batch)
    scale = np.sqrt(np.mean(a * a))
    assert scale > 0
    assert np.max(np.abs(a - b)) <= 1e-4 * scale + 1e-5 * np.max(np.abs(a))
    assert np.sqrt(np.mean((a - b) ** 2)) <= 1e-5 * scale


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_a_vertex_that_is_not_finite(torch, prec):
    net = replace(W.CFG5, precision=prec)
    batch = W.make_batch("surface", 2000, seed=63)
    ref = _grid_grad(torch, net, B.ORDER_SPATIAL, B.SCATTER_ATOMIC, batch)
    batch.dir[0, 777] = np.nan
    got = _grid_grad(torch, net, B.ORDER_SPATIAL, B.SCATTER_ATOMIC, batch)
    bad = ~np.isfinite(got)
    assert 0 < bad.sum() <= net.n_levels * 8 * net.feat
    assert np.all(np.isfinite(ref))
    scale = np.max(np.abs(ref))
    assert np.max(np.abs(got[~bad] - ref[~bad])) <= 1e-5 * scale
