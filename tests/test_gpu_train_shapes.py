"""The training kernels' remaining shapes at the edges of their tiles -- one
vertex, a partial tile, one past a block's four waves, one past eight blocks --
in the caller's and in spatial order.

FP32: the shapes beside test_gpu_train_tile's (one feature on a narrow network,
two hidden layers on 32 inputs, the narrow NPM-product input, every selection
shape with its densities), held to the FP32 tolerance (1e-5 of the oracle's
condition scale of each entry).

Precision form: against the gathering kernel, which rounds the same values to
BF16 at the same points and sums in another order.  A delta's sum that falls on
the other side of a rounding moves by 2^-8 of itself, at most once per layer, so
each entry is held to 2^-8 (layers) of its condition scale, and the whole
gradient, where few deltas do, to a tenth of 2^-8."""
from dataclasses import replace

import numpy as np
import pytest

import parity as P
import test_gpu_select as SEL
from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import workload as W
from test_gpu_parity import check_backward, dev, oracle_net, randomize

pytestmark = pytest.mark.gpu

SIZES = (1, 33, 129, 1025)
ORDERS = {"none": B.ORDER_NONE, "spatial": B.ORDER_SPATIAL}
NARROW_F1 = W.NetConfig(n_levels=9, feat=1, base_res=4, max_res=60, log2_table=12, dense_only=False,
                        n_hidden=2, width=32, seed=21)
TWO_HIDDEN = replace(W.CFG5, n_hidden=2, max_res=200, log2_table=13)
SMALL = dict(max_res=300, log2_table=13)


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("net", [NARROW_F1, TWO_HIDDEN, W.TINYP], ids=["f1", "two hidden", "product"])
def test_fp32_gradient(O, net, order):
    import torch
    net = replace(net, precision="fp32")
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=ORDERS[order]))
    on = oracle_net(O, net)
    params = randomize(model, on, np.random.default_rng(32), grid_sd=0.5)
    for n in SIZES:
        batch = W.make_batch("surface", n, seed=41 + n)
        aux = W.make_aux(batch, 41) if net.sh_degree else None
        print(order, n, flush=True)
        check_backward(O, torch, model, on, params, batch, f"n={n}", aux=aux)
    model.close()


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("net", [W.TINYS, W.CFG1S, W.PAPERS, replace(W.CFG5, select=True, **SMALL)],
                         ids=["tiny", "dense4", "paper", "production"])
def test_fp32_selection_gradient(O, net, order):
    import torch
    net = replace(net, precision="fp32")
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=ORDERS[order]))
    on = SEL.oracle_net(O, net)
    params = SEL.randomize(model, on, np.random.default_rng(33), grid_sd=0.5)
    for n in SIZES:
        b = W.make_batch("surface", n, seed=42 + n)
        bsdf = W.make_bsdf(b, 42)
        g = torch.zeros(on.n_params, dtype=torch.float32, device="cuda")
        loss = torch.zeros(2, dtype=torch.float64, device="cuda")
        print(order, n, flush=True)
        model.backward_select(*[dev(torch, a) for a in (b.pos, b.dir, b.radiance, b.pdf, bsdf)],
                              grad=g, loss=loss)
        args = (on, b.pos, b.dir, b.radiance, b.pdf, params)
        ref = O.backward(*args, bsdf=bsdf)
        P.check_grads(f"n={n}", g.cpu().numpy().astype(np.float64), ref["grad"],
                      O.backward_cond(*args, bsdf=bsdf))
        for got, want in zip(loss.tolist(), (ref["loss"], ref["loss_sel"])):
            assert abs(got - want) <= 1e-5 * max(1.0, abs(want))
    model.close()


BF16 = {"production": replace(W.CFG5, **SMALL), "paper": W.PAPER, "dense4": W.CFG1, "tiny": W.TINY,
        "f1": NARROW_F1, "two hidden": TWO_HIDDEN, "f4x3": replace(W.PAPER, n_hidden=3, width=60),
        "wide product": replace(W.CFG2P, **SMALL), "wide product f4": W.PAPERP, "product": W.TINYP}


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("name", list(BF16))
def test_bf16_gradient(O, name, order):
    import torch
    net = replace(BF16[name], precision="bf16")
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=ORDERS[order],
                                scatter_mode=B.SCATTER_ATOMIC))
    on = oracle_net(O, net)
    params = randomize(model, on, np.random.default_rng(34), grid_sd=0.5)
    layers = len(on.layer_shape)
    for n in SIZES:
        b = W.make_batch("surface", n, seed=43 + n)
        aux = W.make_aux(b, 43) if net.sh_degree else None
        args = [dev(torch, a) for a in (b.pos, b.dir, b.radiance, b.pdf)]
        out = []
        for call in (model.backward, model.backward_static):
            g = torch.zeros(on.n_params, dtype=torch.float32, device="cuda")
            loss = torch.zeros(1, dtype=torch.float64, device="cuda")
            call(*args, grad=g, loss=loss, aux=None if aux is None else dev(torch, aux))
            out.append((g.cpu().numpy().astype(np.float64), float(loss[0])))
        (a, la), (r, lr) = out
        print(name, order, n, flush=True)
        assert abs(la - lr) <= 1e-9 * max(1.0, abs(lr))
        cond = O.backward_cond(on, b.pos, b.dir, b.radiance, b.pdf, params, aux=aux)
        P.assert_within(f"n={n}", a, r, layers * 2.0 ** -8 * cond + 1e-30)
        assert np.sqrt(np.mean((a - r) ** 2)) <= 0.1 * 2.0 ** -8 * np.sqrt(np.mean(r * r))
    model.close()
