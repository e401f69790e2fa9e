"""The training tile kernel at its edges: one vertex, a partial tile, one past
the four waves of a block, one past a whole round of the chip's blocks; every
network shape it is built for in FP32, whose backward products are formed from
operands split into three BF16 numbers.  The gradient is held to the FP32
tolerance (1e-5 of the oracle's condition scale of each entry), which the split
must meet like FP32 products: its six products leave out 2^-26 of each."""
import numpy as np
import pytest

from dataclasses import replace

from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import workload as W
from test_gpu_parity import check_backward, oracle_net, randomize

pytestmark = pytest.mark.gpu

# (feature count, levels, hidden layers, width): the shapes besides the
# workloads' own; F = 1 with an odd number of levels, a width off the tile
SHAPES = {"production": W.CFG5, "paper": W.PAPER, "dense4": W.CFG1, "tiny": W.TINY,
          "f1": replace(W.CFG5, n_levels=19, feat=1, max_res=200, log2_table=14, n_hidden=2),
          "f1x3": replace(W.CFG5, n_levels=32, feat=1, max_res=300, log2_table=13),
          "f2in16": replace(W.CFG5, n_levels=7, max_res=150, log2_table=13, n_hidden=2, width=49),
          "f4x3": replace(W.PAPER, n_hidden=3, width=60),
          "f4in16x3": replace(W.CFG1, n_hidden=3)}


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


@pytest.mark.parametrize("name", list(SHAPES))
def test_gradient_at_tile_edges(O, torch, name):
    net = replace(SHAPES[name], precision="fp32")
    model = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, batch_order=B.ORDER_NONE))
    on = oracle_net(O, net)
    params = randomize(model, on, np.random.default_rng(31), grid_sd=0.5)
    for n in (1, 33, 129, 32 * 1024 + 1 if name == "production" else 1025):
        batch = W.make_batch("surface", n, seed=40 + n)
        print(name, n, flush=True)
        msgs, _, _ = check_backward(O, torch, model, on, params, batch, f"{name} n={n}")
        print("\n".join(msgs))
    model.close()
