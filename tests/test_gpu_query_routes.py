"""A query takes one of several kernels by batch size, grid and precision (the
corners gathered in the query kernel, one wave per tile in small batches, or
the batch encoded level by level first); each does the same arithmetic, so the
outputs equal bit for bit those of the spatially ordered query, which gathers,
at both sides of every size the choice turns on."""
import numpy as np
import pytest

from dataclasses import replace

from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import workload as W

pytestmark = pytest.mark.gpu

# one feature per level, an odd number of levels, two of them hashed
NET_F1 = W.NetConfig(n_levels=9, feat=1, base_res=4, max_res=60, log2_table=12, dense_only=False,
                     n_hidden=2, width=32, seed=21)
NET_F4 = W.NetConfig(n_levels=8, feat=4, base_res=8, max_res=300, log2_table=14, dense_only=False,
                     n_hidden=2, width=64, seed=22)
NETS = {"hash": W.CFG5, "f1": NET_F1, "f4": NET_F4, "dense": W.PAPER, "product": W.CFG2P,
        "tinyp": W.TINYP, "select": W.PAPERS, "tiny": W.TINY}


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("name", list(NETS))
def test_every_route_gives_the_same_bits(torch, name, prec):
    net = NETS[name]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    a = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, precision=prec))
    b = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, precision=prec,
                            batch_order=B.ORDER_SPATIAL))
    p = np.random.default_rng(5).normal(0.0, 0.3, a.n_params).astype(np.float32)
    a.set_state(p)
    b.set_state(p)
    n_max = 65537
    full = W.make_batch("surface", n_max, seed=9)
    full_aux = W.make_aux(full, 9) if net.sh_degree else None
    for n in (1, 31, 33, 2047, 2049, 16384, 16385, 24577, 32768, 32769, n_max):
        pos, d = dev(full.pos[:, :n]), dev(full.dir[:, :n])
        kw = dict(seed=3, stream_id=4)
        if net.sh_degree:
            kw["aux"] = dev(full_aux[:, :n])
        qa, qb = ((m.query_select if net.select else m.query)(pos, d, **kw) for m in (a, b))
        torch.cuda.synchronize()
        for k, v in qa.items():
            assert torch.equal(v, qb[k]), (n, k, (v - qb[k]).abs().max().item())
    # a small batch's blocks share the answers of a tile that asks for both kinds
    pos, d = dev(full.pos[:, :999]), dev(full.dir[:, :999])
    kw = dict(seed=3, stream_id=4)
    if net.sh_degree:
        kw["aux"] = dev(full_aux[:, :999])
    call = a.query_select if net.select else a.query
    every = call(pos, d, **kw)
    for part in (dict(sample=False), dict(lobes=False, pdf=False), dict(lobes=False, sample=False),
                 dict(pdf=False)):
        for k, v in call(pos, d, **part, **kw).items():
            assert v is None or torch.equal(v, every[k]), (part, k)
    a.close()
    b.close()
