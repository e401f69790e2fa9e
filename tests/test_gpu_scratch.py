"""Scratch of a context: a query of fewer than 2^15 vertices allocates nothing, so
that its first call can be captured; a larger call without room for its scratch
(under capture, or on a full device) takes the kernels that need none, or less,
and gives the same results."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import workload as W
from test_gpu_parity import dev

pytestmark = pytest.mark.gpu

SMALL = [(W.CFG5, "bf16"), (W.CFG5, "fp32"), (replace(W.CFG2P, log2_table=14), "fp32")]


def _model(net, prec, seed=5):
    m = B.NPM(B.make_config(net, exec_mode=B.EXEC_FUSED, precision=prec))
    m.set_state(np.random.default_rng(seed).normal(0, 0.3, m.n_params).astype(np.float32))
    return m


def _inputs(torch, net, n, seed=9):
    b = W.make_batch("surface", n, seed=seed)
    aux = dev(torch, W.make_aux(b, seed)) if net.sh_degree else None
    return b, dev(torch, b.pos), dev(torch, b.dir), aux


def _query_into(torch, m, n, pos, d, aux, out):
    B.check(B.lib().npm_query_aux(m.handle, n, B._ptr(pos), B._ptr(aux), B._ptr(d), 3, 4,
                                  *(B._ptr(o) for o in out), B._stream()))


def _outputs(torch, n):
    return [torch.empty((4, 8, n), device="cuda"), torch.empty(n, device="cuda"),
            torch.empty((3, n), device="cuda"), torch.empty(n, device="cuda")]


@pytest.mark.parametrize("net,prec", SMALL, ids=["bf16", "fp32", "product"])
@pytest.mark.parametrize("n", [20011, 32767, 50001])
def test_first_query_under_capture(net, prec, n):
    import torch
    m, other = _model(net, prec), _model(net, prec)
    _, pos, d, aux = _inputs(torch, net, n)
    want, out = _outputs(torch, n), _outputs(torch, n)
    _query_into(torch, other, n, pos, d, aux, want)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        _query_into(torch, m, n, pos, d, aux, out)
    for _ in range(3):
        for o in out:
            o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        _query_into(torch, other, n, pos, d, aux, want)     # the program's own work between
    m.close()
    other.close()


@pytest.mark.parametrize("net,prec", SMALL, ids=["bf16", "fp32", "product"])
def test_small_queries_allocate_nothing(net, prec):
    import torch
    m = _model(net, prec)
    _, pos, d, aux = _inputs(torch, net, 32767)
    sets = []
    for n in (16385, 24577, 32767):
        sets.append((n, pos[:, :n].contiguous(), d[:, :n].contiguous(),
                     None if aux is None else aux[:, :n].contiguous(), _outputs(torch, n)))
    _query_into(torch, m, 64, *(t if t is None else t[:, :64].contiguous() for t in (pos, d, aux)),
                _outputs(torch, 64))                        # loads the code
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for n, p, dd, a, out in sets:
        _query_into(torch, m, n, p, dd, a, out)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    m.close()


def _fill(torch, leave):
    """Takes the device's memory but for `leave` bytes."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    keep = torch.empty(leave, dtype=torch.uint8, device="cuda")
    held, size = [], torch.cuda.mem_get_info()[0]
    while size >= 16 << 20:
        try:
            held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            size //= 2
    del keep
    torch.cuda.empty_cache()
    print(f"holding {sum(t.numel() for t in held) >> 20} MB, {leave >> 20} left", flush=True)
    return held


def _launched(m):
    return {k for k, v in m.kernel_times().items() if v[0]}


def test_query_on_a_full_device():
    import torch
    n = 1 << 21                                             # 134 MB of features
    m, other = _model(W.CFG5, "bf16"), _model(W.CFG5, "bf16")
    _, pos, d, aux = _inputs(torch, W.CFG5, n)
    want, out = _outputs(torch, n), _outputs(torch, n)
    _query_into(torch, other, n, pos, d, aux, want)
    warm = [t[:, :40000].contiguous() for t in (pos, d)]
    _query_into(torch, m, 40000, *warm, None, _outputs(torch, 40000))
    m.set_timing()
    held = _fill(torch, 100 << 20)
    _query_into(torch, m, n, pos, d, aux, out)
    torch.cuda.synchronize()
    assert _launched(m) == {"fused_query"}
    assert all(torch.equal(a, b) for a, b in zip(out, want))
    del held
    torch.cuda.empty_cache()
    m.close()
    other.close()


# (network, precision, vertices, bytes left): room for the order and the dG, not
# for the features behind it; room for both, not for the bins
FULL = {"features": (W.PAPER, "fp32", 1 << 21, 460 << 20),
        "bins": (W.CFG5, "fp32", 1 << 20, 500 << 20)}


@pytest.mark.parametrize("what", list(FULL))
def test_training_on_a_full_device(what):
    import torch
    net, prec, n, leave = FULL[what]
    b, pos, d, _ = _inputs(torch, net, n)
    args = (pos, d, dev(torch, b.radiance), dev(torch, b.pdf))
    few = [t[..., :40000].contiguous() for t in args]
    res = []
    for full in (False, True):
        m = _model(net, prec)
        g = torch.zeros(m.n_params, dtype=torch.float32, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        m.backward(*few)
        m.backward_static(*(t[..., :1000].contiguous() for t in args))
        m.set_timing()
        held = _fill(torch, leave) if full else None
        m.backward(*args, grad=g, loss=loss)
        torch.cuda.synchronize()
        assert ({"features": "train_encode", "bins": "bin_reduce"}[what] in _launched(m)) != full
        del held
        torch.cuda.empty_cache()
        res.append((g.cpu().numpy().astype(np.float64), float(loss[0])))
        m.close()
    (a, la), (c, lc) = res
    assert abs(la - lc) <= 1e-9 * abs(la)
    # two routes of one form: FP32 sums in another order
    assert np.sqrt(np.mean((a - c) ** 2)) <= 1e-5 * np.sqrt(np.mean(a * a))
