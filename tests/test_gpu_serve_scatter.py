"""The training scratch of a serving round: batches on both sides of the binned
scatter's smallest, two sessions in one round beside queries, and a round that
needs more room than the ones before it.  Each batch's first Adam moment equals
the session's own fused step up to the order of FP32 sums (1e-5 of the oracle's
condition scale, the FP32 tolerance), and each query the session's own query
bit for bit."""
from dataclasses import replace

import numpy as np
import pytest

import parity as P
from paper_2504_04315_amd import npm as B
from paper_2504_04315_amd import serve as S
from paper_2504_04315_amd import workload as W
from test_gpu_serve import dev, oracle_net

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rounds", [[(513, 1)], [(3001, 20001), (1, 30003)]])
def test_round_scatters_like_the_own_step(O, rounds):
    import torch
    srv = S.Server(budget_bytes=8 << 30, max_sessions=8)
    for rnd, sizes in enumerate(rounds):
        jobs = []
        srv.hold(True)
        for k, n in enumerate(sizes):
            net = replace(W.CFG5, seed=91 + 2 * rnd + k)
            cfg = B.make_config(net)
            sid = srv.create_session(cfg)
            b = W.make_batch("surface", n, seed=95 + k)
            args = [dev(torch, a) for a in (b.pos, b.dir, b.radiance, b.pdf)]
            out = dict(lobes=torch.empty((4, 8, n), device="cuda"), pdf=torch.empty(n, device="cuda"),
                       sdir=torch.empty((3, n), device="cuda"), spdf=torch.empty(n, device="cuda"))
            torch.cuda.synchronize()
            srv.submit_query(sid, args[0], args[1], seed=5, stream_id=2, **out)
            srv.submit_train(sid, *args)
            jobs.append((net, cfg, sid, b, args, out))
        srv.drain()
        for net, cfg, sid, b, args, out in jobs:
            own = B.NPM(cfg)
            q = own.query(args[0], args[1], seed=5, stream_id=2)
            for name, key in (("lobes", "lobes"), ("pdf", "pdf"), ("sdir", "sample_dir"),
                              ("spdf", "sample_pdf")):
                assert torch.equal(out[name], q[key]), (rnd, b.n, name)
            p0 = own.get_state().astype(np.float64)
            own.train_step(*args)
            torch.cuda.synchronize()
            n_params = own.n_params
            m_own = own.get_state(B.STATE_ADAM_M).astype(np.float64)
            m_srv = srv.session_state(sid, n_params, B.STATE_ADAM_M).astype(np.float64)
            on = oracle_net(O, net)
            cond = O.backward_cond(on, b.pos, b.dir, b.radiance, b.pdf, p0)
            c1 = float(1.0 - np.float32(net.beta1))
            print(P.assert_within(f"n={b.n}", m_srv, m_own, c1 * 1e-5 * cond + 1e-30), flush=True)
            own.close()
    srv.close()
