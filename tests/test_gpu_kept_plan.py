"""The plan kept on the device (k_plan): used again only while it is the same plan.  Steps whose plan is too large for
the kernel arguments, on several layers, with the lists or the deferred rows changing between the calls in ways that
leave the plan's size unchanged; the same calls under stream capture, replayed after other plans have been made."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import _check_step, _out64, _session
from util import OraclePool, check_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page,hq", [(0, 32), (16, 32), (16, 8)])
@pytest.mark.parametrize("explicit", [False, True])
def test_plans_follow_the_lists(page, hq, explicit):
    """Explicit lists that differ only in a start (same number of words), then maintained lists that grow: every step
    against the oracle, the second time from the plan that is there."""
    w = W.single_request("kept", "bf16", hq, 8 if hq == 32 else 1, 128, 1.0, 21, 330, [90, 3, 129, 64, 17, 33, 200, 5] * 3, "random", steps=3,
                         k_std=128 ** -0.5)
    if page:
        w.page_tokens, w.pages_per_request = page, -(-w.pool_tokens // page)
        w.n_phys_pages = w.pages_per_request + 3
        w.page_table = np.random.default_rng(3).permutation(w.n_phys_pages)[:w.pages_per_request].astype(np.int32).reshape(1, -1)
    s, op = _session(w, kv_layout=B.HEAD_MAJOR), OraclePool(w, head_major=True)
    s.append_events(w.n_prefill)
    op.append_events(w.n_prefill)
    keep = []
    for step in range(3):
        s.append_events(w.n_events(step), chunk=w.n, flags=B.APPEND_DEFER if step else 0)
        keep.append(s._keep_rows)
        op.append_events(w.n_events(step))
        for again in range(2):  # the deferred rows ride with the first call, the second reads them in the pool
            _check_step(w, s, op, step, explicit=explicit, what=f"step {step} call {again}")
    if explicit:  # the same lists but for one range that begins a row earlier
        pl, offs, st, ct, sd = [a.copy() for a in w.lists(2)]
        first = set(offs.tolist())
        k = next(k for k in range(len(st)) if k not in first and st[k] - 1 > st[k - 1] + (ct[k - 1] - 1) * sd[k - 1])
        st[k] -= 1
        q = w.q(2)
        qd = to_device(q, w.dtype, s.device)
        out = torch.empty_like(qd)
        s.h.decode_step(0, w.dec_request, w.dec_stream, qd, out, lists=(pl, offs, st, ct, sd))
        ref, _ = oracle.attention(op.g, op.k, op.v, w.dec_request, pl, offs, st, ct, sd, q, w.scale)
        check_close(_out64(w, out), ref, w.dtype, "one start changed")
    s.close()


def test_a_captured_step_does_not_lean_on_the_kept_plan():
    w = W.config4(n_requests=8, seed=5, pmin=200, pmax=900)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = _session(w)
        s.append_events(w.n_prefill)
        qd = to_device(w.q(0), w.dtype, s.device)
        eager, graphed, part = torch.empty_like(qd), torch.zeros_like(qd), torch.empty_like(qd)
        s.h.decode_step(0, w.dec_request, w.dec_stream, qd, eager)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            s.h.decode_step(0, w.dec_request, w.dec_stream, qd, graphed)
        n = w.n - 1  # another plan of the same lists
        want = torch.empty_like(qd)
        s.h.decode_step(0, w.dec_request[:n], w.dec_stream[:n], qd, want)
        for _ in range(3):
            g.replay()
            s.h.decode_step(0, w.dec_request[:n], w.dec_stream[:n], qd, part)
            torch.cuda.synchronize()
            assert torch.equal(graphed.view(torch.int16), eager.view(torch.int16))
            assert torch.equal(part[:n].view(torch.int16), want[:n].view(torch.int16))
            graphed.zero_()
        s.close()
