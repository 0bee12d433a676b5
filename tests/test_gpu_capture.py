"""Calls under stream capture record all the words that their launches read: replayed after later calls have gone round
the pinned staging slots, with lists that were out of date on the device when the step was captured, with plans and
appends too large for the kernel arguments."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import THETA, _check_step, _session
from util import OraclePool

pytestmark = pytest.mark.gpu
SLOTS = 8  # pinned staging slots


def _bits(t):
    return t.view(torch.int16)


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
def test_steps_with_large_plans_and_lists_not_on_the_device(dtype, D, explicit):
    w = W.config4(n_requests=8, seed=5, pmin=200, pmax=900)
    w.dtype, w.D, w.k_std = dtype, D, D ** -0.5
    lists, n = w.lists(0), w.n - 1
    less = (lists[0][:n], lists[1][:n + 1], *lists[2:])  # another plan, as large
    assert sum(len(x) for x in less[2:]) > 2 * 960
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        twin, s = _session(w), _session(w)
        op = OraclePool(w).append_events(w.n_prefill)
        for x in (twin, s):
            x.append_events(w.n_prefill)
        qd = to_device(w.q(0), w.dtype, s.device)
        want, want_less, out, graphed = (torch.empty_like(qd) for _ in range(4))
        twin.h.decode_step(0, w.dec_request, w.dec_stream, qd, want, lists=lists)
        twin.h.decode_step(0, w.dec_request[:n], w.dec_stream[:n], qd, want_less, lists=less)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            s.h.decode_step(0, w.dec_request, w.dec_stream, qd, graphed, lists=lists if explicit else None)
        for _ in range(3):
            for k in range(SLOTS + 1):
                m = n if k % 2 else w.n
                s.h.decode_step(0, w.dec_request[:m], w.dec_stream[:m], qd, out, lists=less if k % 2 else lists)
            graphed.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(_bits(graphed), _bits(want))
            s.h.decode_step(0, w.dec_request[:n], w.dec_stream[:n], qd, out, lists=less)
            torch.cuda.synchronize()
            assert torch.equal(_bits(out[:n]), _bits(want_less[:n]))
        _check_step(w, s, op, explicit=False)  # the lists on the device are those of now
        for x in (twin, s):
            x.close()


@pytest.mark.parametrize("rope", [False, True])
def test_an_append_of_more_runs_than_the_kernel_arguments_hold(rope):
    n, R = 130, 2
    ev_r = (np.arange(n, dtype=np.int32) % R)
    zero, pos = np.zeros(n, np.int32), np.arange(n, dtype=np.int32) + 5
    w = W.Workload(name="capture", dtype="bf16", Hq=4, Hkv=2, D=128, scale=1.0, seed=8, max_requests=R, pool_tokens=1024, max_streams=2)
    flags = B.APPEND_ROPE if rope else 0
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = _session(w, n_layers=2, max_ranges=4096, rope_theta=THETA if rope else 0.0)
        s.k_pool.zero_()
        s.v_pool.zero_()
        rows = torch.randn(n, w.Hkv, w.D, device=s.device, generator=torch.Generator(device=s.device).manual_seed(1)).to(torch.bfloat16)
        s.h.append_kv(0, ev_r, zero, rows, rows, position=pos, flags=flags)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            s.h.append_kv(1, ev_r, zero, rows, rows, position=pos, flags=flags)
        half = s.k_pool.numel() // 2
        want_k, want_v = s.k_pool[:half].clone(), s.v_pool[:half].clone()
        for _ in range(3):
            for k in range(2):
                s.h.append_kv(0, ev_r, zero, rows, rows, position=pos, flags=flags)  # other slots, through other staging slots
            s.k_pool[half:].zero_()
            s.v_pool[half:].zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(_bits(s.k_pool[half:]), _bits(want_k)) and torch.equal(_bits(s.v_pool[half:]), _bits(want_v))
        s.close()


def test_a_captured_step_that_asks_for_lists_not_on_the_device_is_refused():
    w = W.config3(steps=1, prefix=700, n_streams=3)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = _session(w)
        s.append_events(w.n_events(0))
        op = OraclePool(w).append_events(w.n_events(0))
        qd = to_device(w.q(0), w.dtype, s.device)
        out = torch.zeros_like(qd)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            with pytest.raises(B.PastaError) as e:
                s.h.decode_step(0, w.dec_request, w.dec_stream, qd, out, flags=B.DECODE_DEVICE_LISTS)
            out.zero_()
        assert e.value.code == B.E_CAPACITY
        _check_step(w, s, op, explicit=False, flags=B.DECODE_DEVICE_LISTS)
        s.close()
