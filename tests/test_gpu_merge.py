"""The merge launch (GPU) where its width changes with the number of parts, and results at any multiple of 4 bytes."""
from __future__ import annotations

import ctypes as C
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from util import OraclePool, check_close, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 33])  # 33 streams: their records are read from the plan instead of the kernel arguments
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("parts", [1, 16, 17, 32, 33, 64, 65, 128, 129])
def test_parts_around_a_batch(parts, dtype, D, n):
    """One stream over `parts` chunks of 64 tokens: a work-group of 64, 128 or 256 threads takes 8 parts per
    thread at once (16 / 32 / 64 parts of 128 dims, twice as many of 64); one part more is a batch more, or the next width."""
    from paper_2502_11517_amd.harness import Session, to_device, to_host_bits
    if n > 1 and parts > 17:
        pytest.skip("wider steps get longer chunks")
    w = W.single_request("parts", dtype, 4, 1, D, 1.0, 51, 64 * parts - 23, [20] * n, "round_robin", k_std=D ** -0.5)
    s = Session(w)
    s.append_events(w.n_prefill)
    op = OraclePool(w).append_events(w.n_prefill)
    ref, lse_ref = op.attention()
    q = to_device(w.q(0), w.dtype, s.device)
    # 4 bytes past a multiple of 16: a step is split and merged there, however small
    room = torch.full((q.numel() + 8,), float("nan"), dtype=q.dtype, device=s.device)
    skip = 1 if dtype == "f32" else 2
    out = room[skip:skip + q.numel()].view_as(q)
    assert out.data_ptr() % 16 == 4
    lse = torch.empty(w.n, w.Hq, dtype=torch.float32, device=s.device)
    plan = np.zeros(8, np.int64)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, out, out_lse=lse, dbg_plan=plan)
    assert plan[3] > 0 and (n > 1 or plan[1] + plan[2] == parts)
    check_close(to_f64(w, to_host_bits(out.clone(), w.dtype)), ref, w.dtype, "out")
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= (2e-2 if dtype == "bf16" else 1e-4)
    assert bool(torch.isnan(room[:skip]).all()) and bool(torch.isnan(room[skip + q.numel():]).all())
    s.close()


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNode(C.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p), ("shared", C.c_uint32)]


def launches_of(call):
    """(grid, threads) of every kernel that `call` launches on the current stream, in order, from a capture that is never run."""
    hip = C.CDLL(os.path.join(torch.__path__[0], "lib", "libamdhip64.so"))  # the runtime that the library is bound to, too
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
        call()
    raw, n = C.c_void_p(g.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        kind, k = C.c_int(-1), _KernelNode()
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0
        if kind.value == 0:
            assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(k)) == 0
            out.append(((k.grid.x, k.grid.y, k.grid.z), k.block.x))
    return out


@pytest.mark.parametrize("n", [4, 33])  # 33 streams: their records are read from the plan
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("parts", [2, 16, 17, 32, 33, 64, 65, 130])
def test_one_long_row_among_short_ones_sets_the_width(parts, dtype, D, n):
    """A request of `parts` chunks of 64 tokens ahead of n - 1 requests of two: the longest row's parts fit in one batch of the
    work-group's threads (or it has 256), whatever the mean is."""
    from paper_2502_11517_amd.harness import Session, to_device, to_host_bits
    lengths = [64 * parts - 23] + [100] * (n - 1)
    w = W.Workload(name="mixed", dtype=dtype, Hq=4, Hkv=1, D=D, scale=1.0, seed=52, max_requests=n, pool_tokens=64 * (-(-max(lengths) // 64)), max_streams=2, k_std=D ** -0.5)
    w.ev_request = np.repeat(np.arange(n, dtype=np.int32), lengths)
    w.ev_stream, w.ev_parent, w.n_prefill = np.zeros(len(w.ev_request), np.int32), np.full(len(w.ev_request), -1, np.int32), len(w.ev_request)
    w.dec_request, w.dec_stream = np.arange(n, dtype=np.int32), np.zeros(n, np.int32)
    lists = (np.asarray(lengths, np.int32), np.zeros(n + 1, np.int32), *(np.zeros(0, np.int32) for _ in range(3)))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = Session(w)
        s.append_events(w.n_prefill)
        op = OraclePool(w).append_events(w.n_prefill)
        ref, lse_ref = oracle.attention(op.g, op.k, op.v, w.dec_request, *lists, w.q(0), w.scale)
        q = to_device(w.q(0), w.dtype, s.device)
        out, lse, plan = torch.empty_like(q), torch.empty(n, 4, dtype=torch.float32, device=s.device), np.zeros(8, np.int64)
        step = lambda: s.h.decode_step(0, w.dec_request, w.dec_stream, q, out, out_lse=lse, flags=B.DECODE_ROW_GROUPS, dbg_plan=plan)  # noqa: E731
        step()
        torch.cuda.synchronize()
        assert plan[1] == parts + 2 * (n - 1) and plan[2] == 0
        check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
        assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= (2e-2 if dtype == "bf16" else 1e-4)
        grid, threads = launches_of(step)[-1]
        per_64 = 16 if D == 128 else 32
        assert grid == (1, 4, n) and threads == (64 if parts <= per_64 else 128 if parts <= 2 * per_64 else 256)
        s.close()
