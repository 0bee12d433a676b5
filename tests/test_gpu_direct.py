"""The partials kernel of fp32 pools and 64-wide heads (k_direct) against the fp64 oracle, at the sizes where it can go
wrong: row tiles of 16 (15 to 17, 32 and 33 stacked rows), blocks of 16 or 32 tokens, one block and several per
wave, windows of address codes, paged rows, deferred rows, the rotary embedding on the way in."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from test_gpu_parity import THETA, _check_pool, _check_rope_pool, _check_rope_step, _check_step, _out64, _session
from util import OraclePool, check_close

pytestmark = pytest.mark.gpu

KINDS = [("f32", 64), ("f32", 128), ("bf16", 64)]


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("G,Hkv,prefix,lengths", [
    (1, 8, 64, [1]), (1, 2, 65, [17] * 15), (4, 1, 97, [16, 15, 33, 31]), (1, 4, 1000, [5] * 17), (8, 1, 2111, [127, 128, 129, 1]),
    (1, 1, 640, [3] * 33), (2, 1, 9001, [40, 70]), (4, 2, 63, [9, 300])])
def test_tiles_blocks_and_deferred_rows(dtype, D, G, Hkv, prefix, lengths):
    w = W.single_request("direct", dtype, Hkv * G, Hkv, D, 1.0, 11, prefix, lengths, "random", steps=2, k_std=D ** -0.5)
    s, op = _session(w, kv_layout=B.HEAD_MAJOR), OraclePool(w, head_major=True)
    s.append_events(w.n_prefill)
    op.append_events(w.n_prefill)
    keep = []
    for step in range(2):
        s.append_events(w.n_events(step), chunk=w.n, flags=B.APPEND_DEFER)
        keep.append(s._keep_rows)
        op.append_events(w.n_events(step))
        _check_step(w, s, op, step, explicit=bool(step), flags=0 if step else B.DECODE_DEVICE_LISTS)
    _check_pool(w, s, op)
    s.close()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("page", [8, 32])
def test_ragged_paged_batch_with_rotated_rows(dtype, D, page):
    w = W.config4(n_requests=3, seed=91, pmin=40, pmax=700, page_tokens=page, hq=8, hkv=2)
    w.dtype, w.D, w.k_std = dtype, D, D ** -0.5
    pos = w.event_positions()
    s, op = _session(w, rope_theta=THETA), OraclePool(w)
    s.append_events(w.n_prefill - 3, flags=B.APPEND_ROPE, positions=pos)
    s.append_events(w.n_prefill, flags=B.APPEND_ROPE | B.APPEND_DEFER, positions=pos)
    op.append_events(w.n_prefill, positions=pos, theta=THETA)
    _check_rope_step(w, s, op, 0, pos)
    _check_rope_pool(w, s, op, w.n_prefill)
    s.close()


def test_more_tokens_per_chunk_than_a_window_of_address_codes():
    """The no-alloc entry point's 16 MiB of partials make 160 stacked rows over 27k tokens take chunks of more than
    1024 tokens; compared with the vector-ALU walker, which shares nothing with it (fp32: both within 1e-5 of the exact result)."""
    w = W.single_request("window", "f32", 64, 8, 128, 1.0, 12, 27001, [3] * 20, "round_robin", k_std=128 ** -0.5)
    s = _session(w, kv_layout=B.HEAD_MAJOR)
    s.append_events(w.n_prefill)
    q = torch.randn(w.n, w.Hq, w.D, device=s.device, generator=torch.Generator(device=s.device).manual_seed(3))
    a, b = torch.empty_like(q), torch.empty_like(q)
    s.h.decode_step_noalloc(0, w.dec_request, w.dec_stream, q, a)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, b, flags=B.DECODE_NO_MFMA)
    check_close(_out64(w, a), _out64(w, b), w.dtype, "chunks of several windows")
    s.close()
