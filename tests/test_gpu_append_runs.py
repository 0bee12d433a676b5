"""Appends described by runs (K1): one run, as many as travel in the kernel arguments, one more than that; ragged
row counts; kv head counts that are no power of two; rotated keys whose position ids jump inside a request."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from test_gpu_parity import THETA, _check_pool, _check_rope_pool, _session
from util import OraclePool

pytestmark = pytest.mark.gpu


def _rows(kind):
    """request id per appended row, and the position ids' jumps"""
    if kind == "one run":
        return np.zeros(1301, np.int32)
    if kind == "64 runs":
        return np.repeat(np.arange(64, dtype=np.int32) % 2, 5)
    if kind == "65 runs":
        return np.repeat(np.arange(65, dtype=np.int32) % 2, 7)
    return np.random.default_rng(4).integers(0, 3, 33).astype(np.int32)  # "scattered"


@pytest.mark.parametrize("kind", ["one run", "64 runs", "65 runs", "scattered"])
@pytest.mark.parametrize("dtype,Hkv,D,page,rope", [("bf16", 3, 128, 0, False), ("f32", 1, 64, 16, False), ("bf16", 8, 64, 8, True), ("f32", 2, 128, 0, True)])
def test_rows_land_where_the_runs_say(kind, dtype, Hkv, D, page, rope):
    ev_r = _rows(kind)
    w = W.Workload(name="runs", dtype=dtype, Hq=Hkv, Hkv=Hkv, D=D, scale=1.0, seed=8, max_requests=3, pool_tokens=1344, max_streams=2)
    if page:
        w.page_tokens, w.pages_per_request, w.n_phys_pages = page, 1344 // page, 3 * 1344 // page + 3
        w.page_table = np.random.default_rng(5).permutation(w.n_phys_pages)[:3 * w.pages_per_request].astype(np.int32).reshape(3, -1)
    n = len(ev_r)
    w.ev_request, w.ev_stream, w.ev_parent = ev_r, np.zeros(n, np.int32), np.full(n, -1, np.int32)
    w.n_prefill = n
    pos = np.arange(n, dtype=np.int32) * 3 // 2 + 5  # goes on by one now and then, jumps otherwise
    s, op = _session(w, rope_theta=THETA if rope else 0.0), OraclePool(w)
    s.append_events(n, flags=B.APPEND_ROPE if rope else 0, positions=pos if rope else None)
    op.append_events(n, positions=pos if rope else None, theta=THETA)
    if rope:
        _check_rope_pool(w, s, op, n)
    else:
        _check_pool(w, s, op)
    s.close()


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("more", [0, 1])
def test_one_piece_per_thread_and_several(rope, more):
    """The line between them, 2^19 pieces (pairs of pieces, rotated): fp32, 8 heads x 128, 2048 (4096) rows and one more."""
    n = (4096 if rope else 2048) + more
    w = W.Workload(name="thin", dtype="f32", Hq=8, Hkv=8, D=128, scale=1.0, seed=9, max_requests=1, pool_tokens=4160, max_streams=2)
    w.ev_request, w.ev_stream, w.ev_parent, w.n_prefill = np.zeros(n, np.int32), np.zeros(n, np.int32), np.full(n, -1, np.int32), n
    w.ev_request[100:300], w.max_requests = 1, 2
    pos = np.arange(n, dtype=np.int32) + np.arange(n, dtype=np.int32) // 301  # (three runs, a dozen and more with the ids' jumps)
    s, op = _session(w, rope_theta=THETA if rope else 0.0), OraclePool(w)
    s.append_events(n, flags=B.APPEND_ROPE if rope else 0, positions=pos if rope else None)
    op.append_events(n, positions=pos if rope else None, theta=THETA)
    if rope:
        _check_rope_pool(w, s, op, n)
    else:
        _check_pool(w, s, op)
    s.close()


def test_position_ids_that_jump_after_30_to_51_rows():
    """Rows are looked at one at a time up to the 32nd of a run, 16 at a time behind it: runs that end around every such place."""
    lengths = list(range(30, 52)) + [96, 97]
    n = sum(lengths)
    w = W.Workload(name="jumps", dtype="f32", Hq=1, Hkv=1, D=64, scale=1.0, seed=10, max_requests=1, pool_tokens=1088, max_streams=2)
    w.ev_request, w.ev_stream, w.ev_parent, w.n_prefill = np.zeros(n, np.int32), np.zeros(n, np.int32), np.full(n, -1, np.int32), n
    pos = np.concatenate([1000 * (k % 7) + np.arange(m, dtype=np.int32) for k, m in enumerate(lengths)]).astype(np.int32)
    s, op = _session(w, rope_theta=THETA), OraclePool(w)
    s.append_events(n, flags=B.APPEND_ROPE, positions=pos)
    op.append_events(n, positions=pos, theta=THETA)
    _check_rope_pool(w, s, op, n)
    s.close()
