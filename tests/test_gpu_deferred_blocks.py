"""k_attn over several deferred rows of one stream: blocks that hold nothing else (2, 5, 31 and 32 distinct rows, listed and
contiguous, in pools with and without pages, rotated and not), and their copy into the pool by few and by many work-groups."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import THETA, _out64, _session
from util import OraclePool, check_close

pytestmark = pytest.mark.gpu


def _paged(w, rows, page):
    w.page_tokens, w.pages_per_request, w.pool_tokens = page, -(-rows // page), 0
    w.n_phys_pages = w.pages_per_request + 5
    w.page_table = np.random.default_rng(17).permutation(w.n_phys_pages)[:w.pages_per_request].astype(np.int32).reshape(1, -1)


def _check_rows(w, s, op, lo, hi, rope):
    """Pool rows lo .. hi - 1: V bit for bit, K too where it is not turned (else one rounding to bf16 apart)."""
    k, v = s.pool_bits(0)
    for h in range(w.Hkv):
        at = np.array([oracle.elem_offset(op.g, oracle.phys_row(op.g, 0, t), h) for t in range(lo, hi)])
        idx = (at[:, None] + np.arange(w.D)[None, :]).ravel()
        assert np.array_equal(v[idx], op.v[idx])
        if rope:
            a, b = W.bf16_bits_to_f32(k[idx]), W.bf16_bits_to_f32(op.k[idx])
            # neighbours of a value in [2^e, 2^(e+1)) are 2^(e-7) apart: at most 2^-7 of it; and the fp32 error of two products that cancel
            assert np.all(np.abs(a - b) <= 2.0 ** -7 * np.abs(b) + 1e-6 * np.abs(b).max())
        else:
            assert np.array_equal(k[idx], op.k[idx])


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("form", ["piece", "alone", "kept"])
@pytest.mark.parametrize("context,m", [(700, 2), (700, 5), (700, 32), (2500, 31), (2500, 32)])
def test_blocks_of_deferred_rows_alone(context, m, form, rope, page):
    """A fork has 32 rows of its own, scattered among another's, then m deferred ones: the last block of its list holds these alone.
    piece: queries that see 1, half and all of them, and the other fork's; alone: one query; kept: from the device-resident lists."""
    w = W.single_request("blocks", "bf16", 8, 2, 128, 1.0, 31, context, [32, 40], "random", k_std=128 ** -0.5)
    n0 = w.n_prefill
    if page:
        _paged(w, n0 + m, page)
    pos = w.event_positions()
    s, op = _session(w, max_streams=8, rope_theta=THETA if rope else 0.0), OraclePool(w)
    ropes = dict(positions=pos, theta=THETA) if rope else {}
    s.append_events(n0, flags=B.APPEND_ROPE if rope else 0, positions=pos if rope else None)
    op.append_events(n0, **ropes)
    k, v = w.kv_rows(n0, n0 + m)
    kpos = int(pos[w.ev_stream[:n0] == 1].max()) + 1 + np.arange(m)
    kd, vd = to_device(k, w.dtype, s.device), to_device(v, w.dtype, s.device)
    s.h.append_kv(0, [0] * m, [1] * m, kd, vd, position=kpos if rope else None, flags=B.APPEND_DEFER | (B.APPEND_ROPE if rope else 0))
    ko = oracle.round_pool(w.dtype, oracle.rope(oracle.widen_pool(w.dtype, k), kpos, THETA)) if rope else k
    assert oracle.append(op.g, op.k, op.v, [0] * m, ko, v, op.tail)[0] == 0
    who, skip = {"piece": ([1, 1, 1, 2], [m - 1, m // 2, 0, 0]), "alone": ([1], [0]), "kept": ([1, 2], None)}[form]
    n = len(who)
    q = w._encode(np.random.default_rng(6).standard_normal((n, w.Hq, w.D), dtype=np.float32))
    qpos = np.array([kpos[m - 1 - (skip[i] if skip else 0)] if x == 1 else 11 for i, x in enumerate(who)], np.int32)
    q64 = oracle.widen_pool(w.dtype, q).astype(np.float64)
    if rope:
        q64 = oracle.rope(q64, qpos, THETA)
    pl, offs, st, ct, sd = w.lists(0)
    qd = to_device(q, w.dtype, s.device)
    out, plan = torch.empty_like(qd), np.zeros(8, np.int64)
    flags = (B.DECODE_ROPE_Q if rope else 0) | (B.DECODE_DEVICE_LISTS if form == "kept" else 0)
    s.h.decode_step(0, [0] * n, who, qd, out, causal_skip=skip, flags=flags, position=qpos if rope else None, dbg_plan=plan)
    assert plan[3] > 0, "split, not one launch"
    got = _out64(w, out)
    for j, x in enumerate(who):
        i = int(np.nonzero(w.dec_stream == x)[0][0])
        lists = [st[offs[i]:offs[i + 1]].tolist(), ct[offs[i]:offs[i + 1]].tolist(), sd[offs[i]:offs[i + 1]].tolist()]
        if x == 1:
            for a, b in zip(lists, (n0, m - (skip[j] if skip else 0), 1)):
                a.append(b)
        ref, _ = oracle.attention_q64(op.g, op.k, op.v, [0], [int(pl[i])], [0, len(lists[0])], *lists, q64[j:j + 1], w.scale)
        check_close(got[j], ref[0], w.dtype, f"query {j}")
    _check_rows(w, s, op, n0, n0 + m, rope)
    s.close()


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("context,n", [(1000, 9), (1003, 32), (4096, 32)])
def test_a_prompt_piece_over_a_long_context(context, n, rope, page):
    """A prompt fed in pieces, deferred: beyond the context and the piece's first row, every token's own rows are deferred ones alone."""
    w = W.single_request("piece", "bf16", 8, 2, 128, 1.0, 32, context + n, [1], "random", k_std=128 ** -0.5)
    w.ev_stream[:], w.ev_parent[:] = 0, -1  # one stream, no fork
    if page:
        _paged(w, context + n, page)
    pos = w.event_positions()
    s, op = _session(w, max_streams=n, rope_theta=THETA if rope else 0.0), OraclePool(w)
    af, p = (B.APPEND_ROPE, pos) if rope else (0, None)
    s.append_events(context, flags=af, positions=p)
    s.append_events(context + n, flags=af | B.APPEND_DEFER, positions=p)
    op.append_events(context + n, **(dict(positions=pos, theta=THETA) if rope else {}))
    q = w._encode(np.random.default_rng(7).standard_normal((n, w.Hq, w.D), dtype=np.float32))
    q64 = oracle.widen_pool(w.dtype, q).astype(np.float64)
    if rope:
        q64 = oracle.rope(q64, pos[context:context + n], THETA)
    qd = to_device(q, w.dtype, s.device)
    out, plan = torch.empty_like(qd), np.zeros(8, np.int64)
    s.h.decode_step(0, [0] * n, [0] * n, qd, out, causal_skip=list(range(n - 1, -1, -1)), flags=B.DECODE_ROPE_Q if rope else 0,
                    position=pos[context:context + n] if rope else None, dbg_plan=plan)
    assert plan[3] > 0
    ref, _ = oracle.attention_q64(op.g, op.k, op.v, [0] * n, np.arange(context + 1, context + n + 1), np.zeros(n + 1, int), [], [], [], q64, w.scale)
    check_close(_out64(w, out), ref, w.dtype, "piece")
    _check_rows(w, s, op, context, context + n, rope)
    s.close()
