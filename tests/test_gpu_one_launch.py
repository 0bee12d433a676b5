"""The one-launch form of small steps (k_one) against the fp64 oracle, around the edges of its rule and of its blocks: one
token, blocks of 16 and 32 tokens less and plus one, a round of eight waves and the next, the longest lists that it takes
and the first that it does not, rows of a deferred append, paged rows, rotary embedding, results in place of Q."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import THETA, _check_pool, _check_rope_pool, _check_rope_step, _check_step, _out64, _session
from util import OraclePool, check_close

pytestmark = pytest.mark.gpu

KINDS = [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)]


def _most(dtype, D):
    """Tokens of the longest list that one launch takes: 192 KiB of K and V per kv head in bf16, 112 in fp32."""
    return (192 << 10) // (4 * D) if dtype == "bf16" else (112 << 10) // (8 * D)


def _one_launch(w, s, step, lists=None, flags=0, position=None):
    """Whether this step is taken by one launch: it then has no partial rows.  The plan is that of a real call, whose results
    are those of the call without it, bit for bit."""
    q = to_device(w.q(step), w.dtype, s.device)
    out, again = torch.empty_like(q), torch.empty_like(q)
    plan = np.zeros(8, np.int64)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, out, lists=lists, flags=flags, position=position)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, again, lists=lists, flags=flags, position=position, dbg_plan=plan)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.uint8), again.view(torch.uint8))
    assert plan[3] or (plan[1] == 0 and plan[2] == w.n)
    return plan[3] == 0


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("G,Hkv,prefix,lengths,layout", [
    (1, 8, 1, [1], "head"), (2, 2, 14, [1, 2], "token"), (4, 1, 31, [16, 1, 33], "head"), (8, 1, 90, [30, 37, 5], "token"),
    (4, 2, 120, [7] * 6, "head"), (8, 4, 64, [3] * 9, "token")])
def test_edges_of_blocks_and_deferred_rows(dtype, D, G, Hkv, prefix, lengths, layout):
    w = W.single_request("one", dtype, Hkv * G, Hkv, D, 1.0, 21, prefix, lengths, "random", steps=2, k_std=D ** -0.5)
    head = layout == "head"
    s, op = _session(w, kv_layout=B.HEAD_MAJOR if head else B.TOKEN_MAJOR), OraclePool(w, head_major=head)
    s.append_events(w.n_prefill)
    op.append_events(w.n_prefill)
    keep = []
    for step in range(2):
        s.append_events(w.n_events(step), chunk=w.n, flags=B.APPEND_DEFER)
        keep.append(s._keep_rows)
        op.append_events(w.n_events(step))
        _check_step(w, s, op, step, explicit=bool(step))
        assert _one_launch(w, s, step, lists=w.lists(step) if step else None) == (prefix + max(lengths) + step + 1 <= _most(dtype, D))
    _check_pool(w, s, op)
    s.close()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("short", [0, 1])
def test_the_longest_lists_and_the_first_that_are_split(dtype, D, short):
    """The rule's line, from both sides: a stream that sees exactly the most tokens, one more and two more."""
    most = _most(dtype, D)
    w = W.single_request("line", dtype, 8, 2, D, 1.0, 22, most - 9 - short, [5, 9], "round_robin", steps=2, k_std=D ** -0.5)
    s, op = _session(w, kv_layout=B.HEAD_MAJOR), OraclePool(w, head_major=True)
    s.append_events(w.n_prefill)
    op.append_events(w.n_prefill)
    for step in range(2):
        s.append_events(w.n_events(step))
        op.append_events(w.n_events(step))
        _check_step(w, s, op, step)
        assert _one_launch(w, s, step) == (step < short)
    s.close()


def _two_requests(dtype, D, page):
    """Prefixes of 20 and 37 rows, three and two short threads; the newest three rows are two of one thread and one of another."""
    w = W.Workload(name="small batch", dtype=dtype, Hq=8, Hkv=2, D=D, scale=1.0, seed=91, max_requests=2, max_streams=4, k_std=D ** -0.5)
    w.dec_request, w.dec_stream = np.array([0, 0, 0, 1, 1], np.int32), np.array([1, 2, 3, 1, 2], np.int32)
    rng = np.random.default_rng(91)
    ev = []
    for r, (prefix, lengths) in enumerate([(20, [5, 20, 11]), (37, [7, 16])]):
        order = np.repeat(np.arange(len(lengths)), lengths)
        rng.shuffle(order)
        order = np.concatenate([order, [0, 0, 1]])
        ev += [(r, 0, -1)] * prefix
        ev += [(r, 1 + i, -1 if i in order[:k] else 0) for k, i in enumerate(order)]
        w.anc_slots += [list(range(prefix)) for _ in lengths]
    w.ev_request, w.ev_stream, w.ev_parent = (np.array(x, np.int32) for x in zip(*ev))
    w.n_prefill = len(ev)
    if page:
        w.page_tokens, w.pages_per_request = page, 128 // page
        w.n_phys_pages = 2 * w.pages_per_request + 3
        w.page_table = rng.permutation(w.n_phys_pages)[:2 * w.pages_per_request].astype(np.int32).reshape(2, -1)
    else:
        w.pool_tokens = 128
    return w


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("page", [0, 8, 32])
@pytest.mark.parametrize("defer", [False, True])
def test_requests_with_rotated_rows(dtype, D, page, defer):
    """Deferred, the newest rows are turned inside the launch: one where its query stands, one a position ahead of it."""
    w = _two_requests(dtype, D, page)
    pos = w.event_positions()
    s, op = _session(w, rope_theta=THETA), OraclePool(w)
    s.append_events(w.n_prefill - 3, flags=B.APPEND_ROPE, positions=pos)
    s.append_events(w.n_prefill, flags=B.APPEND_ROPE | (B.APPEND_DEFER if defer else 0), positions=pos)
    op.append_events(w.n_prefill, positions=pos, theta=THETA)
    _check_rope_step(w, s, op, 0, pos)
    _check_rope_pool(w, s, op, w.n_prefill)
    assert _one_launch(w, s, 0, flags=B.DECODE_ROPE_Q, position=w.q_positions(0))
    s.close()


# KiB of K and V per kv head up to which a step takes one launch, (plain, rotated) x (one stream or few (stream, kv head) pairs;
# others; others of more than 16 rows stacked over a shared prefix)
LINES = {("bf16", 128): [(192, 272, 288), (272, 384, 384)], ("bf16", 64): [(192, 192, 208), (240, 240, 240)],
         ("f32", 128): [(112, 192, 288), (256, 256, 416)], ("f32", 64): [(112, 144, 224), (192, 224, 256)]}


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("n,Hkv,G,column", [(1, 8, 4, 0), (2, 4, 1, 0), (1, 32, 1, 0), (6, 4, 1, 1), (3, 8, 4, 1), (4, 16, 1, 1), (3, 8, 8, 2), (6, 4, 4, 2)])
def test_the_longest_lists_of_many_pairs(dtype, D, rope, n, Hkv, G, column):
    """Each line from both sides: the longest list sees exactly the most tokens, then one more."""
    most = min(1024, (LINES[dtype, D][rope][column] << 10) // (2 * D * (2 if dtype == "bf16" else 4)))
    w = W.single_request("pairs", dtype, Hkv * G, Hkv, D, 1.0, 24, most - 4, [3] + [2] * (n - 1), "round_robin", steps=2, k_std=D ** -0.5)
    pos = w.event_positions() if rope else None
    s, op = _session(w, rope_theta=THETA if rope else 0.0), OraclePool(w)
    af, df = (B.APPEND_ROPE, B.DECODE_ROPE_Q) if rope else (0, 0)
    s.append_events(w.n_prefill, flags=af, positions=pos)
    for step in range(2):
        s.append_events(w.n_events(step), flags=af | B.APPEND_DEFER, positions=pos)
        op.append_events(w.n_events(step), **(dict(positions=pos, theta=THETA) if rope else {}))
        if rope:
            _check_rope_step(w, s, op, step, pos)
        else:
            _check_step(w, s, op, step)
        assert _one_launch(w, s, step, flags=df, position=w.q_positions(step) if rope else None) == (step == 0)
    s.close()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("G", [1, 2, 8])
@pytest.mark.parametrize("deferred", [0, 1, 9])
def test_rotated_rows_of_narrow_and_wide_groups(dtype, D, G, deferred):
    """Query rows for some of the waves, for each, and for more than there are; a stream's newest rows deferred, nine of them."""
    w = _two_requests(dtype, D, 0)
    w.Hq = w.Hkv * G
    pos = w.event_positions()
    s, op = _session(w, rope_theta=THETA), OraclePool(w)
    s.append_events(w.n_prefill - deferred, flags=B.APPEND_ROPE, positions=pos)
    if deferred:
        s.append_events(w.n_prefill, flags=B.APPEND_ROPE | B.APPEND_DEFER, positions=pos)
    op.append_events(w.n_prefill, positions=pos, theta=THETA)
    _check_rope_step(w, s, op, 0, pos)
    _check_rope_pool(w, s, op, w.n_prefill)
    assert _one_launch(w, s, 0, flags=B.DECODE_ROPE_Q, position=w.q_positions(0))
    s.close()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("page", [0, 8])
@pytest.mark.parametrize("deferred", [2, 17, 32])
def test_many_deferred_rotated_rows(dtype, D, page, deferred):
    """Two deferred rows, more of them than one round of waves turns, and the most that a step takes along; lists that hold one of
    them, several (with other threads' rows between them) and, in the other request, none."""
    w = _two_requests(dtype, D, page)
    pos = w.event_positions()
    s, op = _session(w, rope_theta=THETA), OraclePool(w)
    s.append_events(w.n_prefill - deferred, flags=B.APPEND_ROPE, positions=pos)
    s.append_events(w.n_prefill, flags=B.APPEND_ROPE | B.APPEND_DEFER, positions=pos)
    op.append_events(w.n_prefill, positions=pos, theta=THETA)
    _check_rope_step(w, s, op, 0, pos)
    _check_rope_pool(w, s, op, w.n_prefill)
    assert _one_launch(w, s, 0, flags=B.DECODE_ROPE_Q, position=w.q_positions(0))
    s.close()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("context,n", [(40, 8), (57, 12), (0, 32)])
def test_a_prompt_piece_deferred_and_rotated(dtype, D, context, n):
    """causal_skip: every token of the piece sees its own number of deferred rows; then the last token alone sees all of them."""
    w = W.single_request("piece", dtype, 8, 2, D, 1.0, 23, context + n, [1], "random", k_std=D ** -0.5)
    w.ev_stream[:], w.ev_parent[:] = 0, -1  # one stream, no fork
    pos = w.event_positions()
    s, op = _session(w, rope_theta=THETA, max_streams=n), OraclePool(w)
    if context:
        s.append_events(context, flags=B.APPEND_ROPE, positions=pos)
    q = w._encode(np.random.default_rng(5).standard_normal((n, w.Hq, D), dtype=np.float32))
    op.append_events(context + n, positions=pos, theta=THETA)
    q64 = oracle.rope(oracle.widen_pool(dtype, q), pos[context:context + n], THETA)
    for m in ([n] if n <= 12 else []) + [1]:  # (the plan of 32 of them does not ride in the kernel arguments)
        if s.n_done < context + n:
            s.append_events(context + n, flags=B.APPEND_ROPE | B.APPEND_DEFER, positions=pos)
        qd = to_device(q[n - m:], dtype, s.device)
        out, plan = torch.empty_like(qd), np.zeros(8, np.int64)
        s.h.decode_step(0, [0] * m, [0] * m, qd, out, causal_skip=list(range(m - 1, -1, -1)), flags=B.DECODE_ROPE_Q,
                        position=pos[context + n - m:context + n], dbg_plan=plan)
        seen = np.arange(context + n - m + 1, context + n + 1)
        ref, _ = oracle.attention_q64(op.g, op.k, op.v, [0] * m, seen, np.zeros(m + 1, int), [], [], [], q64[n - m:], w.scale)
        check_close(_out64(w, out), ref, dtype, f"{m} queries")
        assert plan[3] == 0 and plan[2] == m
    _check_rope_pool(w, s, op, context + n)
    s.close()


@pytest.mark.parametrize("shift", ["in place of q", "over part of q", "two elements off"])
def test_results_that_lie_over_the_queries(shift):
    """`out` on top of `q`, half over it, or not on a 16-byte boundary gives what separate buffers give (the last two in
    the split form, which has read Q before anything is written)."""
    w = W.single_request("alias", "bf16", 8, 2, 128, 1.0, 23, 100, [20, 33, 7], "random", k_std=128 ** -0.5)
    s = _session(w)
    s.append_events(w.n_prefill)
    size = w.n * w.Hq * w.D
    buf = torch.randn(2 * size, device=s.device, generator=torch.Generator(device=s.device).manual_seed(3)).to(torch.bfloat16)
    q, ref = buf[:size].view(w.n, w.Hq, w.D), torch.empty(w.n, w.Hq, w.D, dtype=torch.bfloat16, device=s.device)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, ref)
    at = {"in place of q": 0, "over part of q": size // 2, "two elements off": size + 2}[shift]
    n = min(size, 2 * size - at)
    assert n == size or shift == "two elements off"
    if n < size:
        buf = torch.cat([buf, buf])
        q = buf[:size].view(w.n, w.Hq, w.D)
    out = buf[at:at + size].view(w.n, w.Hq, w.D)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, out)
    check_close(_out64(w, out), _out64(w, ref), w.dtype, shift)
    s.close()
