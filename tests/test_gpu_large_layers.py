"""bf16 layers of 4 GiB and more with 128-wide heads (k_direct<uint16_t, 128>): pages on both sides of the 4 GiB offset, more
than one tile and more than one group of stacked rows, private pieces, deferred rows, the rotary embedding on the way in;
weights of fp32's bits, also in steps that are small enough for one launch elsewhere."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device, to_host_bits
from test_gpu_parity import THETA, _check_rope_step, _out64, _session
from test_gpu_weights import _check
from util import OraclePool, check_close, geom_of

pytestmark = pytest.mark.gpu
PAGE, HKV = 16, 2
PAGES = ((1 << 32) + (1 << 28)) // (PAGE * HKV * 128 * 2)  # 4.25 GiB of K, and of V
SHAPES = [(8, 700, [40, 129, 7, 64, 300]), (4, 1090, [50, 33]), (1, 40, [9]), (8, 60, [40, 3])]


def _workload(G, prefix, lengths, pages):
    """The same history over `pages` physical pages: the request's are spread over all of them."""
    w = W.single_request("large", "bf16", HKV * G, HKV, 128, 1.0, 51, prefix, lengths, "random", k_std=128 ** -0.5)
    rng = np.random.default_rng(51)
    w.page_tokens, w.pages_per_request, w.n_phys_pages, w.pool_tokens = PAGE, -(-(w.n_prefill + 8) // PAGE), pages, 0
    w.page_table = np.sort(rng.permutation(pages)[:w.pages_per_request]).astype(np.int32).reshape(1, -1)
    rng.shuffle(w.page_table[0])
    return w


@pytest.mark.parametrize("layout", [B.TOKEN_MAJOR, B.HEAD_MAJOR])
@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("G,prefix,lengths", SHAPES)
def test_rows_beyond_4_gib(layout, rope, G, prefix, lengths):
    w = _workload(G, prefix, lengths, PAGES)
    far = w.page_table[0].astype(np.int64) * PAGE * HKV * 256 >= 1 << 32
    w.page_table[0, [0, -1]] = PAGES - 1, PAGES - 2  # (whatever was drawn: the first and the last rows lie beyond)
    assert not far.all()
    s = _session(w, kv_layout=layout, rope_theta=THETA if rope else 0.0)
    op = OraclePool(_workload(G, prefix, lengths, w.pages_per_request))  # the oracle's pool is a small one
    n, late = w.n_prefill, 3
    pos = w.event_positions() if rope else None
    flags = B.APPEND_ROPE if rope else 0
    s.append_events(n - late, flags=flags, positions=pos)
    s.append_events(n, flags=flags | B.APPEND_DEFER, positions=pos)
    op.append_events(n, positions=pos, theta=THETA)
    if rope:
        _check_rope_step(w, s, op, 0, pos, explicit=False)
    else:
        out, lse, _ = s.decode(0, explicit=False)
        ref, ref_lse = op.attention(0)
        check_close(_out64(w, out), ref, w.dtype, "beyond 4 GiB")
        assert np.max(np.abs(lse.cpu().numpy() - ref_lse)) <= 2e-2
        _check(_out64(w, out), ref, oracle.attention(op.g, op.k, op.v & 0x7FFF, w.dec_request, *w.lists(0), w.q(0), w.scale)[0])
    g = geom_of(w, head_major=layout == B.HEAD_MAJOR)
    for slot in range(n - late, n):  # the deferred rows are in the pool now
        for h in range(HKV):
            at = oracle.elem_offset(g, oracle.phys_row(g, 0, slot), h)
            src = oracle.elem_offset(op.g, oracle.phys_row(op.g, 0, slot), h)
            assert np.array_equal(to_host_bits(s.v_pool[at:at + 128], w.dtype), op.v[src:src + 128])
            k = oracle.widen_pool(w.dtype, to_host_bits(s.k_pool[at:at + 128], w.dtype))
            want = oracle.widen_pool(w.dtype, op.k[src:src + 128])
            assert np.all(np.abs(k - want) <= (2.0 ** -7 * np.abs(want) + 1e-6 if rope else 0))  # (rotated: one unit in the last place)
    plan = np.zeros(8, np.int64)
    q = to_device(w.q(0), w.dtype, s.device)
    s.h.decode_step(0, w.dec_request, w.dec_stream, q, torch.empty_like(q), dbg_plan=plan)
    assert plan[3] > 0  # split
    s.close()
