"""The softmax weights of bf16 pools have fp32's bits with 64-wide heads and 16 of them with 128-wide ones in k_one: an output
element may differ from the exact result by its own rounding to bf16 and by the noise of the sum, and infinite elements
of V come through them."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import THETA, _out64, _session
from util import OraclePool

pytestmark = pytest.mark.gpu

INF = 0x7F80
# (D, prefix, own tokens): short enough for one launch; split into a shared prefix and private lists
FORMS = [(64, 200, [33, 20, 60]), (64, 31, [1, 2, 3]), (128, 150, [33, 20, 60]), (64, 2111, [127, 40, 300])]


def _state(D, prefix, lengths, spoil=None):
    w = W.single_request("weights", "bf16", 16, 4, D, 1.0, 31, prefix, lengths, "random", k_std=2 * D ** -0.5)
    k, v = w.kv_rows(0, w.n_prefill)
    v = v.copy()
    if spoil is not None:
        spoil(v)
    s = _session(w, kv_layout=B.HEAD_MAJOR)
    g = oracle.Geom(w.dtype, w.Hq, w.Hkv, D, pool_tokens=w.pool_tokens, head_major=True)
    kp, vp, tail = g.new_pool(), g.new_pool(), np.zeros(1, np.int64)
    oracle.append(g, kp, vp, w.ev_request, k, v, tail)
    s.h.append_kv(0, w.ev_request, w.ev_stream, to_device(k, "bf16", s.device), to_device(v, "bf16", s.device), parent_stream=w.ev_parent)
    out, _, _ = s.decode(0, explicit=False)
    got = _out64(w, out)
    s.close()

    def exact(values):
        return oracle.attention(g, kp, values, w.dec_request, *w.lists(0), w.q(0), w.scale)[0]

    return got, exact(vp), exact(vp & 0x7FFF)


def _check(got, ref, ref_abs, bits=24):
    """Up to 2^-8 of the element for its rounding to 8 significant bits (half a unit of 2^-7); 1e-5 of sum w |v| for a few hundred fp32 steps and exponents of a few units
    and 2^-bits of it for the weights (of 8 bits they would be off by some 1e-3 of it over these lengths)."""
    bound = np.abs(ref) * 2.0 ** -8 * 1.001 + (1e-5 + 2.0 ** -bits) * ref_abs
    worst = float(np.max(np.abs(got - ref) / bound))
    assert worst <= 1.0


@pytest.mark.parametrize("D,prefix,lengths", FORMS)
def test_outputs_differ_by_their_own_rounding_alone(D, prefix, lengths):
    _check(*_state(D, prefix, lengths), bits=16 if D == 128 else 24)


@pytest.mark.parametrize("D,prefix,lengths", FORMS)
def test_infinite_values_come_through(D, prefix, lengths):
    """+inf in one row of the prefix that every stream sees, -inf in another dim's: these elements are infinite,
    all others as without them."""
    def spoil(v):
        v[7, 1, 5], v[3, 2, D - 1] = INF, INF | 0x8000
    got, _, _ = _state(D, prefix, lengths, spoil)
    _, ref, ref_abs = _state(D, prefix, lengths)
    hit = np.zeros(ref.shape, bool)
    hit[:, 4:8, 5], hit[:, 8:12, D - 1] = True, True
    assert np.all(got[:, 4:8, 5] == np.inf) and np.all(got[:, 8:12, D - 1] == -np.inf)
    _check(np.where(hit, ref, got), ref, ref_abs, bits=16 if D == 128 else 24)


@pytest.mark.parametrize("prefix,own,dtype,D", [
    (p, n, *kind) for p, n in [(48, 16), (200, 16), (1100, 48), (1000, 8)] for kind in [("bf16", 64), ("f32", 64), ("f32", 128)]])
def test_an_infinite_value_in_the_last_row(prefix, own, dtype, D):
    """One thread whose list ends inside a block: the places past its end must not turn its last row's infinity into NaN."""
    w = W.single_request("last", dtype, 8, 2, D, 1.0, 32, prefix, [own], "random", k_std=D ** -0.5)
    k, v = w.kv_rows(0, w.n_prefill)
    v = v.copy()
    v[-1, 0, 3] = INF if dtype == "bf16" else np.inf
    s = _session(w)
    s.h.append_kv(0, w.ev_request, w.ev_stream, to_device(k, dtype, s.device), to_device(v, dtype, s.device), parent_stream=w.ev_parent)
    out, _, _ = s.decode(0, explicit=False)
    got = _out64(w, out)
    s.close()
    hit = np.zeros(got.shape, bool)
    hit[:, :4, 3] = True
    assert np.all(got[hit] == np.inf) and np.all(np.isfinite(got[~hit]))


@pytest.mark.parametrize("D,prefix,lengths", [(128, 1024, [40, 130, 77, 200]), (64, 1024, [40, 130, 77, 200]), (128, 40, [30, 7, 12]), (64, 150, [30, 7, 12])])
def test_fp32_results_are_not_further_off_than_by_short_sums(D, prefix, lengths):
    """Scores of eight sums, outputs of 16 tokens at a time: 1.5e-7 to 1.9e-7 from the exact results over shapes like these (the
    vector-ALU walker 1.6e-7 to 2.1e-7); a chain over all of a row's products gives 2.8e-7 to 4.0e-7."""
    w = W.single_request("sums", "f32", 32, 8, D, 1.0, 33, prefix, lengths, "random", k_std=D ** -0.5)
    s, op = _session(w), OraclePool(w).append_events(w.n_prefill)
    s.append_events(w.n_prefill)
    out, _, _ = s.decode(0, explicit=False)
    ref, _ = op.attention(0)
    assert np.linalg.norm(_out64(w, out) - ref) <= 2.3e-7 * np.linalg.norm(ref)
    s.close()


@pytest.mark.parametrize("D,prefix,rope", [(128, 250, False), (128, 370, True), (64, 400, False), (64, 460, True)])
def test_fp32_lists_read_whole_are_no_further_off_than_the_split_form(D, prefix, rope):
    """Lists of several blocks per wave, 8 streams, in one launch: over 4 draws the error is at most 1.05 of the split form's (the draws leave
    it some 2 % either way: 0.97 to 1.00 over 8 of them; in one chain per wave it is 1.08 to 1.15 with 128-wide heads)."""
    err = {0: [], B.DECODE_ROW_GROUPS: []}
    for seed in range(4):
        w = W.single_request("whole", "f32", 32, 8, D, 1.0, 40 + seed, prefix, [30] * 8, "round_robin", k_std=D ** -0.5)
        pos, qpos = (w.event_positions(), w.q_positions(0)) if rope else (None, None)
        s, op = _session(w, rope_theta=THETA if rope else 0.0), OraclePool(w).append_events(w.n_prefill, **(dict(positions=pos, theta=THETA) if rope else {}))
        s.append_events(w.n_prefill, flags=B.APPEND_ROPE if rope else 0, positions=pos)
        q64 = oracle.widen_pool("f32", w.q(0)).astype(np.float64)
        ref, _ = oracle.attention_q64(op.g, op.k, op.v, w.dec_request, *w.lists(0), oracle.rope(q64, qpos, THETA) if rope else q64, w.scale)
        for flags, errs in err.items():
            out, _, _ = s.decode(0, explicit=False, flags=flags | (B.DECODE_ROPE_Q if rope else 0), position=qpos)
            errs.append(np.linalg.norm(_out64(w, out) - ref) / np.linalg.norm(ref))
        plan = np.zeros(8, np.int64)
        s.h.decode_step(0, w.dec_request, w.dec_stream, out, out, flags=B.DECODE_ROPE_Q if rope else 0, position=qpos, dbg_plan=plan)
        assert plan[3] == 0
        s.close()
    assert np.mean(err[0]) <= 1.05 * np.mean(err[B.DECODE_ROW_GROUPS])
