"""Rows whose score is the lowest finite value (an additive mask carried in one head dim): times log2(e) it is -inf, and
a whole block of them must weigh nothing, whichever wave or chunk has it, first or last -- in every partials kernel."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from paper_2502_11517_amd.harness import to_device
from test_gpu_parity import _check_step, _session
from util import OraclePool

pytestmark = pytest.mark.gpu

LOWEST = np.float32(-3.3895314e38)  # of bf16
KINDS = [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)]


def _check(dtype, D, hq, hkv, prefix, lengths, masked, flags=0):
    """masked: rows that every query scores LOWEST"""
    w = W.single_request("lowest", dtype, hq, hkv, D, 1.0, 41, prefix, lengths, "random", k_std=D ** -0.5)
    cast = W.f32_to_bf16_bits if dtype == "bf16" else np.float32
    k, v = w.kv_rows(0, w.n_prefill)
    q = w.q(0).copy()
    k = k.copy()
    k[:, :, 0], q[:, :, 0] = cast(np.float32(0)), cast(np.float32(1))
    k[masked, :, 0] = cast(LOWEST)
    s, op = _session(w, kv_layout=B.HEAD_MAJOR), OraclePool(w, head_major=True)
    s.h.append_kv(0, w.ev_request, w.ev_stream, to_device(k, dtype, s.device), to_device(v, dtype, s.device), parent_stream=w.ev_parent)
    oracle.append(op.g, op.k, op.v, w.ev_request, k, v, op.tail)
    _check_step(w, s, op, explicit=False, q=q, flags=flags)
    s.close()


# prefixes: short enough for one launch (three blocks of a wave at 300 tokens); one chunk of the split form; several
@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("prefix,lo,hi", [(96, 0, 32), (96, 64, 96), (96, 0, 64), (300, 0, 32), (300, 256, 288), (1000, 0, 32), (1000, 960, 1000),
                                          (1000, 64, 192), (5000, 0, 512)])
def test_a_block_of_the_prefix(dtype, D, prefix, lo, hi):
    _check(dtype, D, 8, 2, prefix, [40, 3], slice(lo, hi))


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("prefix", [40, 1000])
def test_all_rows_of_the_threads(dtype, D, prefix):
    _check(dtype, D, 8, 2, prefix, [40, 3], slice(prefix, None))


@pytest.mark.parametrize("lo,hi", [(0, 32), (32, 160), (1472, 1500)])
def test_a_block_of_the_prefix_under_four_row_groups(lo, hi):
    """5 streams x 8 heads per kv head = 40 stacked rows: the work-groups that serve four row groups each."""
    _check("bf16", 128, 16, 2, 1500, [30, 7, 140, 20, 26], slice(lo, hi), flags=B.DECODE_FOUR_GROUPS)
