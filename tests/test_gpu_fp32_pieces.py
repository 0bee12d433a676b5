"""Private pieces of fp32 steps of 128-wide heads (GPU): 64 tokens where they do not make another turn of work-groups or the plan too large
for the kernel arguments, 128 elsewhere -- either way against the oracle, around a piece's and a block's end."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from test_gpu_merge import launches_of
from util import OraclePool, check_close, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,prefix,lengths,inter,piece", [
    (8, 1024, [15, 64, 65, 128], "round_robin", 64), (8, 1024, [63, 16, 129, 17], "random", 64), (1, 300, [193, 1], "random", 64),
    (8, 1024, [250] * 6, "round_robin", 128), (8, 1024, [320] * 8, "random", 64), (8, 1024, [140] * 8, "round_robin", 128),
])
def test_pieces_of_fp32_lists(hkv, prefix, lengths, inter, piece):
    from paper_2502_11517_amd.harness import Session, to_host_bits
    w = W.single_request("pieces", "f32", 4 * hkv, hkv, 128, 1.0, 61, prefix, lengths, inter, k_std=128 ** -0.5)
    s = Session(w)
    s.append_events(w.n_prefill)
    pl, offs, _, ct, _ = w.lists(0)
    pc = int(pl.min())
    private = [int(pl[i]) - pc + int(ct[offs[i]:offs[i + 1]].sum()) for i in range(w.n)]
    plan = np.zeros(8, np.int64)
    s.h.decode_step(0, w.dec_request, w.dec_stream, None, None, lists=w.lists(0), flags=B.DECODE_PLAN_ONLY, dbg_plan=plan)
    assert plan[2] == sum(-(-t // piece) for t in private), (plan, private)
    ref, lse_ref = OraclePool(w).append_events(w.n_prefill).attention()
    for explicit in (True, False):
        out, lse, _ = s.decode(0, explicit=explicit, flags=B.DECODE_ROW_GROUPS)
        check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
        assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= 1e-4
    s.close()


@pytest.mark.parametrize("length", [79, 80, 83])  # by pieces of 64 (and 8 words of room) the plan takes 766 / 770 / 798 of 768 words, by 128 734 / 738 / 766
def test_noalloc_takes_what_fits_by_pieces_of_128(length):
    from paper_2502_11517_amd.harness import Session, to_device, to_host_bits
    w = W.single_request("pieces", "f32", 8, 2, 128, 1.0, 61, 512, [length] * 4, "random", k_std=128 ** -0.5)
    s = Session(w)
    s.append_events(w.n_prefill)
    ref, lse_ref = OraclePool(w).append_events(w.n_prefill).attention()
    q = to_device(w.q(0), w.dtype, s.device)
    out, lse = torch.full_like(q, float("nan")), torch.empty(w.n, w.Hq, dtype=torch.float32, device=s.device)
    s.h.decode_step_noalloc(0, w.dec_request, w.dec_stream, q, out, lists=w.lists(0), out_lse=lse, flags=B.DECODE_ROW_GROUPS)
    check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= 1e-4
    s.close()


@pytest.mark.parametrize("length,piece", [(103, 64), (108, 128)])  # by pieces of 64 the plan has 942 / 971 words, k_plan's arguments hold 960
def test_captured_plans_stay_in_the_arguments_of_their_launch(length, piece):
    from paper_2502_11517_amd.harness import Session, to_device, to_host_bits
    w = W.single_request("pieces", "f32", 8, 2, 128, 1.0, 61, 512, [length] * 4, "random", k_std=128 ** -0.5)
    ref, lse_ref = OraclePool(w).append_events(w.n_prefill).attention()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = Session(w)
        s.append_events(w.n_prefill)
        q = to_device(w.q(0), w.dtype, s.device)
        out, lse = torch.empty_like(q), torch.empty(w.n, w.Hq, dtype=torch.float32, device=s.device)
        step = lambda: s.h.decode_step(0, w.dec_request, w.dec_stream, q, out, lists=w.lists(0), out_lse=lse, flags=B.DECODE_ROW_GROUPS)  # noqa: E731
        launches = launches_of(step)
        assert len(launches) == 3, launches  # k_plan (a work-group per item, four at least), the attention launch, the merge
        pl, offs, _, ct, _ = w.lists(0)
        assert launches[0][0][0] == max(4, sum(-(-(int(pl[i] - pl.min()) + int(ct[offs[i]:offs[i + 1]].sum())) // piece) for i in range(w.n)))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            step()
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
            assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= 1e-4
        s.close()
