"""The merge launch (GPU) where its width changes with the number of parts, and results at any multiple of 4 bytes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

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
