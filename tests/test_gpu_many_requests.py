"""Which request a shared-prefix work-group belongs to (GPU): more requests than a wave has lanes, requests without a shared
prefix between, in front of and behind those that have one."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from util import OraclePool, check_close, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("n,pmin,pmax", [(2, 40, 70), (64, 70, 140), (65, 30, 100), (130, 20, 140)])
def test_requests_of_the_shared_prefix_work_groups(n, pmin, pmax, dtype, D):
    from paper_2502_11517_amd.harness import Session, to_host_bits
    w = W.config4(n_requests=n, seed=7 + n, pmin=pmin, pmax=pmax, hq=4, hkv=2, smin=1, smax=2)
    w.dtype, w.D, w.scale = dtype, D, D ** -0.5
    s = Session(w)
    s.append_events(w.n_prefill)
    ref, lse_ref = OraclePool(w).append_events(w.n_prefill).attention()
    plan = np.zeros(8, np.int64)
    s.h.decode_step(0, w.dec_request, w.dec_stream, None, None, flags=B.DECODE_PLAN_ONLY, dbg_plan=plan)
    prefixes = np.array([int(w.lists(0)[0][np.nonzero(w.dec_request == r)[0]].min()) for r in range(n)])
    assert plan[5] == prefixes[prefixes >= 64].sum() and (n == 64 or (prefixes < 64).any())
    out, lse, _ = s.decode(0, explicit=False, flags=B.DECODE_ROW_GROUPS)
    check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= (2e-2 if dtype == "bf16" else 1e-4)
    s.close()
