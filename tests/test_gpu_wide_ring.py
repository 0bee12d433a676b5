"""The ring of tiles of the work-groups that serve four row groups (GPU): chunks of one tile to more than twice the ring, ragged ends of
one token to a tile less one, pages smaller than a wave's eight rows (an address per row) up to whole tiles, deferred rows inside."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2502_11517_amd import binding as B
from paper_2502_11517_amd import workloads as W
from util import OraclePool, check_close, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page", [0, 4, 8, 64])
@pytest.mark.parametrize("prefix,tiles,last", [(64, 2, 64), (97, 2, 33), (4129, 4, 33), (6175, 6, 31), (8225, 8, 33), (10273, 10, 33)])
def test_tiles_of_a_chunk(prefix, tiles, last, page):
    """One stream group of 40 rows over 8 kv heads; the chunk holds `tiles` tiles, the last one `last` tokens."""
    from paper_2502_11517_amd.harness import Session, to_host_bits
    w = W.single_request("ring", "bf16", 64, 8, 128, 1.0, 71, prefix, [1] * 5, "round_robin", k_std=128 ** -0.5)
    if page:
        pages = -(-(w.n_prefill + 8) // page)
        w.page_tokens, w.n_phys_pages, w.pages_per_request = page, pages + 3, pages
        w.page_table = np.random.default_rng(3).permutation(pages + 3)[:pages].astype(np.int32)[None, :]
    s = Session(w)
    s.append_events(w.n_prefill - 6)
    s.append_events(w.n_prefill, flags=B.APPEND_DEFER)  # the prefix' last row and the five forks'
    plan = np.zeros(8, np.int64)
    s.h.decode_step(0, w.dec_request, w.dec_stream, None, None, flags=B.DECODE_PLAN_ONLY | B.DECODE_FOUR_GROUPS, dbg_plan=plan)
    assert plan[5] == prefix and plan[4] == 32 * tiles and (prefix - 1) % plan[4] + 1 == last
    ref, lse_ref = OraclePool(w).append_events(w.n_prefill).attention()
    out, lse, _ = s.decode(0, explicit=False, flags=B.DECODE_FOUR_GROUPS)
    check_close(to_f64(w, to_host_bits(out, w.dtype)), ref, w.dtype, "out")
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= 2e-2
    s.close()
