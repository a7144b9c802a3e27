"""The phases of a timed sort (RADSORT_F_TIMING): a phase that a sort does not run takes no
time, and the phases add up to no more than the whole."""
import pytest
import torch

import paper_2607_05302_amd as radsort
import workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("kw,counts", [
    ({}, False),                      # all rounds planned from one count, in setup
    (dict(block_elems=512), True),    # rounds that count their own input
    (dict(seq_draws=True), True),
], ids=["planned", "small-blocks", "sequential-draws"])
def test_counting_is_reported_where_it_is_done(kw, counts):
    n = (1 << 23) + 5
    print(f"phases: n={n} {kw}", flush=True)
    keys = workloads.uniform_t(0x717E, n, 4, DEV)
    vals = torch.arange(n, dtype=torch.int32, device=DEV)
    radsort.sort_(keys.clone(), vals.clone(), check=True, **kw)
    radsort.sort_(keys, vals, timing=True, **kw)
    s = radsort.last_stats()
    assert len(s["round_ms"]) == 4 and all(t > 0 for t in s["round_ms"])
    assert all((t > 0) == counts for t in s["count_ms"]), s["count_ms"]
    assert s["setup_ms"] > 0 and s["fixup_ms"] > 0 and s["finalize_ms"] > 0
    parts = (s["setup_ms"] + sum(s["round_ms"]) + sum(s["count_ms"]) + s["fixup_ms"]
             + s["finalize_ms"])
    assert parts <= s["total_ms"] * 1.001 + 0.01
