"""The host's plan of a batch of very many middle-sized arrays (no GPU needed)."""
import time

import numpy as np

import paper_2607_05302_amd as radsort


def test_plan_of_many_arrays_is_quick():
    """The tables of so many arrays leave no room for groups of any size, which the plan has
    to see without trying them all: 16 bytes of offsets read per array and pass, a few passes
    (each about 10 ms), and not the hundred sizes between the largest and the smallest group
    (840 ms)."""
    off = np.arange(2_000_001, dtype=np.uint64) * np.uint64(8193)
    best = 1e9
    for _ in range(3):
        t = time.perf_counter()
        assert radsort.segments_workspace_bytes(off, 4, 0, None) > 0
        best = min(best, time.perf_counter() - t)
    assert best < 0.3, best
