"""The host's plan of a batch of very many middle-sized arrays (no GPU needed): its time, and
what it does when host memory runs out."""
import os
import subprocess
import sys
import time

import numpy as np

import paper_2607_05302_amd as radsort

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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

OUT_OF_MEMORY = """
import resource
import numpy as np
import paper_2607_05302_amd as radsort
off = np.arange(6_000_001, dtype=np.uint64) * np.uint64(9000)
few = off[:3]
assert radsort.segments_workspace_bytes(few, 4, 4, None) > 0  # the library is loaded
pages = int(open("/proc/self/statm").read().split()[0])
soft, hard = resource.getrlimit(resource.RLIMIT_AS)
resource.setrlimit(resource.RLIMIT_AS, (pages * resource.getpagesize() + (8 << 20), hard))
short = radsort.segments_workspace_bytes(off, 4, 4, None)
resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
assert short == 0, short
assert radsort.segments_workspace_bytes(few, 4, 4, None) > 0
print("refused")
"""


def test_plan_out_of_host_memory_is_refused():
    """A plan that host memory does not hold is an error of the call, not the end of the
    process (a C++ exception must not leave a C entry point)."""
    r = subprocess.run([sys.executable, "-c", OUT_OF_MEMORY], cwd=ROOT, capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0 and "refused" in r.stdout, (r.returncode, r.stderr[-500:])
