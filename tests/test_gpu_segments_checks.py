"""A batch whose device offsets do not hold the host's values is reported, and nothing
outside the planes and the workspace is written (tests/test_seg_plan_host.py models the
same checks on the CPU).  All offsets lie inside the planes."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
import paper_2607_05302_amd as radsort  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
HOST = [8193, 9000, 70001, 150000, 200001, 8193] * 10


def device_sizes(name):
    dev = list(HOST)
    if name == "fewer":
        dev[1], dev[2] = dev[1] + dev[2], 0
    elif name == "more":
        dev[3:4] = [75000, 75000]  # one array more; the last of the batch is not looked at
        dev = dev[:len(HOST)]
    elif name == "none":
        dev = [0] * len(HOST)
    elif name == "reversed":
        dev = sorted(HOST, reverse=True)
    return dev


@pytest.mark.parametrize("kb,vb", [(4, 4), (8, 0)])
@pytest.mark.parametrize("name", ["fewer", "more", "none", "reversed"])
def test_other_offsets_on_the_device_are_reported(name, kb, vb):
    print(f"device offsets: {name} kb={kb} vb={vb}", flush=True)
    host = sorted(HOST) if name == "reversed" else HOST
    off = np.concatenate([[0], np.cumsum(host)]).astype(np.uint64)
    wrong = np.concatenate([[0], np.cumsum(device_sizes(name))]).astype(np.int64)
    n = int(off[-1])
    tk = {4: torch.int32, 8: torch.int64}[kb]
    size = radsort.segments_workspace_bytes(off, kb, vb, None)
    pad = 1 << 16
    planes = torch.full((n + 2 * pad,), 0x5A5A5A5A, dtype=tk, device=DEV)
    buf = torch.full((size + 2 * pad,), 0x5A, dtype=torch.uint8, device=DEV)
    keys = planes[pad:pad + n]
    fresh = workloads.uniform_t(0x0FF5 + kb, n, kb, DEV).to(tk)
    keys.copy_(fresh)
    vals = torch.arange(n, dtype=torch.int32, device=DEV) if vb else None
    ws = buf[pad:pad + size]
    with pytest.raises(radsort.RadsortError):
        radsort.sort_segments_(keys, vals, off, tuning=None, workspace=ws, check=True,
                               offsets_dev=torch.from_numpy(wrong).to(DEV))
    assert radsort.last_stats()["error_bits"] == 2
    for t in (planes[:pad], planes[pad + n:]):
        assert bool((t == 0x5A5A5A5A).all())
    for t in (buf[:pad], buf[pad + size:]):
        assert bool((t == 0x5A).all())
    # the same workspace, with the host's values
    keys.copy_(fresh)
    if vb:
        vals.copy_(torch.arange(n, dtype=torch.int32, device=DEV))
    radsort.sort_segments_(keys, vals, off, tuning=None, workspace=ws, check=True,
                           offsets_dev=torch.from_numpy(off.view(np.int64)).to(DEV))
    flip = -(1 << (8 * kb - 1))
    for a, b in zip(off[:-1].astype(np.int64), off[1:].astype(np.int64)):
        want, order = torch.sort(fresh[a:b] ^ flip, stable=True)
        assert torch.equal(keys[a:b], want ^ flip)
        if vb:
            assert torch.equal(vals[a:b].to(torch.int64), order + int(a))
