"""Batches of arrays that are sorted on chip, most of them short: a few of the large shape
among very many of the small one, spread out or side by side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2607_05302_amd as radsort  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (arrays, of them long ones, where: a start and a step)
MIX = [(200000, 1, 123456, 1), (200000, 40, 77, 4096), (100000, 600, 50000, 1), (4096, 8, 5, 512),
       (4097, 3, 0, 4096), (5, 1, 4, 1), (3000000, 2, 2999990, 9)]


def sizes_of(arrays, longs, start, step):
    sizes = np.full(arrays, 24, np.int64)
    sizes[::3] = 31
    at = start + step * np.arange(longs)
    at = at[at < arrays]
    sizes[at] = 2049 + 977 * np.arange(len(at)) % 2048
    return sizes


def best_ms(call, reps=3):
    out = []
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        call()
        e1.record()
        e1.synchronize()
        out.append(e0.elapsed_time(e1))
    return min(out)


@pytest.mark.parametrize("kb,vb", [(4, 4), (8, 8)])
@pytest.mark.parametrize("mix", MIX, ids=lambda m: "-".join(map(str, m)))
def test_few_long_arrays_among_short_ones(mix, kb, vb):
    """The order of every array is a stable sort's; and the long arrays cost no more than
    their own work: a batch of short arrays alone, the lone sort of each long one (40 us),
    and a millisecond."""
    print(f"mix {mix} kb={kb} vb={vb}", flush=True)
    sizes = sizes_of(*mix)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    n = int(off[-1])
    g = torch.Generator(device=DEV).manual_seed(7)
    tk = {4: torch.int32, 8: torch.int64}[kb]
    keys = torch.randint(0, 1 << 20, (n,), generator=g, device=DEV, dtype=tk)
    keys0 = keys.clone()
    vals = torch.arange(n, device=DEV, dtype=torch.int32 if vb == 4 else torch.int64)
    off_dev = torch.from_numpy(off.view(np.int64)).to(DEV)
    radsort.sort_segments_(keys, vals, off, tuning=None, check=True, offsets_dev=off_dev)
    seg = torch.repeat_interleave(torch.arange(len(sizes), device=DEV),
                                  torch.from_numpy(sizes).to(DEV))
    want, order = torch.sort(seg * (1 << 20) + keys0.to(torch.int64), stable=True)
    assert torch.equal(keys.to(torch.int64), want % (1 << 20))
    assert torch.equal(vals.to(torch.int64), order)

    short = np.minimum(sizes, 24)
    soff = np.concatenate([[0], np.cumsum(short)]).astype(np.uint64)
    soff_dev = torch.from_numpy(soff.view(np.int64)).to(DEV)
    ws = torch.empty(1 << 16, dtype=torch.uint8, device=DEV)
    alone = best_ms(lambda: radsort.sort_segments_(keys, vals, soff, tuning=None, workspace=ws,
                                                   offsets_dev=soff_dev))
    mixed = best_ms(lambda: radsort.sort_segments_(keys, vals, off, tuning=None, workspace=ws,
                                                   offsets_dev=off_dev))
    print(f"short arrays alone {alone:.3f} ms, with {int((sizes > 2048).sum())} long ones "
          f"{mixed:.3f} ms", flush=True)
    assert mixed <= alone + 0.04 * (sizes > 2048).sum() + 1.0
