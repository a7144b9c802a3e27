"""Batches of arrays sorted on chip around the rules that choose their launches: all long, all
short, just under and over half long, with arrays of other paths among them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2607_05302_amd as radsort  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
T = {4: torch.int32, 8: torch.int64}

MIX = {
    "all long": [2049, 3000, 4096, 4095, 2560] * 13,
    "most long": ([4096, 2049, 3001, 700] * 9 + [0, 1, 2, 63]),
    "half long": [2500, 1000] * 21,
    "under half": [2500, 1000] * 20 + [5],
    "long among larger": [2500] * 10 + [20000] * 25,
    "all short": [2048, 1, 511, 64, 1025] * 11,
    "one long": [4001],
}


@pytest.mark.parametrize("kb,vb", [(4, 0), (4, 4), (4, 8), (8, 0), (8, 4), (8, 8)])
@pytest.mark.parametrize("keys", ["uniform", "few", "high digit"])
@pytest.mark.parametrize("mix", sorted(MIX))
def test_every_array_of_the_batch(mix, keys, kb, vb):
    print(f"small mix {mix} {keys} kb={kb} vb={vb}", flush=True)
    sizes = np.array(MIX[mix])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    n, g = int(off[-1]), torch.Generator(device=DEV).manual_seed(11)
    k0 = torch.randint(-(1 << 31), (1 << 31) - 1, (n,), generator=g, device=DEV, dtype=torch.int64)
    if kb == 8:
        k0 = k0 * 0x9E3779B1 + (k0 >> 7)
    if keys == "few":
        k0 = k0 % 3
    elif keys == "high digit":
        k0 = (k0 & 0xFF) << (8 * kb - 8)
    k0 = k0.to(T[kb])
    dk = k0.clone()
    dv = torch.arange(n, device=DEV).to(T[vb]) if vb else None
    radsort.sort_segments_(dk, dv, off, tuning=None, check=True)
    flip = -(1 << (8 * kb - 1))
    for a, b in zip(off[:-1].astype(np.int64), off[1:].astype(np.int64)):
        want, order = torch.sort(k0[a:b] ^ flip, stable=True)
        assert torch.equal(dk[a:b], want ^ flip)
        if vb:
            assert torch.equal(dv[a:b].to(torch.int64), order + int(a))
