"""The out-of-place sort around the sizes where its form changes, alone and shared (there from
2^24 elements on), and large blocks whose workspace holds such an array once more."""
import pytest

torch = pytest.importorskip("torch")
import paper_2607_05302_amd as radsort  # noqa: E402
import workloads  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("shared", [False, True], ids=["alone", "shared"])
@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24, (1 << 24) + 12345, (1 << 26) - 1])
@pytest.mark.parametrize("kb,vb", [(4, 4), (8, 4)])
def test_out_of_place_forms(n, kb, vb, shared):
    print(f"out of place n={n} kb={kb} vb={vb} shared={shared}", flush=True)
    k0 = workloads.make_t("zipf", 0x0F5 + kb, n, kb, torch.device(DEV))
    flip = -(1 << (8 * kb - 1))
    want, order = torch.sort(k0 ^ flip, stable=True)
    for call, b in ((radsort.oop_sort_, 1024), (radsort.sort_, 65536)):
        keys, vals = k0.clone(), torch.arange(n, dtype=torch.int32, device=DEV)
        call(keys, vals, block_elems=b, check=True, shared=shared)
        assert torch.equal(keys, want ^ flip)
        assert torch.equal(vals.to(torch.int64), order)
