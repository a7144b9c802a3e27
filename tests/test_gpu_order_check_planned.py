"""The ordering check (see test_gpu_order_check.py) on the rounds that one-call sorts plan
ahead: look-back over all tiles with a word per tile and digit, and through the ring with its
slots used again; rounds left out; the packed last round, also of the general round kernel.
And on the rounds of the step interface, which count their own input."""
import ctypes

import pytest
import torch

import paper_2607_05302_amd as radsort
import test_gpu_order_check as check
import workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [
    # dist, n, key bytes, payload, digit bits, b, flags
    ("uniform", 50001, 4, True, 8, 1024, 0),                            # a word per tile
    ("zipf", (1 << 22) + 3, 4, True, 8, 2048, radsort.F_SHARED),
    ("uniform", (1 << 21) + 8191, 8, True, 8, 8192, 0),
    ("low20", (1 << 22) + 12345, 8, False, 8, 1024, radsort.F_SHARED),  # rounds left out
    ("equal", 300001, 4, True, 8, 1024, 0),
    ("uniform", (1 << 25) + 77, 4, True, 8, 2048, radsort.F_SHARED),    # the ring, used again
    ("zipf", (1 << 25) + (1 << 24) - 1, 4, False, 8, 16384, 0),
    ("zipf", (1 << 24) + (1 << 22), 8, True, 8, 4096, 0),
    ("uniform", (1 << 25) + 5, 8, True, 7, 2048, radsort.F_SHARED),
    ("zipf", (1 << 20) + 11, 4, True, 10, 512, 0),                      # packed, k_round
    ("uniform", (1 << 20) + 1, 4, True, 8, 1024, radsort.F_SEQ_DRAWS),
]


def inputs(dist, n, kb, pay, seed):
    k0 = workloads.make_t(dist, seed, n, kb, torch.device(DEV))
    vals = torch.arange(n, dtype=torch.int32 if kb == 4 else torch.int64, device=DEV) if pay \
        else None
    return k0, vals


def expect(k0, keys, vals):
    flip = -(1 << (8 * keys.element_size() - 1))
    want, order = torch.sort(k0 ^ flip, stable=True)
    assert torch.equal(keys, want ^ flip)
    if vals is not None:
        assert torch.equal(vals.to(torch.int64), order)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_planned_rounds_draw_no_block_before_its_loads(case):
    dist, n, kb, pay, bits, b, flags = case
    print(f"ordering check, planned rounds: {case}", flush=True)
    lib = check.debug_lib()
    k0, vals = inputs(dist, n, kb, pay, 0x0D1E + b)
    keys = k0.clone()
    rc, bits_set = check.run(lib, keys, vals, bits, b, flags | radsort.F_DEBUG_ORDER)
    assert rc == radsort.OK and bits_set == 0, (radsort.strerror(rc), bits_set)
    expect(k0, keys, vals)


@pytest.mark.parametrize("n,kb,b", [((1 << 22) + 9, 4, 1024), ((1 << 25) + 77, 4, 2048),
                                    ((1 << 21) + 5, 8, 2048)])
def test_planned_rounds_report_wrong_marks(n, kb, b):
    """With the planted tag the check reports on every form (the kernels end normally)."""
    print(f"ordering check, planned rounds, planted tag: n={n}", flush=True)
    k0, vals = inputs("uniform", n, kb, True, 0x0D2F)
    rc, bits_set = check.run(check.debug_lib(), k0, vals, 8, b,
                             radsort.F_DEBUG_ORDER | radsort.F_DEBUG_PLANT)
    assert rc == radsort.E_ORDER and bits_set & 4


@pytest.mark.parametrize("n,kb,bits,b,flags", [
    (50001, 4, 8, 1024, 0), ((1 << 20) + 5, 4, 8, 1024, 0), (1 << 24, 4, 8, 2048, 0), ((1 << 23) + 12345, 8, 8, 1024, 0),
    (1 << 22, 4, 8, 512, 0), (1 << 21, 4, 11, 1024, 0), (1 << 22, 4, 8, 1024, radsort.F_SEQ_DRAWS)])
@pytest.mark.parametrize("plant", [False, True], ids=["right", "planted"])
def test_step_rounds_draw_no_block_before_its_loads(n, kb, bits, b, flags, plant):
    print(f"ordering check, step interface: n={n} kb={kb} bits={bits} b={b} {plant}", flush=True)
    lib = check.debug_lib()
    k0, vals = inputs("uniform", n, kb, True, 0x0D3E + b)
    keys = k0.clone()
    o = radsort.Opts()
    o.block_elems = b
    o.flags = flags | radsort.F_DEBUG_ORDER | (radsort.F_DEBUG_PLANT if plant else 0)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    st = ctypes.c_void_p()
    assert lib.radsort_state_create(ctypes.byref(st), ctypes.c_void_p(keys.data_ptr()),
                                    ctypes.c_void_p(vals.data_ptr()), n, kb, kb, bits,
                                    ctypes.byref(o)) == radsort.OK
    assert lib.radsort_state_setup(st, stream) == radsort.OK
    for _ in range((8 * kb + bits - 1) // bits):
        assert lib.radsort_state_round(st, stream) == radsort.OK
    assert lib.radsort_state_finalize(st, stream) == radsort.OK
    rc = lib.radsort_state_read(st, None, None, None, None, stream)
    lib.radsort_state_destroy(st)
    # a round draws blocks only where some digit fills one (at 50001 keys none does)
    digits = [(k0 >> (bits * r)) & ((1 << bits) - 1) for r in range((8 * kb + bits - 1) // bits)]
    draws = any(int(torch.bincount(d.to(torch.int64)).max()) >= b for d in digits)
    assert draws == (n != 50001)
    assert rc == (radsort.E_ORDER if plant and draws else radsort.OK)
    if not plant:
        expect(k0, keys, vals)
