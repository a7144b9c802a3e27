"""GPU parity: the HIP path against the sequential oracle, through the C ABI.

Every comparison is exact.  Radsort's integer state is deterministic.  With
RADSORT_F_SEQ_DRAWS the GPU draws blocks from the pool in the same order as the
sequential algorithm, so pi, P and f after setup and after every round must
equal the oracle's bit for bit.  Without it (the default) a tile draws the same
pool entries in (digit, block) order: P, f, the permuted representation read in
logical order and the final arrays must still equal the oracle's, pi must be a
permutation, and the sets of physical blocks in the head start, the allocated
range and the unallocated tail must equal the oracle's (pi itself is not unique
across valid draw orders).
"""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
import paper_2607_05302_amd as radsort  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NP = {4: np.uint32, 8: np.uint64}
TV = {4: torch.int32, 8: torch.int64}


def to_dev(a):
    a = np.ascontiguousarray(a)
    view = {4: np.int32, 8: np.int64}[a.dtype.itemsize]
    return torch.from_numpy(a.view(view)).to(DEV)


def from_dev(t, width):
    return t.cpu().numpy().view(NP[width])


def inputs(dist, n, kb, vb, seed=1):
    keys = workloads.make(dist, seed * 1000003 + n, n, kb)
    vals = np.arange(n, dtype=NP[vb]) if vb else None
    return keys, vals


def say(*a):
    print(*a, flush=True)


# ---------------------------------------------------------------- a0: histograms

@pytest.mark.parametrize("kb,bits", [(4, 8), (4, 4), (4, 11), (8, 8), (8, 11), (4, 1)])
@pytest.mark.parametrize("n", [0, 1, 1000, (1 << 20) + 5])
def test_histograms(kb, bits, n):
    say(f"histograms kb={kb} bits={bits} n={n}")
    keys, _ = inputs("uniform", n, kb, 0)
    sigma, nt = oracle.digit_params(kb, bits)
    h = radsort.histograms(to_dev(keys), bits)
    torch.cuda.synchronize()
    got = h.cpu().numpy().view(np.uint32).astype(np.uint64)
    assert np.array_equal(got, oracle.histograms(keys, sigma, nt))


# ---------------------------------------------------------------- a1-a7: rounds

ROUND_CASES = [
    # (dist, n, key bytes, payload bytes, digit bits, b)
    ("uniform", 5000, 4, 4, 8, 64),
    ("uniform", (1 << 16) + 777, 4, 4, 8, 1024),
    ("uniform", 1 << 20, 4, 4, 8, 1024),
    ("uniform", 300000, 4, 0, 8, 256),
    ("uniform", 100000, 8, 4, 8, 512),
    ("uniform", 70000, 8, 8, 11, 1024),
    ("uniform", 50000, 4, 8, 4, 128),
    ("equal", 200000, 4, 4, 8, 1024),
    ("sorted", 200000, 4, 4, 8, 1024),
    ("zipf", 300000, 8, 4, 8, 1024),
    ("low20", 200000, 8, 0, 8, 1024),
    ("few", 123457, 4, 4, 8, 64),
    ("uniform", 1000, 4, 4, 8, 4096),       # fewer elements than one block
    ("uniform", 70000, 4, 4, 8, 16384),     # blocks larger than a tile
    ("uniform", 3, 4, 4, 8, 64),
]


def check_pi(pi, prev, opi, i_out, sigma, exact, r):
    """pi after round r: equal to the oracle's (sequential draws).  Otherwise it
    must follow from the GPU's own pi before the round (prev) as Alg. 6 builds it
    from any valid draw order: the round used the pool entries prev[0 .. i_out)
    (i_out: the oracle's count of blocks taken), which now form the allocated
    range sigma .. f-1 in some order; the next head start is prev[i_out ..
    i_out + sigma) and the tail prev[i_out + sigma ..], both in order."""
    pi = pi.astype(np.uint64)
    if exact:
        assert np.array_equal(pi, opi), f"pi differs after round {r}"
        return
    prev = prev.astype(np.uint64)
    f = i_out + sigma
    assert np.array_equal(pi[:sigma], prev[i_out:f]), f"head start after round {r}"
    assert np.array_equal(np.sort(pi[sigma:f]), np.sort(prev[:i_out])), f"allocated, round {r}"
    assert np.array_equal(pi[f:], prev[f:]), f"tail after round {r}"


@pytest.mark.parametrize("seq", [True, False], ids=["seqdraws", "tiledraws"])
@pytest.mark.parametrize("case", ROUND_CASES, ids=lambda c: "-".join(map(str, c)))
def test_rounds_match_oracle(case, seq):
    dist, n, kb, vb, bits, b = case
    say(f"rounds {case} seq_draws={seq}")
    keys, vals = inputs(dist, n, kb, vb)
    sigma, nt = oracle.digit_params(kb, bits)
    dk = to_dev(keys)
    dv = to_dev(vals) if vb else None
    st = radsort.State(dk, dv, digit_bits=bits, block_elems=b, seq_draws=seq)
    R = oracle.Radsort(keys, vals, sigma, nt, b)
    st.setup()
    R.setup()
    # digits of more than 8 bits always draw in the sequential order
    exact = seq or bits > 8
    prev = None
    for r in range(-1, nt):
        if r >= 0:
            st.round()
            R.round(nt - 1 - r)
        pi, pidx, plen, f = st.read()
        assert f == R.f, (r, f, R.f)
        check_pi(pi, prev, R.pi(), R.i_out, sigma, exact or r < 0, r)
        prev = pi
        oidx, olen = R.P()
        assert np.array_equal(pidx.astype(np.uint64), oidx), f"P idx differs after round {r}"
        assert np.array_equal(plen.astype(np.uint64), olen), f"P len differs after round {r}"
        lk, lv = st.logical()
        ok, ov, cnt = R.logical()
        assert cnt == n
        assert np.array_equal(from_dev(lk, kb).astype(np.uint64), ok), f"logical keys, round {r}"
        if vb:
            assert np.array_equal(from_dev(lv, vb).astype(np.uint64), ov), f"logical payload {r}"
    st.close()


# ---------------------------------------------------------------- a8: finalize

@pytest.mark.parametrize("case", ROUND_CASES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("mode", ["parallel", "sequential"])
def test_finalize_matches_oracle(case, mode):
    dist, n, kb, vb, bits, b = case
    if mode == "sequential" and n > 300000:
        pytest.skip("the one-workgroup finalize is slow at this size")
    say(f"finalize {mode} {case}")
    keys, vals = inputs(dist, n, kb, vb, seed=2)
    sigma, nt = oracle.digit_params(kb, bits)
    dk = to_dev(keys)
    dv = to_dev(vals) if vb else None
    st = radsort.State(dk, dv, digit_bits=bits, block_elems=b)
    st.setup()
    for _ in range(nt):
        st.round()
    (st.finalize if mode == "parallel" else st.finalize_sequential)()
    st.read()  # waits and reports device-side errors
    ok, ov = oracle.radsort(keys, vals, sigma, nt, b)
    assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ok)
    if vb:
        assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ov)
    st.close()


# ---------------------------------------------------------------- end to end

E2E = [
    ("uniform", 1 << 20, 4, 4, 8, 1024),      # the small configuration
    ("uniform", (1 << 20) + 12345, 4, 4, 8, 1024),
    ("uniform", 1 << 22, 4, 4, 8, 1024),
    ("uniform", 1 << 21, 8, 4, 8, 1024),
    ("uniform", 1 << 20, 4, 0, 8, 2048),
    ("uniform", 1 << 20, 8, 8, 4, 1024),
    ("uniform", 1 << 20, 4, 4, 11, 1024),
    ("zipf", 1 << 21, 8, 4, 8, 1024),
    ("equal", 1 << 21, 8, 4, 8, 1024),
    ("sorted", 1 << 21, 8, 4, 8, 1024),
    ("low20", 1 << 21, 8, 4, 8, 1024),
    ("reverse", 1 << 20, 4, 4, 8, 1024),
    ("uniform", 2, 4, 4, 8, 1024),
    ("uniform", 65, 4, 4, 8, 64),
    ("uniform", 0, 4, 4, 8, 1024),            # empty
    ("uniform", 1, 8, 8, 8, 1024),
    ("uniform", 1024, 4, 4, 8, 1024),         # exactly one block
    ("uniform", 2 * 256 * 64, 4, 4, 8, 64),   # exactly the 2 sigma b of the head blocks
    ("uniform", 2000, 8, 4, 1, 64),           # 1-bit digits: 64 rounds, the most there are
    ("zipf", 30000, 4, 4, 2, 64),
    ("few", 40000, 4, 4, 6, 256),
    # the packed last round: many buckets within one block of A, blocks larger than a
    # tile, fewer elements than a block, ragged tails
    ("uniform", 300, 4, 4, 8, 64),
    ("uniform", 70000, 4, 4, 8, 16384),
    ("uniform", 5000, 8, 4, 8, 4096),
    ("zipf", 123457, 4, 0, 8, 128),
    ("low20", 1000003, 8, 8, 8, 512),
    # wide records (12 and 16 bytes: smaller tiles) and 11-bit digits, packed, ragged
    ("uniform", (1 << 20) + 777, 8, 8, 11, 1024),
    ("zipf", 777777, 4, 8, 11, 2048),
    ("uniform", 3000001, 8, 8, 8, 4096),
]


@pytest.mark.parametrize("case", E2E, ids=lambda c: "-".join(map(str, c)))
def test_sort_pairs_matches_oracle(case):
    dist, n, kb, vb, bits, b = case
    say(f"sort_pairs {case}")
    keys, vals = inputs(dist, n, kb, vb, seed=3)
    sigma, nt = oracle.digit_params(kb, bits)
    dk = to_dev(keys)
    dv = to_dev(vals) if vb else None
    radsort.sort_(dk, dv, digit_bits=bits, block_elems=b, check=True)
    ok, ov = oracle.radsort(keys, vals, sigma, nt, b)
    assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ok)
    if vb:
        assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ov)


@pytest.mark.parametrize("case", E2E[:8], ids=lambda c: "-".join(map(str, c)))
def test_oop_matches_oracle(case):
    dist, n, kb, vb, bits, b = case
    say(f"oop {case}")
    keys, vals = inputs(dist, n, kb, vb, seed=4)
    sigma, nt = oracle.digit_params(kb, bits)
    dk = to_dev(keys)
    dv = to_dev(vals) if vb else None
    radsort.oop_sort_(dk, dv, digit_bits=bits, block_elems=b, check=True)
    ok, ov = oracle.oop_lsd(keys, vals, sigma, nt)
    assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ok)
    if vb:
        assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ov)


def test_caller_workspace_and_stats():
    n = 1 << 20
    keys, vals = inputs("uniform", n, 4, 4, seed=5)
    need = radsort.workspace_bytes(n, 4, 4, 8, 1024)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    dk, dv = to_dev(keys), to_dev(vals)
    radsort.sort_(dk, dv, workspace=ws, check=True)
    ok, ov = oracle.radsort(keys, vals, 256, 4, 1024)
    assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)
    assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov)
    s = radsort.last_stats()
    assert s["workspace_bytes"] == need and s["error_bits"] == 0


def test_repeated_calls_on_one_stream():
    """Back-to-back sorts reuse nothing stale: the ring, counters and pi are reset."""
    n = 1 << 18
    s = torch.cuda.Stream()
    ws = torch.empty(radsort.workspace_bytes(n, 4, 4, 8), dtype=torch.uint8, device=DEV)
    for seed in range(3):
        keys, vals = inputs("uniform", n, 4, 4, seed=10 + seed)
        dk, dv = to_dev(keys), to_dev(vals)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            radsort.sort_(dk, dv, workspace=ws, stream=s, check=True)
        s.synchronize()
        ok, ov = oracle.radsort(keys, vals, 256, 4, 1024)
        assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)
        assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov)


def test_ring_wraps_within_a_round():
    """2^24 pairs: more tiles per round than look-back ring slots."""
    n = 1 << 24
    say(f"ring wrap n={n}")
    keys, vals = inputs("uniform", n, 4, 4, seed=6)
    dk, dv = to_dev(keys), to_dev(vals)
    radsort.sort_(dk, dv, check=True)
    ok, ov = oracle.radsort(keys, vals, 256, 4, 1024)
    assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)
    assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov)


# ---------------------------------------------------------------- full sizes

@pytest.mark.parametrize("b", [2048, 1024])
def test_large_uniform_u32_matches_oracle(b):
    """n = 2^28 uint32 + index: the benchmark's input, compared element by element
    with the oracle's result (b = 2048 with the tile draw order the benchmark runs,
    b = 1024 with the sequential one); the out-of-place baseline on the same input
    too."""
    n = 1 << 28
    say(f"2^28 uint32 b={b}")
    keys = workloads.uniform(workloads.SEED_LARGE, n, 4)
    vals = np.arange(n, dtype=np.uint32)
    ok, ov = oracle.radsort(keys, vals, 256, 4, b)
    dk, dv = to_dev(keys), to_dev(vals)
    # b = 1024 also covers the sequential draw order at full size
    radsort.sort_(dk, dv, block_elems=b, check=True, seq_draws=(b == 1024))
    assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)
    assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov)
    if b == 2048:
        dk, dv = to_dev(keys), to_dev(vals)
        radsort.oop_sort_(dk, dv, block_elems=b, check=True)
        assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)
        assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov)


def test_large_tile_keys_only_ragged():
    """n = 2^28 + 12345 uint32 keys without payload, b = 4096: the 16384-slot tile of
    large sorts with a ragged last tile and a partial last block, compared element by
    element with the oracle."""
    n = (1 << 28) + 12345
    say(f"2^28+12345 uint32 keys only b=4096")
    keys = workloads.uniform(0x5EED00A1, n, 4)
    ok, _ = oracle.radsort(keys, None, 256, 4, 4096)
    dk = to_dev(keys)
    radsort.sort_(dk, None, block_elems=4096, check=True)
    assert np.array_equal(from_dev(dk, 4).astype(np.uint64), ok)


def test_large_tile_u64_keys_only_ragged():
    """n = 2^28 + 777 uint64 keys without payload, b = 4096: the large tile of 8-byte
    keys (8192 slots, one workgroup per compute unit) with a ragged last tile,
    compared element by element with the oracle."""
    n = (1 << 28) + 777
    say(f"2^28+777 uint64 keys only b=4096")
    keys = workloads.uniform(0x5EED00A2, n, 8)
    ok, _ = oracle.radsort(keys, None, 256, 8, 4096)
    dk = to_dev(keys)
    radsort.sort_(dk, None, block_elems=4096, check=True)
    assert np.array_equal(from_dev(dk, 8).astype(np.uint64), ok)


@pytest.mark.parametrize("dist", ["zipf", "equal", "sorted", "low20"])
def test_structured_u64_2e30(dist):
    """n = 2^30 uint64 keys + uint32 index, 8-bit digits (8 rounds), b = 1024.  The
    oracle does not run at this size; the output is checked by the properties
    that fix a stable sort's result: keys ascending (unsigned), indices
    ascending within equal keys, the indices a permutation, and every key equal
    to the input key at its index."""
    n = 1 << 30
    say(f"2^30 uint64 {dist}")
    keys = workloads.make_t(dist, workloads.SEED_SKEWED, n, 8, DEV)
    orig = keys.clone()
    vals = torch.arange(n, dtype=torch.int32, device=DEV)
    radsort.sort_(keys, vals, block_elems=1024, check=True)
    flip = keys ^ (-(1 << 63))  # unsigned order as signed order
    assert bool((flip[1:] >= flip[:-1]).all())
    del flip
    eq = keys[1:] == keys[:-1]
    assert bool((vals[1:][eq] > vals[:-1][eq]).all())
    del eq
    assert bool(((vals >= 0) & (vals < n)).all())  # before indexing with them
    seen = torch.zeros(n, dtype=torch.bool, device=DEV)
    seen[vals.long()] = True
    assert bool(seen.all())
    del seen
    assert bool((orig[vals.long()] == keys).all())


@pytest.mark.parametrize("kb", [4, 8])
def test_shared_launch_forms_at_scale(kb):
    """RADSORT_F_SHARED (one workgroup per tile, claimed in order; dynamic
    compaction) on 2^26 elements, for Radsort and the baseline, against the oracle."""
    n = 1 << 26
    say(f"shared 2^26 kb={kb}")
    keys = workloads.uniform(0x5EED0006 + kb, n, kb)
    vals = np.arange(n, dtype=np.uint32)
    ok, ov = oracle.radsort(keys, vals, 256, kb, 1024)
    for fn in (radsort.sort_, radsort.oop_sort_):
        dk, dv = to_dev(keys), to_dev(vals)
        fn(dk, dv, check=True, shared=True)
        assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ok), fn.__name__
        assert np.array_equal(from_dev(dv, 4).astype(np.uint64), ov), fn.__name__


# ---------------------------------------------------------------- the round's tiles

# The large tile of the default draw order (from 2^22 records of at most 8 bytes with
# 4-byte keys, 2^20 of the others) at the edges of its range: one element below, at and
# above the threshold, a whole number of tiles, a ragged last tile, blocks of exactly 1024
# elements, of one tile and larger than a tile, narrow digits, and digits spread or
# skewed within a wave (ranks by OR table or by ballots).
TILE_EDGE = [
    ("uniform", (1 << 22) - 1, 4, 4, 8, 1024),
    ("uniform", (1 << 22) + 1, 4, 4, 8, 1024),
    ("zipf", 1 << 22, 4, 4, 8, 2048),
    ("uniform", (1 << 22) + 16383, 4, 0, 8, 16384),
    ("few", (1 << 22) + 5, 4, 4, 8, 65536),
    ("low20", (1 << 22) + 4097, 4, 4, 4, 1024),
    ("uniform", (1 << 20) - 1, 8, 0, 8, 1024),
    ("zipf", (1 << 20) + 8191, 8, 0, 8, 8192),
    ("uniform", (1 << 20) + 1, 8, 4, 8, 1024),
    ("sorted", (1 << 20) + 77, 8, 8, 8, 2048),
    ("equal", (1 << 20) + 1023, 4, 8, 8, 1024),
    ("zipf", (1 << 20) + 8193, 4, 8, 5, 65536),
]


@pytest.mark.parametrize("case", TILE_EDGE, ids=lambda c: "-".join(map(str, c)))
def test_tile_edges_match_oracle(case):
    """Every round's P, f and logical contents, and the finalized arrays, both through
    the step interface; then the one-call sort of the same input."""
    dist, n, kb, vb, bits, b = case
    say(f"tile edges {case}")
    keys, vals = inputs(dist, n, kb, vb, seed=7)
    sigma, nt = oracle.digit_params(kb, bits)
    dk, dv = to_dev(keys), to_dev(vals) if vb else None
    st = radsort.State(dk, dv, digit_bits=bits, block_elems=b)
    R = oracle.Radsort(keys, vals, sigma, nt, b)
    st.setup()
    R.setup()
    for r in range(min(nt, 3)):
        st.round()
        R.round(nt - 1 - r)
        _, pidx, plen, f = st.read()
        oidx, olen = R.P()
        assert f == R.f
        assert np.array_equal(pidx.astype(np.uint64), oidx)
        assert np.array_equal(plen.astype(np.uint64), olen)
        lk, lv = st.logical()
        ok, ov, _ = R.logical()
        assert np.array_equal(from_dev(lk, kb).astype(np.uint64), ok), f"round {r}"
        if vb:
            assert np.array_equal(from_dev(lv, vb).astype(np.uint64), ov), f"round {r}"
    for _ in range(nt - min(nt, 3)):
        st.round()
    st.finalize()
    st.read()
    ek, ev = oracle.radsort(keys, vals, sigma, nt, b)
    sk, sv = to_dev(keys), to_dev(vals) if vb else None
    radsort.sort_(sk, sv, digit_bits=bits, block_elems=b, check=True)
    for gk, gv in ((dk, dv), (sk, sv)):
        assert np.array_equal(from_dev(gk, kb).astype(np.uint64), ek)
        if vb:
            assert np.array_equal(from_dev(gv, vb).astype(np.uint64), ev)
    st.close()


# ---------------------------------------------------------------- rounds left out

# Keys whose digits vary at some positions only (vary: the mask of the bits that do): the
# one-call sort leaves out the rounds of the others and packs the last one that runs,
# wherever it is; no bit varies at all; one element differs from all the others.
VARY = [
    (0x000000FF, 50001, 4, 4, 8, 1024),
    (0x0000FF00, (1 << 22) + 3, 4, 4, 8, 2048),
    (0xFF0000FF, 300000, 4, 0, 8, 1024),
    (0x00FF0000, 70001, 4, 8, 4, 1024),
    (0x0, 40000, 4, 4, 8, 1024),
    (0x80000000, 123457, 4, 4, 6, 1024),
    (0xFF << 56, (1 << 20) + 9, 8, 4, 8, 1024),
    (0xF << 28 | 1, 90000, 8, 0, 8, 4096),
    (0x0, (1 << 20) + 1, 8, 8, 8, 1024),
    (0xFFFF << 20, 200003, 8, 4, 5, 1024),
]


@pytest.mark.parametrize("shared", [False, True], ids=["alone", "shared"])
@pytest.mark.parametrize("case", VARY, ids=lambda c: "-".join(map(str, c)))
def test_constant_digits_match_oracle(case, shared):
    mask, n, kb, vb, bits, b = case
    say(f"constant digits {case} shared={shared}")
    keys, vals = inputs("uniform", n, kb, vb, seed=9)
    fixed = keys.dtype.type(0x5A5A5A5AA5A5A5A5 & ((1 << 8 * kb) - 1))
    keys = (keys & keys.dtype.type(mask)) | (fixed & keys.dtype.type(~mask & ((1 << 8 * kb) - 1)))
    if mask == 0 and kb == 8:
        keys[n // 3] ^= np.uint64(1 << 40)
    sigma, nt = oracle.digit_params(kb, bits)
    dk, dv = to_dev(keys), to_dev(vals) if vb else None
    radsort.sort_(dk, dv, digit_bits=bits, block_elems=b, check=True, shared=shared)
    ek, ev = oracle.radsort(keys, vals, sigma, nt, b)
    assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ek)
    if vb:
        assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ev)


# ------------------------------------------------ look-back over all tiles of a round

# One-call sorts whose look-back words fit one per (tile, digit), at the last such size
# and past it, and those of a ring whose slots are used again (over 1024 tiles of 8192 or
# 16384 slots at 8-bit digits; few digits make many slots).
CHAIN = [
    ("uniform", (1 << 24) + 16385, 8, 0, 8, 1024),
    ("few", (1 << 24) + (1 << 22), 8, 4, 8, 4096),
    ("zipf", (1 << 25) + 77, 4, 4, 8, 1024),
    ("zipf", (1 << 25) + (1 << 24) - 1, 4, 0, 8, 32768),
    ("uniform", (1 << 25) + 5, 8, 8, 7, 2048),
    ("low20", (1 << 25) + 8191, 4, 8, 3, 1024),
]


@pytest.mark.parametrize("case", CHAIN, ids=lambda c: "-".join(map(str, c)))
def test_long_lookback_matches_stable_sort(case):
    """The order of a stable sort, exactly: payloads are positions."""
    dist, n, kb, vb, bits, b = case
    say(f"long look-back {case}")
    keys, _ = inputs(dist, n, kb, vb, seed=13)
    dk = to_dev(keys)
    dv = torch.arange(n, device="cuda").to(torch.int32 if vb == 4 else torch.int64) if vb else None
    want = dk.to(torch.int64)
    want = want & 0xFFFFFFFF if kb == 4 else want ^ -(1 << 63)
    order = torch.sort(want, stable=True)[1]
    ek = dk[order]
    radsort.sort_(dk, dv, digit_bits=bits, block_elems=b, check=True)
    assert torch.equal(dk, ek)
    if vb:
        assert torch.equal(dv.to(torch.int64), order)


# ---------------------------------------------------------------- arrays sorted on chip

SMALL_N = [2, 63, 256, 511, 512, 513, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193]


@pytest.mark.parametrize("kb,vb", [(4, 0), (4, 4), (4, 8), (8, 0), (8, 4), (8, 8)])
@pytest.mark.parametrize("dist", ["uniform", "zipf", "low20", "equal"])
def test_small_arrays_match_oracle(kb, vb, dist):
    """One-call sorts around the sizes where the on-chip shapes begin and end, through
    every entry point that takes them, and the same arrays as one batch."""
    say(f"small arrays kb={kb} vb={vb} {dist}")
    ks, vs, eks, evs = [], [], [], []
    for n in SMALL_N:
        keys, vals = inputs(dist, n, kb, vb, seed=11)
        ek, ev = oracle.radsort(keys, vals, 256, kb, 1024)
        ws = torch.empty(radsort.workspace_bytes(n, kb, vb), dtype=torch.uint8, device=DEV)
        ws.fill_(0xA5)
        for entry in ("sort", "workspace", "oop", "noalloc"):
            dk, dv = to_dev(keys), to_dev(vals) if vb else None
            if entry == "sort":
                radsort.sort_(dk, dv, check=True)
            elif entry == "workspace":
                radsort.sort_(dk, dv, workspace=ws)
                assert radsort.workspace_error(dk, dv, workspace=ws) == 0
            elif entry == "oop":
                radsort.oop_sort_(dk, dv)
            else:
                radsort.sort_noalloc_(dk, dv, check=True)
            assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ek), (entry, n)
            if vb:
                assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ev), (entry, n)
        ks.append(keys)
        eks.append(ek)
        if vb:
            vs.append(vals)
            evs.append(ev)
    offsets = np.concatenate([[0], np.cumsum(SMALL_N)]).astype(np.uint64)
    dk, dv = to_dev(np.concatenate(ks)), to_dev(np.concatenate(vs)) if vb else None
    radsort.sort_segments_(dk, dv, offsets, tuning=None, check=True)
    assert np.array_equal(from_dev(dk, kb).astype(np.uint64), np.concatenate(eks))
    if vb:
        assert np.array_equal(from_dev(dv, vb).astype(np.uint64), np.concatenate(evs))


# ---------------------------------------------------------------- out of place in the workspace

# One-call sorts whose records fit their own workspace once more, at the edges of the tile
# shapes and of the range (3 * 256 blocks of b records, less the tables), and the same
# inputs through the out-of-place entry point.
IN_WS = [
    ("uniform", 8193, 4, 4, 1024),
    ("zipf", 2048 * 5, 4, 0, 1024),
    ("low20", (1 << 16) + 1, 8, 4, 1024),
    ("uniform", (1 << 18) - 1, 4, 8, 1024),
    ("uniform", (1 << 18) + 1, 4, 4, 1024),
    ("equal", 300000, 8, 8, 1024),
    ("sorted", 700001, 4, 4, 1024),
    ("uniform", 768 * 1024 + 5, 4, 4, 1024),
    ("uniform", 1 << 20, 8, 0, 2048),
    ("few", (1 << 22) + 3, 4, 4, 8192),
]


@pytest.mark.parametrize("shared", [False, True], ids=["alone", "shared"])
@pytest.mark.parametrize("case", IN_WS, ids=lambda c: "-".join(map(str, c)))
def test_sorts_in_workspace_match_oracle(case, shared):
    dist, n, kb, vb, b = case
    say(f"in workspace {case} shared={shared}")
    keys, vals = inputs(dist, n, kb, vb, seed=13)
    ek, ev = oracle.radsort(keys, vals, 256, kb, 1024)
    size = radsort.workspace_bytes(n, kb, vb, 8, b, shared=shared)
    buf = torch.empty(size + 512, dtype=torch.uint8, device=DEV)
    buf.fill_(0x5A)
    for oop in (False, True):
        dk, dv = to_dev(keys), to_dev(vals) if vb else None
        if oop:
            radsort.oop_sort_(dk, dv, block_elems=b, check=True, shared=shared)
        else:
            radsort.sort_(dk, dv, block_elems=b, workspace=buf[:size], shared=shared)
            assert radsort.workspace_error(dk, dv, block_elems=b, workspace=buf[:size]) == 0
            assert bool((buf[size:] == 0x5A).all())  # nothing past the workspace is written
        assert np.array_equal(from_dev(dk, kb).astype(np.uint64), ek)
        if vb:
            assert np.array_equal(from_dev(dv, vb).astype(np.uint64), ev)
