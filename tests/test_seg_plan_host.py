"""Grouped arrays of a batch when the host's and the device's offsets disagree (CPU model).

The host plans a batch's groups, tables and launches from its copy of the offsets
(plan_groups in radsort.hip); the kernels (kernel_seg.hpp) take sizes and places from the
device's copy.  The two must hold the same values; where they do not, the kernels may only
report it.  The steps below restate the plan of both sides and every index that the kernels
use, on tables that hold stale words where nothing was written.  With the kernels' checks no
index leaves its table and no array is sorted in a scratch that is not its own; without
them the same model finds indices that do.
"""
import random

import pytest

E, RECORD, NT = 8192, 8, 4  # uint32 pairs, shape 1
LO, TOP = 8192, 4320 * 1024


def tables_bytes(arrays, tiles, all_arrays, all_tiles):
    up = lambda x: (x + 255) // 256 * 256
    return (up(arrays * NT * 1024) + up(arrays * 4) + up(tiles * 1024) + up(4 * NT)
            + up(arrays * 4) + up(all_tiles * 4) + up(all_arrays * 32))


def host_plan(sizes, avail):
    """plan_groups: (groups [(a0, na, t0, t1, id)], arrays, tiles, G64, hi, D64, amax, tmax)."""
    D64 = avail // (64 * RECORD)
    while D64 >= 128:
        take = [n for n in sizes if LO < n <= TOP and (n + 63) // 64 <= D64 // 2]
        if not take:
            return None
        G64 = D64 - max((n + 63) // 64 for n in take)
        groups, pos, arrays, tiles = [], 0, 0, 0
        for n in take:
            if not groups or pos // G64 != groups[-1][4]:
                groups.append([arrays, 0, tiles, tiles, pos // G64])
            arrays += 1
            tiles += -(-n // E)
            pos += (n + 63) // 64
            groups[-1][1] += 1
            groups[-1][3] = tiles
        amax, tmax = max(g[1] for g in groups), max(g[3] - g[2] for g in groups)
        total = tables_bytes(amax, tmax, arrays, tiles)
        if (total + D64 * 64 * 4 + 255) // 256 * 256 + D64 * 64 * 4 <= avail:
            return groups, arrays, tiles, G64, min(D64 // 2 * 64, TOP), D64, amax, tmax
        D64 -= D64 // 16 + 1
    return None


class OutOfRange(Exception):
    pass


def at(table, i):
    if not 0 <= i < len(table):
        raise OutOfRange(i)
    return table[i]


def device_run(plan, sizes, checked, rng):
    """Runs the kernels' index arithmetic on the device's sizes; returns (error reported,
    arrays whose rounds ran)."""
    groups, count, tiles, G64, hi, D64, amax, tmax = plan
    stale = lambda: rng.randrange(1 << 32)
    arr = [(stale(), stale(), stale(), stale()) for _ in range(count)]  # n, place, tile0, group
    map_ = [stale() for _ in range(tiles)]
    idx = pos = tile = 0
    for n in sizes:  # k_seg_plan
        if not LO < n <= hi:
            continue
        if idx < count:
            arr[idx] = (n, pos % G64, tile, pos // G64)
        idx += 1
        pos += (n + 63) // 64
        tile += -(-n // E)
    if checked and (idx != count or tile != tiles):
        arr = [(0, 0, 0, 0)] * count
        map_ = [0xFFFFFFFF] * tiles
    for i, (n, _, tile0, _) in enumerate(arr):  # k_seg_map
        for t in range(min(-(-n // E), 1 << 20)):
            if (tile0 + t) & 0xFFFFFFFF < tiles:
                map_[(tile0 + t) & 0xFFFFFFFF] = i
    error, ran = False, []
    rounds = {}
    for a0, na, t0, t1, gid in groups:
        hist, state = [0] * amax, [0] * tmax
        rounds = {k: 0 for k in range(amax)} if checked else rounds
        arrived = [0] * amax
        for t in range(t0, t1):  # k_seg_hist
            ai = at(map_, t)
            if checked and not 0 <= ai - a0 < na:
                error = True
                map_[t] = a0
                continue
            n, place, tile0, group = at(arr, ai)
            ti, ntiles = (t - tile0) & 0xFFFFFFFF, -(-n // E)
            if ti >= ntiles or (checked and group != gid):
                error = True
                map_[t] = a0 if checked else ai
                continue
            at(hist, ai - a0)
            arrived[ai - a0] += 1
            if arrived[ai - a0] == ntiles:
                rounds[ai - a0] = 1
        owner = {}
        for t in range(t0, t1):  # k_seg_round
            ai = at(map_, t)
            n, place, tile0, group = at(arr, ai)
            at(hist, ai - a0)  # rounds has as many entries
            if not rounds.get(ai - a0, stale() & 1):
                continue
            ti = (t - tile0) & 0xFFFFFFFF
            if ti * E >= n:
                error = True
                continue
            for earlier in range(max(0, ti - 3), ti):  # look-back
                at(state, t - t0 - (ti - earlier))
            if place * 64 + n > D64 * 64:
                raise OutOfRange(place)
            for x in (place, place + (n - 1) // 64):  # the scratch is the array's own
                if owner.setdefault(x, ai) != ai:
                    raise OutOfRange(x)
            ran.append((gid, ai))
    return error, set(ran)


def cases(seed):
    rng = random.Random(seed)
    sizes = [rng.choice([8193, 9000, 70001, 150000, 200001]) for _ in range(60)]
    yield "same", sizes, sizes
    fewer = list(sizes)
    fewer[7], fewer[8] = fewer[7] + fewer[8], 0
    yield "fewer", sizes, fewer
    more = list(sizes)
    more[11:12] = [9001, 30000]
    yield "more", sizes, more
    yield "none", sizes, [0] * 60
    yield "reversed", sorted(sizes), sorted(sizes, reverse=True)
    yield "larger", sizes, [n + 40000 for n in sizes]


@pytest.mark.parametrize("seed", range(4))
def test_no_index_leaves_its_table(seed):
    rng = random.Random(100 + seed)
    for name, host, dev in cases(seed):
        plan = host_plan(host, 60 * 65536 * RECORD)
        assert len(plan[0]) > 1
        error, ran = device_run(plan, dev, True, rng)
        assert error == (name != "same"), name
        if name == "same":
            assert len(ran) == len(host)


def test_without_the_checks_indices_leave_their_tables():
    found = set()
    for seed in range(4):
        rng = random.Random(200 + seed)
        for name, host, dev in cases(seed):
            try:
                device_run(host_plan(host, 60 * 65536 * RECORD), dev, False, rng)
            except OutOfRange:
                found.add(name)
    assert "same" not in found and {"fewer", "none", "reversed"} <= found
