"""A model of the look-back over all tiles of a round, the form of the one-call sorts
(kernel_tile.hpp: kChainRows and kChainRing), run under random schedules on the CPU.

Per tile, in the kernel's order: load its blocks; with the ring, wait until the tiles that
the reuse of its slot depends on are done; publish its count of every digit; per digit look
back over the earlier tiles, some at a time, to the nearest inclusive count, and publish its
own; once every digit has finished, its done word (ring only), its draws; the blocks that
earlier tiles drew and this one continues; its writes.  There are no done words in front of
the draws: a finished look-back has seen a word of every earlier tile.

Every read and write of a word is a step of its own, so that the words of one look-back step
are read at different times; at most `resident` tiles run at once, taken in order, and some
of them lag behind.  Checked: the counts that each look-back finds, that no block is written
before the tile that holds its old contents has loaded it, and that every tile ends.
"""
import random

import pytest

AGG, INCL = 1, 2


def plan(digits, sigma, b, E, offsets):
    """Per tile: its counts, the counts before it, its draws {(d, q): k} and the blocks
    (d, q) it writes.  Bucket d starts at offset offsets[d] of its first block."""
    base, F, out = [0] * sigma, 0, []
    for ds in digits:
        cnt, draws = [0] * sigma, {}
        for d in ds:
            r = offsets[d] + base[d] + cnt[d]
            cnt[d] += 1
            if (r + 1) % b == 0:
                draws[(d, (r + 1) // b)] = None
        for i, blk in enumerate(sorted(draws)):  # in (digit, block) order
            draws[blk] = F + i
        writes = {(d, q) for d in range(sigma) if cnt[d]
                  for q in range((offsets[d] + base[d]) // b,
                                 (offsets[d] + base[d] + cnt[d] - 1) // b + 1)}
        out.append((cnt, list(base), draws, writes))
        F += len(draws)
        base = [x + y for x, y in zip(base, cnt)]
        assert F == sum((o + x) // b for o, x in zip(offsets, base))
    return out


class Round:
    """One round.  W: the ring's slots, or None for a word per tile.  reuse: how many tiles
    from t - W on must be done before tile t takes its slot (the kernel: 2).  packed: the
    first sigma draws take extra blocks and the buckets start at offsets.  early: counts
    published before the loads have returned (a mutant)."""

    def __init__(self, seed, n_t, sigma, b, E, W, lbw, reuse=2, packed=False, early=False):
        rng = random.Random(seed)
        self.rng, self.n_t, self.sigma, self.W, self.lbw = rng, n_t, sigma, W, lbw
        self.reuse, self.early = reuse, early
        hot = rng.random() < 0.3  # skewed digits
        digits = [[0 if hot and rng.random() < 0.7 else rng.randrange(sigma) for _ in range(E)]
                  for _ in range(n_t)]
        offsets = [rng.randrange(b) if packed else 0 for _ in range(sigma)]
        self.plan = plan(digits, sigma, b, E, offsets)
        # the tile that holds the old contents of draw k (None: an extra block)
        self.reader = lambda k: (k if not packed else k - sigma) * b // E if \
            not packed or k >= sigma else None
        self.drawer = {blk: (t, k) for t, p in enumerate(self.plan) for blk, k in p[2].items()}
        slots = n_t if W is None else W
        self.words = [[(0, 0, 0)] * sigma for _ in range(slots)]  # status, tile + 1, value
        self.done, self.loaded, self.drawn = [0] * (2 * W if W else 1), set(), set()
        self.version = 0
        self.wrong, self.unread = [], []

    def slot(self, t):
        return t if self.W is None else t % self.W

    def write(self, t, d, status, value):
        self.words[self.slot(t)][d] = (status, t + 1, value)
        self.version += 1

    def is_done(self, t):
        return self.done[t % len(self.done)] > t

    def look_back(self, t, d):
        """Yields None (a step) or a predicate to wait for."""
        k, acc, stalled, start = t, 0, False, self.version
        while k > 0:
            m = 1 if stalled else min(self.lbw, k)
            seen, w = self.version, [None] * m
            for i in self.rng.sample(range(m), m):
                w[i] = self.words[self.slot(k - 1 - i)][d]
                yield None
            used, found, again, ready = 0, False, False, True
            for i in range(m):
                status, tag, value = w[i]
                ready = status != 0 and tag == k - i
                if not ready:
                    again = tag > k - i
                    break
                acc += value
                used = i + 1
                if status == INCL:
                    found = True
                    break
            k -= used
            if found:
                break
            stalled = not ready and used == 0 and not again
            if again:  # the same words would give the same again
                yield lambda: self.version != start
                k, acc, start = t, 0, self.version
            elif not ready:
                yield lambda: self.version != seen
        cnt, base = self.plan[t][0], self.plan[t][1]
        if acc != base[d]:
            self.wrong.append((t, d, acc, base[d]))
        yield None
        if t:
            self.write(t, d, INCL, base[d] + cnt[d])

    def tile(self, t):
        cnt, _, draws, writes = self.plan[t]
        yield None
        if not self.early:
            self.loaded.add(t)
        if self.W and t >= self.W:
            for j in range(t - self.W, t - self.W + self.reuse):
                yield lambda j=j: self.is_done(j)
        for d in self.rng.sample(range(self.sigma), self.sigma):
            self.write(t, d, AGG if t else INCL, cnt[d])
            yield None
        threads = [[self.look_back(t, d), None] for d in range(self.sigma)]
        while threads:  # the digits' threads, interleaved
            run = [x for x in threads if x[1] is None or x[1]()]
            if not run:
                yield lambda: any(x[1]() for x in threads)
                continue
            x = self.rng.choice(run)
            try:
                x[1] = next(x[0])
            except StopIteration:
                threads.remove(x)
            yield None
        if self.W:
            self.done[t % len(self.done)] = t + 1
            self.version += 1
            yield None
        self.drawn |= set(draws)
        self.loaded.add(t)
        yield None
        for blk in writes:
            if blk in self.drawer and self.drawer[blk][0] != t:
                yield lambda blk=blk: blk in self.drawn
        for blk in writes:
            if blk in self.drawer:
                r = self.reader(self.drawer[blk][1])
                if r is not None and r not in self.loaded:
                    self.unread.append((t, blk, r))

    def run(self, resident, slow=0.2):
        """False if some tile cannot go on."""
        tiles, nxt = {}, 0
        while True:
            while len(tiles) < resident and nxt < self.n_t:
                tiles[nxt] = [self.tile(nxt), None, self.rng.random() < slow]
                nxt += 1
            if not tiles:
                return True
            run = [t for t, x in tiles.items() if x[1] is None or x[1]()]
            if not run:
                return False
            fast = [t for t in run if not tiles[t][2]]
            t = self.rng.choice(fast or run)
            try:
                tiles[t][1] = next(tiles[t][0])
            except StopIteration:
                del tiles[t]


GEO = dict(n_t=40, sigma=4, b=32, E=16)
FORMS = [dict(W=None, lbw=8), dict(W=16, lbw=1), dict(W=16, lbw=2), dict(W=4, lbw=1),
         dict(W=8, lbw=4), dict(W=2, lbw=1)]


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("form", FORMS, ids=lambda f: f"W{f['W']}-step{f['lbw']}")
def test_counts_and_draws_under_any_schedule(form, packed):
    for seed in range(30):
        r = Round(seed, packed=packed, **GEO, **form)
        assert r.run(resident=3 + seed % 24), (seed, "a tile cannot go on")
        assert r.wrong == [] and r.unread == [], seed


def outcome(**kw):
    """How many of the schedules end wrong: (cannot go on, wrong counts, unread blocks)."""
    stuck = wrong = unread = 0
    for seed in range(40):
        r = Round(seed, **{**GEO, **kw})
        stuck += not r.run(resident=3 + seed % 24)
        wrong += bool(r.wrong)
        unread += bool(r.unread)
    return stuck, wrong, unread


def test_slot_reuse_must_wait_for_the_next_tile_too():
    """A slot taken over once its tile is done: the tile after it may still need the word."""
    stuck, wrong, _ = outcome(W=4, lbw=1, reuse=1)
    assert stuck + wrong > 0


def test_slot_reuse_must_wait():
    stuck, wrong, _ = outcome(W=4, lbw=1, reuse=0)
    assert stuck + wrong > 0


@pytest.mark.parametrize("form", FORMS[:2], ids=["words", "ring"])
def test_counts_must_follow_the_loads(form):
    """The draws wait for nothing but the look-back: a count in front of its tile's loads
    lets a later tile write into a block that is still to be read."""
    assert outcome(early=True, **form)[2] > 0
