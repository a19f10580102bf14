"""Protocol of the sampler by local decisions (csrc/local_sampler.hip), and of what it has in common with the index-ordered
one (csrc/sampler.hip), on a model: the workgroups of a cloud as programs
that take turns in a random sequence of single reads and writes, with the words, stamps, parities and counters of the kernels.
A wait for a word that never comes leaves no program able to go on.  The faulty forms the model has been used
to find are kept as switches: the tests show that it still tells them from the present ones."""
import random

import pytest

WIPE = 15                   # rounds after which stamps start again, less one


class Stuck(Exception):
    pass


def run(programs, rng, slow):
    """Takes random programs one step further until all have ended.  A program yields a condition it waits for, or None;
    `slow` is picked rarely."""
    waiting = {g: next(p) for g, p in enumerate(programs)}
    while waiting:
        ready = [g for g, cond in waiting.items() if cond is None or cond()]
        if not ready:
            raise Stuck(sorted(waiting))
        fast = [g for g in ready if g != slow]
        g = rng.choice(fast) if fast and rng.random() < 0.995 else rng.choice(ready)
        try:
            waiting[g] = next(programs[g])
        except StopIteration:
            del waiting[g]


class Cloud:
    """What the workgroups of one group share in memory."""
    def __init__(self, G):
        self.G, self.word = G, {}

    def get(self, *key):
        return self.word.get(key, (0, None))


class Workgroup:
    def __init__(self, mem, g, seed):
        self.mem, self.g, self.seed = mem, g, seed
        self.cnt, self.round, self.seq = [0, 0], 0, 0

    def stamped(self, stamp, *key):
        return lambda: self.mem.get(*key)[0] == stamp

    def meet(self):                                     # plain_pick
        self.seq += 1
        self.mem.word["pk", self.seq & 1, self.g] = self.seq, None
        yield None
        for t in range(self.mem.G):
            yield self.stamped(self.seq, "pk", self.seq & 1, t)

    def renew(self):
        if self.mem.G == 1:
            return
        yield from self.meet()
        for key in list(self.mem.word):
            if key[0] in ("hdr", "list") and key[2] == self.g:
                del self.mem.word[key]
        yield None
        yield from self.meet()

    def agree(self):                                    # agree_in_order
        if self.mem.G == 1:
            return
        self.round += 1
        r, par = self.round, self.round & 1
        self.mem.word["hdr", par, self.g] = ("agree", r), None
        yield None
        for t in range(self.mem.G):
            yield self.stamped(("agree", r), "hdr", par, t)

    def follow(self, points, meet_first):
        """follow_order on a cloud that is in order to the end: the values of its points take the place of candidates."""
        G, word = self.mem.G, self.mem.word
        if not meet_first or G == 1 or self.round == 0:
            self.round += 1
        else:
            yield from self.agree()
        stamp = "value", self.round
        for k in range(points):
            if k % G == self.g:
                word["list", 0, 0, k] = stamp, None
                yield None
        for k in range(points):
            yield self.stamped(stamp, "list", 0, 0, k)
        yield from self.agree()
        yield from self.agree()                         # (all have read the values)

    def list_round(self, skip=False, decisions=True):
        """Scan, list and decisions of a round; checks every candidate read.  The workgroups from `deciding` on have no share
        of the list and publish no decisions; in the index-ordered sampler nobody does."""
        G, word = self.mem.G, self.mem.word
        if (self.round & WIPE) == WIPE:
            if skip:
                self.round += 1
            yield from self.renew()
        self.round += 1
        r, par, stamp = self.round, self.round & 1, ((self.round & WIPE) >> 1) + 1
        mine = lambda g: 1 + (7 * r + 3 * g + self.seed) % 3  # noqa: E731
        self.cnt[par] += mine(self.g)
        total = self.cnt[par]
        word["hdr", par, self.g] = stamp, total
        yield None
        self.cnt[par ^ 1] = 0
        for k in range(mine(self.g)):
            word["list", par, self.g, k] = stamp, (r, self.g, k)
            yield None
        if G == 1:
            assert total == mine(0), "the list of a round has candidates of an earlier one"
            return
        for t in range(G):
            yield self.stamped(stamp, "hdr", par, t)
            n = self.mem.get("hdr", par, t)[1]
            for k in range(n):
                yield self.stamped(stamp, "list", par, t, k)
                assert self.mem.get("list", par, t, k)[1] == (r, t, k)
        deciding = max(1, G // 2) if decisions else 0
        if self.g < deciding:
            word["mask", par, self.g] = r, None
            yield None
        for t in range(deciding):
            yield self.stamped(r, "mask", par, t)


def finish(G, seed, slow, skip=False, rounds=5 * WIPE):
    rng, mem = random.Random(seed), Cloud(G)

    def program(wg):
        for _ in range(rounds):
            yield from wg.list_round(skip)
    run([program(Workgroup(mem, g, seed)) for g in range(G)], rng, slow)


@pytest.mark.parametrize("G", [1, 2, 3, 5])
def test_stamps_start_again(G):
    for seed in range(12):
        finish(G, seed, seed % G)


@pytest.mark.parametrize("G", [1, 2, 3, 5])
def test_a_round_left_out_at_the_renewal_is_found(G):
    with pytest.raises(AssertionError if G == 1 else Stuck):
        finish(G, 0, 0, skip=True)


def clouds(G, seed, slow, decisions, meet_first=True):
    """Clouds of a group in turn: rounds, a cloud followed to its end, rounds, two followed."""
    rng, mem = random.Random(seed), Cloud(G)

    def program(wg):
        for kind in "RFRFFRRF":
            wg.cnt = [0, 0]
            if kind == "F":
                yield from wg.follow(1 + seed % 5, meet_first)
            else:
                for _ in range(1 + seed % 3):
                    yield from wg.list_round(decisions=decisions)
    run([program(Workgroup(mem, g, seed)) for g in range(G)], rng, slow)


@pytest.mark.parametrize("decisions", [True, False])
@pytest.mark.parametrize("G", [1, 2, 3, 5])
def test_followed_clouds_between_others(G, decisions):
    for seed in range(40):
        clouds(G, seed, seed % G, decisions)


@pytest.mark.parametrize("decisions", [True, False])
@pytest.mark.parametrize("G", [3, 5])
def test_values_written_over_a_list_still_read_are_found(G, decisions):
    stuck = 0
    for seed in range(40):
        try:
            clouds(G, seed, seed % G, decisions, meet_first=False)
        except (Stuck, AssertionError, TypeError):
            stuck += 1
    assert stuck > 0
