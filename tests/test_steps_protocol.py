"""CPU model of how the blocks of a launch of several steps (k_steps) keep
apart: they count themselves in, together each keeps its chunk, and where they
do not all meet those that run take the chunk-steps from a counter.  Blocks
are generators that give way at every access to what they share and are
resumed in random order, a limited number at a time, later ones as earlier
ones leave.  Every gather must find its source's state of that step (the two
buffers take turns, so a write too early shows as well as a read too early),
every launch must end, and the words must be back in place for the next."""
import random

import pytest

CLOSED = 1 << 31


class Launch:
    def __init__(self, rng, chunks, reach, states, words, before, steps, patience):
        self.rng, self.G, self.steps, self.before, self.patience = rng, chunks, steps, before, patience
        self.near = [[(c + d) % chunks for d in range(-reach, reach + 1) if (c + d) % chunks != c] for c in
                     range(chunks)]
        self.state, self.w = states, words          # state[buffer][chunk]: the step it is the result of
        self.sums = set()
        self.finished = 0

    def step(self, c, t):
        src, dst = self.state[t & 1], self.state[1 - (t & 1)]
        for q in [c] + self.near[c]:
            yield
            assert src[q] == self.first + t, (c, t, q)
        yield
        dst[c] = self.first + t + 1
        yield
        self.w["done"][c] = self.before + t + 1
        yield
        assert (t, c) not in self.sums
        self.sums.add((t, c))

    def wait(self, chunks, target):
        for q in chunks:
            while self.w["done"][q] < target:
                yield
            yield

    def block(self, b):
        w, G = self.w, self.G
        w["count"] += 1
        v, polls = w["count"], 0
        yield
        while not v & CLOSED and v < G:
            polls += 1
            if polls > self.patience and w["count"] == v:      # compare and exchange
                w["count"] = v = v | CLOSED
                break
            v = w["count"]
            yield
        together = not v & CLOSED
        if together:
            for t in range(self.steps):
                yield from self.step(b, t)
                if t + 1 < self.steps:
                    yield from self.wait(self.near[b], self.before + t + 1)
            w["done"][b] = self.before + self.steps + 1
            yield
            yield from self.wait(range(G), self.before + self.steps + 1)
        else:
            while True:
                q = w["next"]
                w["next"] += 1
                yield
                t, c = divmod(q, G)
                if t >= self.steps:
                    break
                yield from self.wait(self.near[c] + [c], self.before + t)
                yield from self.step(c, t)
            w["left"] += 1
            last = w["left"] == G
            yield
            if not last:
                return
            w["done"] = [self.before + self.steps + 1] * G
            w["left"] = w["next"] = 0
        if b == 0 or not together:
            assert len(self.sums) == self.steps * G            # all sums are there to be reduced
            w["count"] = 0
            self.finished += 1

    def run(self, first, room):
        self.first = first
        waiting = list(range(self.G))
        running = []
        budget = 4000 * self.G * self.steps
        while waiting or running:
            while waiting and len(running) < room:
                running.append(self.block(waiting.pop(0)))
            g = self.rng.choice(running)
            try:
                next(g)
            except StopIteration:
                running.remove(g)
            budget -= 1
            assert budget > 0, "the launch does not end"
        assert self.finished == 1


@pytest.mark.parametrize("chunks,reach,room", [(1, 1, 1), (2, 1, 2), (2, 1, 1), (5, 1, 5), (5, 2, 3), (9, 2, 4),
                                               (12, 3, 12), (12, 3, 11), (12, 1, 2)])
@pytest.mark.parametrize("seed", range(4))
def test_steps_of_a_launch_keep_apart(chunks, reach, room, seed):
    rng = random.Random(100 * seed + chunks)
    states = [[0] * chunks, [None] * chunks]
    words = dict(count=0, left=0, next=0, done=[0] * chunks)
    first = before = 0
    for steps in (4, 5, 3):
        a = Launch(rng, chunks, reach, states, words, before, steps, patience=rng.choice([0, 30, 10**6 if room >= chunks
                                                                                          else 200]))
        a.run(first, room)
        before += steps + 1
        first += steps
        if steps & 1:                  # the next launch starts from the other buffer
            states.reverse()
        assert states[0] == [first] * chunks
        assert words == dict(count=0, left=0, next=0, done=[before] * chunks)
