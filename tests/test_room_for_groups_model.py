"""The argument behind the stream phase's room for groups, as a host model checked against brute force.

A wave comes by the 16-byte groups of its share of a row in the order of their coordinates and sets aside those that may
hold one of the row's k best sums.  When a column of 64 groups finds no room, it makes some: the k-th greatest of
the groups' greatest sums is a bar (k different elements of the row reach it), groups below it go, of those that only
tie at it the first ones stay, up to k groups in all, and once there are k, later groups have to be better than the bar.
At the end of the row what is left is looked at element by element.  This file restates that on plain Python lists,
for several waves with the floor they share, and checks that no key of a row's k best is ever lost - ties go to
the lower coordinate - and that room is always found, on sums full of ties, in every order.  No GPU, no library
call: it pins the reasoning, the GPU tests pin the code.
"""
import random

import pytest

LANES = 64


class Wave:
    def __init__(self, k, room, floor, blocked):
        self.k, self.room, self.bar, self.strict, self.blocked = k, room, floor, False, blocked
        self.groups = []                                   # (coordinate of the first element, sums), in order

    def best(self, group):
        at, sums = group
        return max((s for c, s in enumerate(sums) if at + c != self.blocked), default=float("-inf"))

    def passes(self, group):
        """The quick test: the blocked entry takes part in it, so it may say yes too often."""
        top = max(group[1])
        return top > self.bar if self.strict else top >= self.bar

    def make_room(self):
        images = sorted((self.best(g) for g in self.groups), reverse=True)
        if len(images) >= self.k:
            self.bar = max(self.bar, images[self.k - 1])
        left = self.k - sum(1 for i in images if i > self.bar)
        self.strict = sum(1 for i in images if i == self.bar) >= left
        kept, ties = [], 0
        for g in self.groups:
            b = self.best(g)
            if b > self.bar or (b == self.bar and ties < left):
                kept.append(g)
            ties += b == self.bar
        self.groups = kept

    def column(self, column):
        """64 groups side by side: all that pass are set aside, or none and room is made."""
        while True:
            mine = [g for g in column if self.passes(g)]
            if len(self.groups) + len(mine) <= self.room:
                self.groups += mine
                return
            before = len(self.groups)
            self.make_room()
            assert len(self.groups) <= self.k and len(self.groups) < before   # room is found, at once

    def keys(self):
        return [(s, -(at + c)) for at, sums in self.groups for c, s in enumerate(sums)
                if at + c != self.blocked and s >= self.bar]


def best_by_model(sums, k, waves, per_group, room, blocked, floor):
    groups = [(i, sums[i:i + per_group]) for i in range(0, len(sums), per_group)]
    columns = [groups[i:i + LANES] for i in range(0, len(groups), LANES)]
    keys = []
    for w in range(waves):
        wave = Wave(k, room, floor, blocked)
        for i in range(w, len(columns), waves):
            wave.column(columns[i])
        if len(wave.groups) > k:
            wave.make_room()                               # what the end of a row does before keys overflow
        keys += wave.keys()
    return sorted(keys, reverse=True)[:k]


def rows(rng, n, kind):
    if kind == "equal":
        return [1.0] * n
    levels = {"two": 2, "few": 7, "many": 10 ** 6}.get(kind, 40)
    out = [float(rng.randint(1, levels)) for _ in range(n)]
    if kind == "rising":
        out.sort()
    elif kind == "falling":
        out.sort(reverse=True)
    elif kind == "plateau":
        out[n // 4:n // 2] = [50.0] * (n // 2 - n // 4)
    elif kind == "stairs":
        out = [float(i * 8 // n) for i in range(n)]
    return [float("-inf") if rng.random() < 0.02 else s for s in out]


@pytest.mark.parametrize("kind", ["equal", "two", "few", "many", "rising", "falling", "plateau", "stairs"])
@pytest.mark.parametrize("k", [1, 5, 20, 63, 64])
def test_no_key_of_the_k_best_is_lost(kind, k):
    rng = random.Random(1000 * k + len(kind))
    for trial in range(12):
        per_group, waves = rng.choice([4, 8]), rng.choice([1, 4, 8])
        n = per_group * LANES * rng.randint(1, 24) - rng.randint(0, per_group * LANES - 1)
        sums = rows(rng, n, kind)
        blocked = rng.choice([-1, rng.randrange(n), max(range(n), key=lambda c: sums[c])])
        keys = sorted(((s, -c) for c, s in enumerate(sums) if c != blocked and s > float("-inf")), reverse=True)
        # a valid floor is any sum that k elements reach; the lowest finite one stands for no floor at all
        floor = keys[k - 1][0] if len(keys) >= k and rng.random() < 0.3 else -1.0
        got = best_by_model(sums, k, waves, per_group, 128, blocked, floor)
        assert got == keys[:k], (kind, k, trial, per_group, waves, n, blocked, floor)


def test_a_strict_bar_without_the_order_of_coordinates_would_lose_a_key():
    """The one step that rests on the order: were a wave to come by its groups backwards, a later tie would have
    the lower coordinate and the strict bar would pass over it."""
    k, per_group = 5, 4
    sums = [1.0] * (per_group * LANES * 4)
    groups = [(i, sums[i:i + per_group]) for i in range(0, len(sums), per_group)]
    wave = Wave(k, 128, -1.0, -1)
    for i in range(len(groups) - LANES, -1, -LANES):
        wave.column(groups[i:i + LANES])
    assert sorted(wave.keys(), reverse=True)[:k] != [(1.0, -c) for c in range(k)]
    assert best_by_model(sums, k, 1, per_group, 128, -1, -1.0) == [(1.0, -c) for c in range(k)]
