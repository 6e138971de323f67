"""The argument behind the merge phase's shortcut for the sentence's k best (Sec. 3.1 item 1), as a
host model checked against brute force.

The device code never sorts the sentence's k best keys.  It finds the k-th best score among the 32-bit score
images of the row lists and decides:
  * exactly k listed keys have that score or a better one: those k keys are the k best;
  * otherwise the same search over the low words of the keys with exactly that score finds the last
    one that gets in.
Three forms of the search, chosen by k as the dispatch does:
  * k <= 11: every wave holds the k best of every row and bisects between the least and the greatest image,
    stopping early once exactly k reach the bound;
  * k = 12..32: lists cut to 32 entries, two rows side by side in a register, trees of merges that keep 32 in each
    half, both halves joined, then the same over the waves.  At k = 32 every place is taken and counting
    alone cannot see a tie among the dropped images, so the greatest of those is remembered;
  * k > 32: lists of 64, two chains of merges per wave (a list whose head is below place k-1 of its chain is
    skipped), a tree over the waves; the same remark holds at k = 64.
This file restates those steps on plain Python lists and checks the outcome - which keys are among
the k best - against a full sort of all keys, on inputs full of ties, with rows longer than their
lists, for four and for eight waves.  No GPU, no library call: it pins the reasoning, the GPU tests pin the code.
"""
import random

import pytest


def keep_best(a, b, keep, fell):
    """Top `keep` of two decreasing lists (equal values allowed); fell[0] = greatest value dropped."""
    allv = sorted(a + b, reverse=True)
    for v in allv[keep:]:
        fell[0] = max(fell[0], v)
    return allv[:keep]


def place(lst, i):
    return lst[i] if i < len(lst) else 0


def tree(lists, keep, fell):
    while len(lists) > 1:
        lists = [keep_best(lists[i], lists[i + 1], keep, fell) if i + 1 < len(lists) else lists[i]
                 for i in range(0, len(lists), 2)]
    return lists[0]


# ---- k <= 11: bisection over all entries
def kth_greatest(values, k):
    """(k-th greatest value or 0 if there are fewer, how many reach it: k unless several equal it)"""
    def reached(x):
        return sum(1 for v in values if v >= x)

    def least_from(x):
        return min(v for v in values if v >= x)

    count = reached(1)
    if count < k:
        return 0, count
    lo, hi = least_from(1), max(values)
    while count != k and lo < hi:
        mid = lo + ((hi - lo + 1) >> 1)
        c = reached(mid)
        if c >= k:
            lo, count = mid, c
        else:
            hi = mid - 1
    return least_from(lo), count


def search_by_bisection(rows, k):
    keys = [key for r in rows for key in r]
    tau, count = kth_greatest([s for s, _ in keys], k)
    if tau == 0 or count == k:
        return tau, None
    low, _ = kth_greatest([lo for s, lo in keys if s == tau], k - sum(1 for s, _ in keys if s > tau))
    return tau, low


# ---- k = 12..32: two lists of 32 to a register
def best32(lists, fell):
    """Lists two to a register (0 and 1, 2 and 3, ..): a tree over the registers, half by half, then both halves."""
    lists = lists + [[]] * (len(lists) % 2)
    return keep_best(tree(lists[0::2], 32, fell), tree(lists[1::2], 32, fell), 32, fell)


def search_by_halves(rows, k, waves):
    by_wave = [rows[w::waves] for w in range(waves)]
    fell = [0]
    accs = best32([best32([[s for s, _ in r] for r in rs] or [[]], fell) for rs in by_wave], fell)
    tau = place(accs, k - 1)
    if tau == 0:
        return 0, None
    settled = sum(1 for v in accs if v >= tau) == k
    if settled and k == 32:
        settled = fell[0] < tau
    if settled:
        return tau, None
    need = k - sum(1 for v in accs if v > tau)
    lows = best32([best32([[lo for s, lo in r if s == tau] for r in rs] or [[]], [0]) for rs in by_wave], [0])
    return tau, lows[need - 1]


# ---- k > 32: lists of 64
def wave_best(lists, kth, fell):
    """Two chains side by side (rows 0, 2, 4, .. and 1, 3, 5, .. of the wave), joined at the end."""
    chain = [list(lists[0]) if lists else [], list(lists[1]) if len(lists) > 1 else []]
    for i in range(2, len(lists)):
        a = chain[i % 2]
        if lists[i] and lists[i][0] >= place(a, kth):
            chain[i % 2] = keep_best(a, lists[i], 64, fell)
    return keep_best(chain[0], chain[1], 64, fell) if chain[1] else chain[0]


def search_by_merging(rows, k, waves):
    by_wave = [rows[w::waves] for w in range(waves)]
    fell = [0]
    accs = tree([wave_best([[s for s, _ in r] for r in rs], k - 1, fell) for rs in by_wave], 64, fell)
    tau = place(accs, k - 1)
    if tau == 0:
        return 0, None
    settled = sum(1 for v in accs if v >= tau) == k
    if settled and k == 64:
        settled = fell[0] < tau
    if settled:
        return tau, None
    need = k - sum(1 for v in accs if v > tau)
    lows = tree([wave_best([[lo for s, lo in r if s == tau] for r in rs], need - 1, [0]) for rs in by_wave], 64, [0])
    return tau, lows[need - 1]


def members_by_model(rows, k, waves):
    """rows[h] = decreasing list of distinct keys (score, low) with at most 64 entries.  Returns the
    set of keys the model puts among the k best."""
    if k <= 32:
        rows = [r[:k] for r in rows]               # what the wave holds: no other key of a row can be among the k best
    if k <= 11:
        tau, low = search_by_bisection(rows, k)
    elif k <= 32:
        tau, low = search_by_halves(rows, k, waves)
    else:
        tau, low = search_by_merging(rows, k, waves)
    if tau == 0:                                   # fewer than k keys in all: every key is in
        return {key for r in rows for key in r}
    return {(s, lo) for r in rows for s, lo in r if s > tau or (s == tau and (low is None or lo >= low))}


def random_rows(rng, k, levels, row_len):
    """k rows of row_len distinct keys each; scores on a few levels (ties everywhere), low words
    distinct over the whole sentence.  Each row keeps its best 64 keys, as the stream phase does."""
    lows = rng.sample(range(1, 1 << 20), k * row_len)
    rows = []
    for h in range(k):
        n = rng.choice([0, 1, 3, row_len // 2, row_len]) if rng.random() < 0.3 else row_len
        keys = [(rng.randint(1, levels) + (rng.randint(0, 3) if rng.random() < 0.2 else 0), lows[h * row_len + j])
                for j in range(n)]
        rows.append(sorted(keys, reverse=True)[:64])
    return rows


@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 11, 12, 16, 17, 20, 31, 32, 33, 48, 63, 64])
@pytest.mark.parametrize("levels", [1, 2, 5, 40, 100000])
def test_the_model_finds_exactly_the_k_best(k, levels):
    rng = random.Random(1000 * k + levels)
    for trial in range(60):
        rows = random_rows(rng, k, levels, rng.choice([4, 20, 64, 100]))
        every = sorted((key for r in rows for key in r), reverse=True)
        want = set(every[:k])
        for waves in (4, 8):
            got = members_by_model(rows, k, waves)
            assert got == want, (k, levels, trial, waves, len(every))


@pytest.mark.parametrize("k", [32, 64])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("other", [1, 4, 8, 31])
def test_a_tie_hidden_among_dropped_keys_is_noticed(k, waves, other):
    """Every place taken: two rows of k keys, all with one score, in the same register, wave or not: every place of
    the merged list is taken and counting alone cannot see the tie; the greatest dropped image gives it away."""
    rows = [[] for _ in range(k)]
    rows[0] = [(7, 1000 - j) for j in range(k)]
    rows[other] = [(7, 2000 - j) for j in range(k)]
    assert members_by_model(rows, k, waves) == set(rows[other])


@pytest.mark.parametrize("waves", [4, 8])
def test_without_the_dropped_maximum_the_tie_would_pass_unnoticed(waves, monkeypatch):
    """The case above is one that the remembered maximum decides: a model that forgets it lets both rows in."""
    real = keep_best
    monkeypatch.setitem(globals(), "keep_best", lambda a, b, keep, fell: real(a, b, keep, [0]))
    for k in (32, 64):
        rows = [[(7, 1000 - j) for j in range(k)], [(7, 2000 - j) for j in range(k)]] + [[] for _ in range(k - 2)]
        assert members_by_model(rows, k, waves) == set(rows[0] + rows[1])


@pytest.mark.parametrize("waves", [4, 8])
def test_a_list_whose_head_ties_with_the_running_bar_is_not_skipped(waves):
    """k = 40: one row fills all k places with one score, a later row of the same chain holds one more
    key with that score.  Skipping it (its head does not beat place k-1) would leave exactly k keys in
    sight and let the k+1 keys with that score all pass."""
    k = 40
    rows = [[] for _ in range(k)]
    rows[0] = [(9, 5000 - j) for j in range(40)]
    rows[2 * waves] = [(9, 9000)]                  # wave 0 again, the chain row 0 is in; best low word of all
    every = sorted((key for r in rows for key in r), reverse=True)
    got = members_by_model(rows, k, waves)
    assert got == set(every[:k])
    assert (9, 9000) in got and (9, 5000 - 39) not in got


def test_bisection_stops_early_with_the_right_bound():
    """As soon as exactly k values reach the bound it is lowered to the least of them, wherever the
    bisection stood; with several equal ones at the end it runs until they are all that is left."""
    rng = random.Random(3)
    for trial in range(4000):
        values = [rng.choice([0, rng.randint(1, 6), rng.randint(1, 1 << 32) - 1]) for _ in range(rng.randint(1, 40))]
        k = rng.randint(1, 20)
        live = sorted((v for v in values if v), reverse=True)
        want = live[k - 1] if len(live) >= k else 0
        got, count = kth_greatest(values, k)
        assert got == want, (trial, values, k)
        if want:
            assert (count == k) == (sum(1 for v in live if v >= want) == k), (trial, values, k)
