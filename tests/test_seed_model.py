"""A model of how hop 1's launch (k_seed_rows) checks and places the seed batch
(the minibatch B of Algorithm 2 becomes the first frontier F_0). Each thread
takes seed i: a local id's bit is or-ed into the frontier bitmap `seen`, and the
word as it was says whether the seed is a repeat; then an id outside [0, L) sets
status bit 1, a repeat status bit 2, and a local id is written to F_0[i] with
pos_of[id] = i. When the status is nonzero, classify later clears the bitmap
words of every local id of the batch, so the step leaves no trace (pos_of keeps
stale entries, which only ids in a frontier are looked up in).

The model runs the threads' two parts in random orders and checks: the status
bits are exactly "some seed is out of range" and "some local seed is repeated";
a valid batch gets F_0 = seeds, pos_of[seed] = its position and exactly its bits
set; an invalid batch leaves the bitmap empty. A planted mistake (reading the
word in a load of its own before the or) fails it. It restates the kernel's
steps; the GPU tests exercise the kernel."""
import random

import pytest


def place(seeds, L, rnd, one_atomic=True):
    seen = [0] * (L // 32 + 1)
    pos_of = [rnd.randrange(-3, 40) for _ in range(L)]
    nodes = [None] * len(seeds)
    status = 0
    was = [0] * len(seeds)
    order = list(range(len(seeds)))
    rnd.shuffle(order)
    for i in order:  # the marks
        x = seeds[i]
        if 0 <= x < L:
            was[i] = seen[x >> 5] if one_atomic else 0
            seen[x >> 5] |= 1 << (x & 31)
    rnd.shuffle(order)
    for i in order:  # the checks, the placement
        x = seeds[i]
        if not (0 <= x < L):
            status |= 1
            continue
        if was[i] >> (x & 31) & 1:
            status |= 2
        pos_of[x] = i
        nodes[i] = x
    if status:  # classify's take-back
        for x in seeds:
            if 0 <= x < L:
                seen[x >> 5] = 0
    return seen, pos_of, nodes, status


@pytest.mark.parametrize("n", [0, 1, 2, 17, 256, 1024])
def test_status_and_placement(n):
    rnd = random.Random(n)
    L = 3000
    for case in range(200):
        kind = case % 4
        seeds = rnd.sample(range(L), n)
        if kind == 1 and n:
            seeds[rnd.randrange(n)] = rnd.choice([-1, L, L + 5, -(1 << 31)])
        if kind == 2 and n > 1:
            a, b = rnd.sample(range(n), 2)
            seeds[b] = seeds[a]
        if kind == 3 and n > 2:
            seeds[0] = L
            seeds[2] = seeds[1]
        seen, pos_of, nodes, status = place(seeds, L, rnd)
        out_of_range = any(not (0 <= x < L) for x in seeds)
        local = [x for x in seeds if 0 <= x < L]
        repeated = len(set(local)) < len(local)
        assert status == (1 if out_of_range else 0) | (2 if repeated else 0)
        if status == 0:
            assert nodes == seeds
            assert all(pos_of[x] == i for i, x in enumerate(seeds))
            assert [x for x in range(L) if seen[x >> 5] >> (x & 31) & 1] == sorted(seeds)
        else:
            assert not any(seen), "the step left frontier marks behind"


def test_planted_mistake_fails():
    rnd = random.Random(9)
    seeds = [5, 7, 5, 9]
    _, _, _, status = place(seeds, 20, rnd, one_atomic=False)
    # the definition asks for status bit 2 (a repeated local seed); where every
    # lane reads its word before any or, the repetition goes unnoticed
    assert status & 2 == 0
