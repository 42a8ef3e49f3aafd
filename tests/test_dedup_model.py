"""A model of the frontier scan (the NeighborSampler's frontier update of
Algorithm 2 in the DGL block convention). The sampler sets bit u of one copy of
the sampled-id bitmap for every id u that it writes; k_frontier then takes

- tiles of old rows (the rows of the frontier so far, NT * ITEMS each; none
  after the last hop), then tiles of TW bitmap words, in any order of blocks;
- in a bitmap tile, w = (copies or-ed) & ~seen: the new nodes. The thread's
  words give its place in the tile (exclusive scan of their counts); the set
  bits are spread into a list of NT * ITEMS entries, chunk by chunk, so that
  thread x of a chunk takes items x, x + NT, ...; every copy's words are cleared,
  the new bits join `seen` (after the last hop `seen` is cleared instead);
- each tile's count of new nodes and of sampled positions (min(row length,
  fanout) of its rows) and their sums over the tiles before it; item j of the
  tile is then row n_prev + nodes before + j (old tiles: row0 + j), with offset
  positions before + those of the tile's items up to j.

Checked against the definition: the new nodes are the ascending unique sampled
ids not in the frontier; every id points at its row; offsets are the prefix sums
over all rows; the count of new local ids is written once; bitmaps end clear (or
hold exactly the frontier). The model restates the kernel's steps at its three
tile shapes; the GPU tests exercise the kernel."""
import random

import pytest

SHAPES = [(256, 64, 8, 8), (256, 256, 4, 1), (512, 2048, 4, 1)]  # threads, words per tile, items, bitmap copies


def popcount(x):
    return bin(x).count("1")


def frontier_scan(shape, F, seen, pos_of, bits, L, last, deg, fo, bptr, rnd):
    NT, TW, items_, copies = shape
    W, chunk = len(seen), NT * items_
    wpt = max(1, TW // NT)
    n_prev = len(F)
    old_tiles = 0 if last else -(-n_prev // chunk)
    ntiles = old_tiles + -(-W // TW)
    # every tile's own part: items in order, words cleared
    tiles, below = [None] * ntiles, []
    for b in rnd.sample(range(ntiles), ntiles):
        if b < old_tiles:
            tiles[b] = [("old", i, F[i]) for i in range(b * chunk, min((b + 1) * chunk, n_prev))]
            continue
        word0, items, place = (b - old_tiles) * TW, {}, 0
        for x in range(min(NT, TW)):
            i0 = word0 + x * wpt
            if i0 >= W:
                continue
            words = [i0 + y for y in range(wpt) if i0 + y < W]
            new = []
            for i in words:
                got = 0
                for c in range(copies):
                    got |= bits[c][i]
                    bits[c][i] = 0
                new.append(got & ~seen[i])
                seen[i] = 0 if last else seen[i] | new[-1]
            if words[0] <= L >> 5 <= words[-1]:
                n = sum(popcount(w) for i, w in zip(words, new) if i < L >> 5)
                below.append((b, place + n + popcount(new[(L >> 5) - words[0]] & ((1 << (L & 31)) - 1))))
            o = place
            for i, w in zip(words, new):
                for bit in range(32):
                    if w >> bit & 1:
                        items[o] = 32 * (i - word0) + bit  # (the list entry: relative to the tile)
                        o += 1
            place = o
        assert sorted(items) == list(range(place)), "every item of the tile exactly once"
        tiles[b] = [("new", j, (word0 << 5) + items[j]) for j in range(place)]
    # sums over the tiles before each (the look-back's result), then the emission
    newF, offs = list(F) + [None] * sum(len(t) for t in tiles[old_tiles:]), {}
    nodes = positions = 0
    sums = []
    for t in tiles:
        sums.append((nodes, positions))
        nodes += sum(k == "new" for k, _, _ in t)
        positions += sum(min(deg[v], fo) for _, _, v in t)
    for b in rnd.sample(range(ntiles), ntiles):
        n_before, run = sums[b]
        for c0 in range(0, len(tiles[b]), chunk):
            for kind, j, v in tiles[b][c0:c0 + chunk]:  # items in list order: NT threads x ITEMS
                i = j if kind == "old" else n_prev + n_before + j
                if kind == "new":
                    assert newF[i] is None
                    newF[i] = v
                    pos_of[v] = i
                run += min(deg[v], fo)
                assert i + 1 not in offs
                offs[i + 1] = run
    if not last:
        bptr[:] = [0] + [offs[i + 1] for i in range(len(newF))]
    local = [sums[b][0] + n for b, n in below]
    if L >> 5 >= W:
        local.append(nodes)  # the last tile: every id is below L
    assert len(local) == 1, "one writer of the local count"
    return newF, local[0]


def run_hops(shape, R, L, density, hops, seed):
    rnd = random.Random(seed)
    W = -(-R // 32)
    deg = [rnd.choice([0, 1, 3, 7, 40]) for _ in range(R)]
    F = rnd.sample(range(L), max(1, L // 50)) if L else []
    pos_of = [rnd.randrange(-5, 5) for _ in range(R)]  # stale positions of earlier steps
    seen = [0] * W
    for i, v in enumerate(F):  # the seeds' launch
        seen[v >> 5] |= 1 << (v & 31)
        pos_of[v] = i
    bits = [[0] * W for _ in range(shape[3])]
    for hop in range(1, hops + 1):
        sampled = [rnd.randrange(R) for _ in range(int(R * density))] + F[:3]  # repeats and ids already in F
        for u in sampled:
            bits[rnd.randrange(shape[3])][u >> 5] |= 1 << (u & 31)
        bptr, fo = [], rnd.randint(1, 9)
        newF, local = frontier_scan(shape, F, seen, pos_of, bits, L, hop == hops, deg, fo, bptr, rnd)
        want = sorted(set(sampled) - set(F))
        assert newF == F + want
        assert local == sum(u < L for u in want)
        assert all(newF[pos_of[u]] == u for u in sampled)
        assert not any(any(c) for c in bits), "bitmap not cleared"
        if hop < hops:
            acc = [0]
            for v in newF:
                acc.append(acc[-1] + min(deg[v], fo))
            assert bptr == acc
            assert [u for u in range(R) if seen[u >> 5] >> (u & 31) & 1] == sorted(newF)
        F = newF
    assert not any(seen), "the frontier bitmap is clear for the next step"


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("R,density,hops", [(33, 0.5, 2), (700, 0.4, 3), (64 * 32 + 5, 0.6, 2), (3 * 64 * 32 + 40, 0.05, 3)])
def test_new_nodes_rows_and_offsets(shape, R, density, hops):
    for seed, L in enumerate((R, R // 2, 1, (R // 64) * 32, R - 1)):
        run_hops(shape, R, L, density, hops, 100 * R + seed)


def test_tiles_of_several_chunks():
    # 2048 words nearly all set: 32 chunks of a tile; and two tiles
    run_hops(SHAPES[2], 2048 * 32 + 77, 40000, 1.5, 1, 5)
    # more old rows than a tile of them holds
    run_hops(SHAPES[0], 5000, 4000, 1.0, 3, 6)


def test_planted_mistake_fails():
    # without `seen` a node of the frontier that is sampled again is new again
    with pytest.raises(AssertionError):
        rnd = random.Random(1)
        F, pos_of = [3, 9], [0] * 64
        pos_of[9] = 1
        newF, _ = frontier_scan(SHAPES[0], F, [0, 0], pos_of, [[1 << 9, 2] if c == 0 else [0, 0] for c in range(8)], 20,
                                True, [1] * 64, 1, [], rnd)
        assert newF == F + [33]
