"""Host model of the packed gather kernel's split summations: every step of
every shared tile belongs to one share, and the fix-up reads, in share order,
exactly the workspace slots the shares wrote."""
import pytest


def begin(I, S, s):
    return I * s // S


@pytest.mark.parametrize("tiles,steps", [(1, 1), (1, 9), (2, 7), (3, 1), (5, 12), (17, 4), (100, 23)])
def test_shares_cover_the_steps_and_the_fixup_finds_them(tiles, steps):
    I = tiles * steps
    for S in sorted({1, 2, 3, tiles, tiles + 1, 2 * tiles - 1, max(1, I // 2), I - 1, I} & set(range(1, I + 1))):
        done, slots, whole = {}, {}, set()
        for s in range(S):
            it, end = begin(I, S, s), begin(I, S, s + 1)
            first = it // steps
            assert end > it   # no share is empty
            while it < end:
                tile = it // steps
                s0 = it - tile * steps
                s1 = min(steps, s0 + end - it)
                for x in range(s0, s1):
                    assert (tile, x) not in done
                    done[tile, x] = s
                if s1 - s0 == steps:
                    whole.add(tile)
                else:
                    slot = 2 * s + (0 if tile == first else 1)
                    assert slot not in slots   # a share begins at most two split tiles
                    slots[slot] = (tile, s)
                it += s1 - s0
        assert len(done) == I
        for tile in range(tiles):
            x0, x1 = tile * steps, (tile + 1) * steps - 1
            lo, hi = ((x0 + 1) * S - 1) // I, ((x1 + 1) * S - 1) // I
            assert lo == done[tile, 0] and hi == done[tile, steps - 1]
            if lo == hi:
                assert tile in whole
                continue
            assert tile not in whole
            read = [2 * lo + (0 if begin(I, S, lo) >= x0 else 1)] + [2 * s for s in range(lo + 1, hi + 1)]
            assert [slots[r] for r in read] == [(tile, s) for s in range(lo, hi + 1)]


@pytest.mark.parametrize("tiles,steps", [(1, 2), (2, 7), (5, 12), (17, 4), (64, 9), (100, 23)])
def test_slots_of_at_most_as_many_tiles_as_shares(tiles, steps):
    """With the slot s + t every piece has its own, below shares + tiles, and a
    tile's pieces lie next to each other in share order."""
    I = tiles * steps
    for S in sorted({tiles, tiles + 1, 2 * tiles - 1, 3 * tiles, I - 1, I} & set(range(tiles, I + 1))):
        slots = {}
        for s in range(S):
            it, end = begin(I, S, s), begin(I, S, s + 1)
            while it < end:
                t = it // steps
                n = min(end, (t + 1) * steps) - it
                if n < steps:
                    assert s + t not in slots and s + t < S + tiles
                    slots[s + t] = (s, t, n)
                it += n
        for t in range(tiles):
            x0, x1 = t * steps, (t + 1) * steps - 1
            lo, hi = ((x0 + 1) * S - 1) // I, ((x1 + 1) * S - 1) // I
            if lo < hi:
                assert [slots[s + t][:2] for s in range(lo, hi + 1)] == [(s, t) for s in range(lo, hi + 1)]
                assert sum(slots[s + t][2] for s in range(lo, hi + 1)) == steps
