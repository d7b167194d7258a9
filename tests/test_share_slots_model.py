"""Model check, on the CPU, of the share slots of the persistent mini-batch kernel (the output sums
that the tiles of a CN exchange each batch step, eq. (2)-(3), section "Fundamentals").

Model: a tile has one word in each of four slots, by step mod 4; an empty word says that its share
has not been published.  At step c a tile publishes its word of slot c, reads every tile's word of
that slot until none is empty, then clears its word of slot c + 2 in another wave.  Stores become
visible some time after they were issued, in order within a wave and in any order between waves.  At
the launch slots 0 and 1 are empty and the others hold what the launch before left.  Random
interleavings check that the rule in use (a tile publishes only when its clears are visible) never
lets a tile take another step's share or lose one, and that without that wait one is taken or
lost, so the check can tell the two apart.
"""
import random


def run(tiles, steps, wait, rng):
    """One random interleaving; returns True if a share of another step was taken, or one was lost."""
    word = [[None, None, "old", "old"] for _ in range(tiles)]
    flight = [([], []) for _ in range(tiles)]     # stores in flight: publishing wave, clearing wave
    at = [0] * tiles                              # step of each tile
    left = [None] * tiles                         # tiles whose share it has yet to read (None: not published)
    idle = 0
    while min(at) < steps:
        if idle > 400 * tiles and not any(w for f in flight for w in f):
            return True                           # (every tile waits for a share that was cleared)
        idle += 1
        i = rng.randrange(tiles)
        if rng.random() < 0.4:
            w = rng.choice(flight[i])
            if w:
                slot, v = w.pop(0)
                word[i][slot] = v
                idle = 0
        elif at[i] == steps or (left[i] is None and wait and flight[i][1]):
            continue
        elif left[i] is None:
            flight[i][0].append((at[i] & 3, at[i]))
            left[i] = set(range(tiles))
        else:
            j = rng.choice(sorted(left[i]))
            v = word[j][at[i] & 3]
            if v is None:
                continue
            if v != at[i]:
                return True
            left[i].discard(j)
            idle = 0
            if not left[i]:
                flight[i][1].append(((at[i] + 2) & 3, None))
                at[i] += 1
                left[i] = None
    return False


def test_publishing_behind_the_clears_is_safe():
    rng = random.Random(11)
    for _ in range(1500):
        assert not run(rng.randint(1, 5), rng.randint(1, 12), True, rng)


def test_publishing_before_the_clears_are_visible_is_not():
    rng = random.Random(12)
    assert sum(run(rng.randint(2, 5), rng.randint(4, 12), False, rng) for _ in range(1500)) > 0
