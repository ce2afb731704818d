"""The two counters that the waves of a slab kernel meet at (SlabGate in csrc/lmkan_slab_common.h), as a model on the
host: waves that run in any order and at any speed, some of them without samples.  No slab is read before all of
it has landed, none is overwritten before all have read it, and every walk ends."""
import random

import pytest


def _walk(waves, idle, pairs, rng, first_wait=True):
    landed = read = 0
    slab = [[None] * waves, [None] * waves]      # pair that each wave's part of the two buffers belongs to

    def complete(i):
        assert all(v == i for v in slab[i & 1]), f"pair {i}: {slab[i & 1]}"

    def with_samples(w):
        nonlocal landed, read
        slab[0][w] = 0
        yield
        landed += 1
        for i in range(pairs):
            while landed < waves * (i + 1):
                yield
            complete(i)
            yield
            while read < waves * i:
                yield
            if i + 1 < pairs:
                slab[(i + 1) & 1][w] = i + 1
            yield
            complete(i)
            landed += 1
            yield
            complete(i)
            read += 1
            yield

    def without_samples(w):
        nonlocal landed, read
        slab[0][w] = 0
        yield
        landed += 1
        while first_wait and landed < waves:
            yield
        for i in range(pairs):
            while read < waves * i:
                yield
            if i + 1 < pairs:
                slab[(i + 1) & 1][w] = i + 1
            yield
            landed += 1
            yield
            read += 1
            yield

    running = {w: (without_samples if w < idle else with_samples)(w) for w in range(waves)}
    weight = [rng.random() ** 3 + 1e-3 for _ in range(waves)]     # some waves hardly get a turn
    for _ in range(500000):
        if not running:
            return
        w, = rng.choices(list(running), [weight[v] for v in running])
        for _ in range(rng.randint(1, 20)):
            if next(running[w], "end") == "end":
                del running[w]
                break
    raise AssertionError("a wave waits for ever")


@pytest.mark.parametrize("seed", range(4))
def test_slabs_are_read_complete_and_every_walk_ends(seed):
    rng = random.Random(seed)
    for _ in range(150):
        waves = rng.randint(2, 6)
        _walk(waves, rng.randint(0, waves - 1), rng.randint(1, 7), rng)


def test_the_model_sees_a_missing_wait():
    """Without the wait for the first slab a wave that only fetches reports its second one too early."""
    rng = random.Random(0)
    with pytest.raises(AssertionError, match="pair 0"):
        for _ in range(2000):
            _walk(4, 3, 3, rng, first_wait=False)
