"""Seed candidates of calls that reuse an index's buffers: batches that fit what
earlier calls left, that outgrow it, and that leave it far too large.  Whole
numbers: equal to the oracle's."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import lib

pytestmark = pytest.mark.gpu


def _batch(g, ref, n, L, seed, repeat=0):
    rng = np.random.default_rng(seed)
    at = rng.integers(0, ref.size - L, n)
    if repeat:
        at[:repeat] = 5000                      # the tandem stretch: long hit lists
    codes = np.concatenate([ref[a:a + L] for a in at]) if n else np.zeros(0, np.uint8)
    off = np.arange(n, dtype=np.uint64) * L
    ln = np.full(n, L, np.uint32)
    batch = g.Batch(codes, off, ln, np.zeros(n, np.uint32), 10000, np.zeros(n + 1, np.uint64),
                    np.zeros(0, np.uint32), max_len=L)
    return batch, codes, off, ln


@pytest.mark.parametrize("keep", [False, True])
def test_growing_and_shrinking_batches(keep):
    """n reads in turn: first buffers, a fit, an overflow (the call runs its
    second round), a small one in large buffers, no reads; lists freed before
    the next call or all kept."""
    g = lib()
    rng = np.random.default_rng(8)
    ref = gs.reference(17, 300_000, 0.3, 4, 300, 0.9, 0.99)
    ref[5000:8000] = np.tile(rng.integers(0, 4, 3).astype(np.uint8), 1000)
    si = g.SeedIndex(ref, 8)
    held = []
    for i, (n, L, rep) in enumerate([(50, 60, 0), (40, 60, 0), (3000, 100, 40), (2900, 100, 40),
                                     (3, 20, 1), (0, 20, 0), (6000, 120, 100), (500, 33, 5)]):
        batch, codes, off, ln = _batch(g, ref, n, L, i, rep)
        c = g.grim_seed_candidates(si, batch, 200)
        want_off, want_bin = oracle.seed_candidates(ref, 8, codes, off, ln, 200, 4096)
        got_off, got_bin = c.to_host()
        assert c.n_pairs == want_bin.size, (i, c.n_pairs, want_bin.size)
        assert np.array_equal(got_off, want_off) and np.array_equal(got_bin, want_bin), i
        if keep:
            held.append((c, want_bin))
        del c
    for c, want in held:
        assert np.array_equal(c.to_host()[1], want)


@pytest.mark.parametrize("B", [1, 3, 64, 200, 8191, 1 << 20, (1 << 31) + 1, (1 << 32) - 1, 1 << 32,
                               1 << 40])
def test_strides_and_long_groups(B):
    """Strides around what the multiplied division takes, on reads whose seeds hit
    once, not at all and thousands of times (groups of 64 items with hits beyond
    one round of 2048 places)."""
    g = lib()
    rng = np.random.default_rng(12)
    ref = rng.integers(0, 4, 40_000).astype(np.uint8)
    ref[1000:4100] = 2                          # one k-mer, about 3100 places
    ref[9000:9600] = np.tile([0, 1], 300)
    si = g.SeedIndex(ref, 9)
    batch, codes, off, ln = _batch(g, ref, 300, 95, 5)
    pick = [(1200, 0), (1200, 50), (9100, 0), (39_905, 0), (0, 0)]
    for r, (at, flip) in enumerate(pick):
        codes[r * 95:(r + 1) * 95] = ref[at:at + 95]
        codes[r * 95 + flip] ^= 1
    batch = g.Batch(codes, off, ln, np.zeros(300, np.uint32), 10000, np.zeros(301, np.uint64),
                    np.zeros(0, np.uint32), max_len=95)
    c = g.grim_seed_candidates(si, batch, B)
    want_off, want_bin = oracle.seed_candidates(ref, 9, codes, off, ln, B, 4096)
    got_off, got_bin = c.to_host()
    assert np.array_equal(got_off, want_off) and np.array_equal(got_bin, want_bin)
