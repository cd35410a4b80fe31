"""Device memory held by candidate lists: small lists kept after large ones were
freed hold buffers of their own size, whatever buffers the index has to hand."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import lib

pytestmark = pytest.mark.gpu

K, B = 6, 20


def _batch(g, codes, n, L):
    off = np.arange(n, dtype=np.uint64) * L
    ln = np.full(n, L, np.uint32)
    return g.Batch(codes, off, ln, np.zeros(n, np.uint32), 10000, np.zeros(n + 1, np.uint64),
                   np.zeros(0, np.uint32), max_len=L), codes, off, ln


@pytest.mark.parametrize("small", ["few reads", "no hits"])
def test_small_lists_after_large_ones(small):
    """`few reads`: the small batch is small.  `no hits`: it has as many seeds as the
    large one, which occur nowhere, so that its size shows only at its end."""
    import torch
    g = lib()
    rng = np.random.default_rng(3)
    ref = rng.integers(0, 3, 300_000).astype(np.uint8)        # no base 3
    si = g.SeedIndex(ref, K)
    n, L = 9_000, 96
    at = rng.integers(0, ref.size - L, n)
    big, *_ = _batch(g, np.concatenate([ref[a:a + L] for a in at]), n, L)
    if small == "few reads":
        little = _batch(g, ref[500:500 + 3 * 30].copy(), 3, 30)
    else:
        codes = np.full(n * L, 3, np.uint8)
        codes[5 * L:6 * L] = ref[40:40 + L]                   # but for one read
        little = _batch(g, codes, n, L)
    want_off, want_bin = oracle.seed_candidates(ref, K, *little[1:], B, 4096)

    first = g.grim_seed_candidates(si, big, B)
    size = first.n_pairs * 4
    assert size > 90 << 20                # past the 64 MiB that any list may leave unused
    del first
    held = []
    free0 = None
    for i in range(7):
        c = g.grim_seed_candidates(si, big, B)
        assert c.n_pairs * 4 == size
        del c
        held.append(g.grim_seed_candidates(si, little[0], B))
        torch.cuda.synchronize()
        if i == 0:
            free0 = torch.cuda.mem_get_info()[0]
    assert free0 - torch.cuda.mem_get_info()[0] < size
    for c in held:
        got_off, got_bin = c.to_host()
        assert np.array_equal(got_off, want_off) and np.array_equal(got_bin, want_bin)
