"""The alignment check's piece search and diagonal bands on the GPU: distances
are whole numbers and equal the oracle's dynamic programme."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import custom_workload, lib

pytestmark = pytest.mark.gpu


def _mutate(rng, read, k):
    """k random edits (substitution, insertion, deletion), any places."""
    r = list(read)
    for _ in range(k):
        what = rng.integers(0, 3)
        at = int(rng.integers(0, max(1, len(r))))
        if what == 0 and r:
            r[at] = (r[at] + int(rng.integers(1, 4))) & 3
        elif what == 1:
            r.insert(at, int(rng.integers(0, 4)))
        elif r:
            del r[at]
    return np.array(r, dtype=np.uint8)


def _check(ref, B, O, reads, e_nums, bins, max_len, copies=1):
    import torch
    g = lib()
    w = custom_workload(ref, 5, B, O, reads, [[] for _ in reads], e_nums)
    idx = g.grim_build_bins(ref, 5, B, O)
    idx.attach_reference(ref)
    batch = g.Batch.from_workload(w, max_len=max_len)
    sr = np.repeat(np.arange(len(reads), dtype=np.uint32), [len(b) for b in bins])
    sb = np.concatenate([np.asarray(b, dtype=np.uint32) for b in bins])
    want = oracle.verify(ref, B, O, w["codes"], w["read_off"], w["read_len"], w["read_e"],
                         w["e_den"], sr, sb)
    E = (w["read_e"].astype(np.int64) * w["read_len"] + w["e_den"] - 1) // w["e_den"]
    perm = np.random.default_rng(5).permutation(sr.size * copies) % sr.size
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x[perm]).view(np.int32)).cuda()  # noqa: E731
    dist, ok = g.grim_verify_survivors(idx, batch, t(sr), t(sb), perm.size)
    dist = dist.cpu().numpy()
    bad = np.nonzero(dist != want[perm])[0]
    assert bad.size == 0, [(int(sr[perm[i]]), int(sb[perm[i]]), len(reads[sr[perm[i]]]),
                            int(dist[i]), int(want[perm[i]])) for i in bad[:5]]
    okn = np.unpackbits(ok.cpu().numpy().view(np.uint8), bitorder="little")[:perm.size]
    assert np.array_equal(okn.astype(bool), (want <= E[sr])[perm])
    return want, E[sr]


@pytest.mark.parametrize("max_len,B,O", [(64, 50, 90), (128, 200, 140), (256, 200, 275),
                                         (256, 37, 400), (512, 300, 560), (512, 1000, 2200)])
def test_edits_around_the_tolerance(max_len, B, O):
    """Reads with up to two edits more than tolerated, from none to 31 tolerated
    (the most that pieces serve) and past it, in their own bin, the bins beside
    it and others; reads that hang over either end of a bin's span."""
    rng = np.random.default_rng(max_len + B)
    ref = gs.reference(11, 30_011, 0.3, 5, 300, 0.85, 0.98)
    nb = -(-ref.size // B)
    reads, es, bins = [], [], []
    for i in range(220):
        L = int(rng.integers(9, max_len - 36)) if i % 3 else max_len - 36
        E = int(rng.integers(0, max(1, min(33, L // 8) + (i % 5 == 0))))
        st = [0, ref.size - L][i % 2] if i < 6 else int(rng.integers(0, ref.size - L))
        r = _mutate(rng, ref[st:st + L], int(rng.integers(0, E + 3)))
        reads.append(r)
        es.append(E * 10000 // max(1, r.size))
        own = min(st // B, nb - 1)
        bins.append([own, max(0, own - 1), min(nb - 1, own + 1), int(rng.integers(0, nb)), nb - 1])
    want, E = _check(ref, B, O, reads, es, bins, max_len)
    assert (want <= E).sum() > 100 and (want > E).sum() > 100   # the oracle sees both


def test_pieces_that_hit_everywhere():
    """Tandem repeats and long runs: pieces hit on many diagonals (several bands
    of one read, lists of bands running full, the scan of all columns), in
    chunks of every size."""
    rng = np.random.default_rng(3)
    parts = []
    for unit in (1, 2, 3, 7, 13, 29, 61, 90):
        u = rng.integers(0, 4, unit).astype(np.uint8)
        x = np.tile(u, 1500 // unit + 1)[:1500]
        at = rng.random(x.size) < 0.02
        x[at] = rng.integers(0, 4, int(at.sum()))
        parts += [x, rng.integers(0, 4, 500).astype(np.uint8)]
    ref = np.concatenate(parts)
    B, O = 200, 275
    nb = -(-ref.size // B)
    reads, es, bins = [], [], []
    for _ in range(160):
        L = int(rng.choice([80, 100, 150, 240]))
        st = int(rng.integers(0, ref.size - L))
        reads.append(_mutate(rng, ref[st:st + L], int(rng.integers(0, 9)))[:256])
        es.append(int(rng.choice([0, 300, 500, 1000, 1100, 2500])))
        bins.append([st // B, int(rng.integers(0, nb))])
    _check(ref, B, O, reads, es, bins, 256)
    _check(ref, B, O, reads, es, bins, 256, copies=400)
    _check(ref, B, O, reads, es, bins, 256, copies=2000)
