"""The batched filter's work split on the GPU: pairs cut into tickets, reads
taken 64 at a time, packed bases held by the lanes.  Counts and pass bits are
whole numbers: every one equals the oracle's."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import custom_workload, gpu_index, lib, oracle_run

pytestmark = pytest.mark.gpu


def _run(g, idx, batch, ws_bytes, tune=None):
    import torch
    n = batch.n_pairs
    counts, bits = g.alloc_outputs(n)
    counts.fill_(-7)
    bits.fill_(-1)
    ws = torch.full((ws_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
    g.grim_filter_batch(idx, batch, counts, bits, ws, tune)
    rc, flags = g.grim_filter_status(ws)
    return (counts.cpu().numpy()[:n], bits.cpu().numpy().view(np.uint32)[:(n + 31) // 32],
            rc, flags)


def _edge_workload(q, seed):
    """Reads around every limit of the lane-held form (no token, one token, 16-base
    words, the 1024 bases a wavefront holds at any offset in a word, longer ones),
    candidate lists around block and step sizes, and runs of over 64 reads
    without candidates."""
    rng = np.random.default_rng(seed)
    ref = gs.reference(31 + seed, 60_000, 0.3, 5, 300, 0.85, 0.98)
    B, O = 500, 1700
    nb = -(-ref.size // B)
    lens = [0, 1, q - 1, q, 15, 16, 17, 63, 64 + q, 255 + q, 256 + q, 257 + q, 1000] + \
        list(range(1008, 1027)) + [1500]
    rng.shuffle(lens)
    counts = [1, 2, 15, 16, 17, 31, 63, 64, 65, 130, 700]
    reads, cands = [], []
    for i, L in enumerate(lens):
        at = int(rng.integers(0, ref.size - L))
        read = ref[at:at + L].copy()
        if i % 7 == 3 and L:
            read[:] = i % 4                      # one token, multiplicity L - q + 1
        reads.append(read)
        cands.append(rng.integers(0, nb, counts[i % len(counts)]).tolist())
        if i in (2, 9):
            for _ in range(70 if i == 2 else 130):
                reads.append(ref[:20])
                cands.append([])
        if i == 20:
            for _ in range(150):                 # more reads than a wavefront holds, one pair each
                reads.append(ref[i:i + 40])
                cands.append([int(rng.integers(0, nb))])
    e = rng.integers(0, 1500, len(reads))
    e[0] = 0xFFFFFFFF                            # threshold far below zero
    return custom_workload(ref, q, B, O, reads, cands, e), 1500


@pytest.mark.parametrize("q", [4, 5, 6, 7])
def test_ticket_and_read_edges(q):
    g = lib()
    w, max_len = _edge_workload(q, q)
    oc, ob, bad, _ = oracle_run(w)
    idx = gpu_index(w)
    batch = g.Batch.from_workload(w, max_len=max_len)
    n = batch.n_pairs
    small = g.grim_workspace_size(idx, n)        # no room for a table of 64-pair tickets
    large = 256 + 4 * n
    tunes = [None] + [g.tuning(0, 0, t, 1) for t in (64, 192, 4096)] + list(g.grim_tuning_candidates(q))
    for c in tunes[4:]:
        c.tile_pairs = 0
    for i, tune in enumerate(tunes):
        for ws in (small, large):
            if ws == small and i in (1, 2):
                ws = g.grim_workspace_size(idx, n, tune)
            c, b, rc, flags = _run(g, idx, batch, ws, tune)
            assert rc == 0 and flags == 0
            assert np.array_equal(c, oc), (q, i, ws)
            assert np.array_equal(b, ob), (q, i, ws)


@pytest.mark.parametrize("n_reads,k", [(65, 1), (1, 5000), (1100, 120), (4000, 900)])
def test_tickets_by_batch_size(n_reads, k):
    """From fewer pairs than one ticket to enough that waves draw several."""
    g = lib()
    rng = np.random.default_rng(n_reads)
    ref = gs.reference(7, 400_000)
    lens = rng.integers(20, 60, n_reads)
    reads = [ref[a:a + L] for a, L in zip(rng.integers(0, 399_000, n_reads), lens)]
    nb = -(-ref.size // 200)
    counts = np.full(n_reads, k) if n_reads < 1000 else rng.integers(0, 2 * k, n_reads)
    flat = rng.integers(0, nb, int(counts.sum())).astype(np.uint32)
    cands = np.split(flat, np.cumsum(counts)[:-1])
    w = custom_workload(ref, 5, 200, 105, reads, cands, [500] * n_reads)
    oc, ob, _, _ = oracle_run(w)
    idx = gpu_index(w)
    batch = g.Batch.from_workload(w)
    for ws in (g.grim_workspace_size(idx, batch.n_pairs), 256 + batch.n_pairs // 8):
        c, b, rc, _ = _run(g, idx, batch, max(ws, 512))
        assert rc == 0
        assert np.array_equal(c, oc) and np.array_equal(b, ob)


def test_pairs_outside_every_read():
    """Offsets that start late or end early: the pairs no read owns count -1 and
    flag the batch, the others keep their results."""
    g = lib()
    rng = np.random.default_rng(1)
    ref = gs.reference(3, 100_000)
    reads = [ref[a:a + 100] for a in (0, 500, 7000, 9000)]
    cands = [rng.integers(0, 500, m).tolist() for m in (200, 70, 0, 333)]
    w = custom_workload(ref, 5, 200, 105, reads, cands, [500] * 4)
    oc, ob, _, _ = oracle_run(w)
    p = oracle.pack_bitmask
    bits = np.unpackbits(ob.view(np.uint8), bitorder="little")[:oc.size]
    idx = gpu_index(w)
    for lo, hi in ((70, 0), (0, 100), (130, 65)):
        w2 = dict(w, cand_off=np.clip(w["cand_off"], lo, oc.size - hi).astype(np.uint64))
        batch = g.Batch.from_workload(w2)
        batch.c.n_pairs = oc.size
        batch.n_pairs = oc.size
        want, wbits = oc.copy(), bits.copy()
        out = np.r_[0:lo, oc.size - hi:oc.size]
        want[out], wbits[out] = -1, 0
        for ws in (512, 4096):
            c, b, rc, flags = _run(g, idx, batch, ws)
            assert rc == g.GRIM_E_READ and flags == g.GRIM_FLAG_CAND_OFF
            assert np.array_equal(c, want) and np.array_equal(b, p(wbits))
