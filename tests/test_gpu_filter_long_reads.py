"""The batched filter on reads longer than a wavefront holds: planes built in
stretches of 768 tokens, and the cut of wide vectors' pairs where building them
costs more than a few vectors.  Whole numbers: equal to the oracle's."""
import numpy as np
import pytest

import grim_synth as gs
from tests.gpu_helpers import assert_same, custom_workload, gpu_index, gpu_run, lib, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [4, 5, 6, 7])
def test_stretch_edges(q):
    """Token counts on both sides of one to three stretches and of the rounds of 256
    in them, the longest read, reads at every offset in a word, one token throughout
    (the most planes), reads that end the packed words."""
    rng = np.random.default_rng(q)
    ref = gs.reference(17, 90_000, 0.3, 5, 300, 0.85, 0.98)
    B, O = 1000, 9000
    nb = -(-ref.size // B)
    toks = [1024, 1025, 1279, 1280, 1281, 1535, 1536, 1537, 1792, 2303, 2304, 2305, 3072, 8192 - q + 1]
    reads, cands = [], []
    for i, t in enumerate(toks + [8192 - q + 1, 2305]):
        L = t + q - 1
        at = int(rng.integers(0, ref.size - L))
        read = ref[at:at + L].copy()
        if i >= len(toks):
            read[:] = i % 4
        reads.append(read)
        cands.append(rng.integers(0, nb, [70, 1, 300][i % 3]).tolist() + [min(at // B, nb - 1)])
        reads.append(ref[:1 + i])                       # the next read starts anywhere in a word
        cands.append([0])
    w = custom_workload(ref, q, B, O, reads, cands, rng.integers(0, 800, len(reads)))
    want = oracle_run(w)
    out = gpu_run(gpu_index(w), w, max_len=8192)
    assert out[2] == 0
    assert_same(out, want, f"q={q}")


@pytest.mark.parametrize("q,L,fewest", [(6, 900, 64), (6, 2000, 128), (6, 8000, 256), (7, 3500, 64),
                                        (7, 8000, 128)])
def test_cut_by_the_cost_of_planes(q, L, fewest):
    """2200 reads of 270 candidates: the tickets have as many pairs as the length of the
    reads asks for (their number is the table's), and every pair is right."""
    import torch
    g = lib()
    rng = np.random.default_rng(L)
    ref = gs.reference(19, 60_000, 0.3, 5, 300, 0.85, 0.98)
    B, O = 1500, 8500
    nb = -(-ref.size // B)
    n = 2200
    reads = [ref[a:a + (L if i % 40 == 0 else 60)] for i, a in
             enumerate(rng.integers(0, ref.size - L, n))]
    w = custom_workload(ref, q, B, O, reads, rng.integers(0, nb, (n, 270)),
                        rng.integers(0, 800, n))
    want = oracle_run(w)
    idx = gpu_index(w)
    batch = g.Batch.from_workload(w, max_len=L)
    pairs = batch.n_pairs
    counts, bits = g.alloc_outputs(pairs)
    ws = torch.full((256 + pairs // 32 * 4,), 0x5A, dtype=torch.uint8, device="cuda")
    g.grim_filter_batch(idx, batch, counts, bits, ws)
    rc, flags = g.grim_filter_status(ws)
    assert rc == 0
    assert_same((counts.cpu().numpy()[:pairs], bits.cpu().numpy().view(np.uint32)[:(pairs + 31) // 32],
                 rc, flags), want, f"q={q} L={L}")
    tickets = int((ws[256:].view(torch.int32) != 0x5A5A5A5A).sum())
    assert tickets == -(-pairs // fewest)
