"""grim_tune and the cut of the pairs: what a large sample chose leaves the cut of
later, smaller batches to their own size."""
import numpy as np
import pytest

import grim_synth as gs
from tests.gpu_helpers import custom_workload, lib, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [4, 5, 6])
def test_small_batch_after_a_large_tune(q):
    import torch
    g = lib()
    max_len = 333 + q                        # a key of its own in the tuning cache
    rng = np.random.default_rng(q)
    ref = gs.reference(5, 300_000)
    B, O = 200, 300
    nb = -(-ref.size // B)

    def batch(n_reads, k):
        reads = [ref[a:a + 100] for a in rng.integers(0, ref.size - 100, n_reads)]
        cands = rng.integers(0, nb, (n_reads, k))
        w = custom_workload(ref, q, B, O, reads, cands, [500] * n_reads)
        return w, g.Batch.from_workload(w, max_len=max_len)

    w, small = batch(64, 64)
    oc, ob, _, _ = oracle_run(w)
    idx = g.grim_build_bins(ref, q, B, O)

    def tickets():
        """Entries of the table of first reads that a tune = NULL call writes."""
        counts, bits = g.alloc_outputs(small.n_pairs)
        ws = torch.full((4096,), 0x5A, dtype=torch.uint8, device="cuda")
        g.grim_filter_batch(idx, small, counts, bits, ws)
        assert g.grim_filter_status(ws) == (0, 0)
        assert np.array_equal(counts.cpu().numpy()[:small.n_pairs], oc)
        assert np.array_equal(bits.cpu().numpy().view(np.uint32)[:ob.size], ob)
        return int((ws.view(torch.int32)[64:] != 0x5A5A5A5A).sum())

    before = tickets()
    assert before == small.n_pairs // 64     # one for every 64 pairs: no wave waits
    _, large = batch(3000, 1000)
    counts, bits = g.alloc_outputs(large.n_pairs)
    ws = g.alloc_workspace(idx, large.n_pairs)
    t = g.grim_tune(idx, large, counts, bits, ws)
    assert t.tile_pairs in (0, 512, 1024, 2048)
    assert tickets() == before
    # a workspace sized for the result serves tune = NULL
    n = g.grim_workspace_size(idx, large.n_pairs, t)
    if t.tile_pairs:
        n = (256 + 4 * -(-large.n_pairs // t.tile_pairs) + 255) & ~255
    ref_counts = counts.clone()
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    for tune in (t, None):
        counts.fill_(-7)
        g.grim_filter_batch(idx, large, counts, bits, ws, tune)
        assert g.grim_filter_status(ws) == (0, 0)
        assert torch.equal(counts, ref_counts)
