"""The batched filter's own cut of large batches with wide vectors (q = 6, 7):
large tickets followed by a tail of 64-pair ones, their first reads from a table or
searched, as the workspace allows.  Every pair equals the plain form's, a sample
the oracle's."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [6, 7])
@pytest.mark.parametrize("n_pairs", [20_000_003, 70_000_000])
def test_large_and_small_tickets(q, n_pairs):
    import torch
    g = lib()
    rng = np.random.default_rng(q)
    B, O = 500, 300
    ref = gs.reference(3, 2_000_000, 0.3, 20, 300, 0.85, 0.98)
    nb = -(-ref.size // B)
    idx = g.grim_build_bins(ref, q, B, O)
    n = n_pairs // 300
    lens = rng.integers(30, 161, n).astype(np.uint32)
    lens[::7] = 0
    off = np.zeros(n, np.uint64)
    off[1:] = np.cumsum(lens[:-1].astype(np.uint64))
    at = rng.integers(0, ref.size - 200, n)
    src = np.repeat(at - off.astype(np.int64), lens) + np.arange(int(lens.sum()))
    codes = ref[src]
    k = rng.integers(0, 601, n)
    k[rng.integers(0, n, n // 50)] = 0
    k[n // 2:n // 2 + 200] = 0                            # more empty reads than a wavefront holds
    k[5] += 9000
    while k.sum() != n_pairs:
        i = rng.integers(0, n, 1 << 16)
        d = int(n_pairs - k.sum())
        i = np.unique(i)[:abs(d)]
        k[i] = np.maximum(k[i] + np.sign(d), 0)
    coff = np.concatenate([[0], np.cumsum(k)]).astype(np.uint64)
    e = rng.integers(0, 1200, n).astype(np.uint32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(q)
    bins = torch.randint(0, nb, (n_pairs,), generator=gen, device="cuda", dtype=torch.int32)
    batch = g.Batch(codes, off, lens, e, 10000, coff, np.zeros(1, np.uint32), max_len=200 + q)
    batch.c.cand_bin, batch.c.n_pairs, batch.n_pairs = bins.data_ptr(), n_pairs, n_pairs
    want, wbits = g.alloc_outputs(n_pairs)
    g.grim_filter_plain(idx, batch, want, wbits, g.alloc_workspace(idx, n_pairs))

    m = 400                                               # the oracle on the first reads
    p = int(coff[m])
    index = oracle.build_index(ref, B, O, q, n_threads=8)
    oc, op, _ = oracle.filter_batch(index, q, codes, off[:m], lens[:m], e[:m], 10000, coff[:m + 1],
                                    bins[:p].cpu().numpy().view(np.uint32), n_threads=8)
    assert np.array_equal(want[:p].cpu().numpy(), oc)

    counts, bits = g.alloc_outputs(n_pairs)
    for ws_bytes in (g.grim_workspace_size(idx, n_pairs, g.tuning(0, 0, 1024)),
                     g.grim_workspace_size(idx, n_pairs), 256 + n_pairs // 8):
        counts.fill_(-7)
        bits.fill_(-1)
        ws = torch.full((ws_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
        g.grim_filter_batch(idx, batch, counts, bits, ws)
        assert g.grim_filter_status(ws) == (0, 0)
        assert torch.equal(counts, want)
        assert torch.equal(bits[:n_pairs // 32], wbits[:n_pairs // 32])
        table = int((ws[256:].view(torch.int32) != 0x5A5A5A5A).sum())
        # the table has over 32768 tickets of the tail, or the reads were searched
        assert table == 0 or table > 32768
    assert table > n_pairs // 1024 + 32768 // 2
