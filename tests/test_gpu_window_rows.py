"""Bin windows on a row buffer past 4 GiB (64-bit row offsets), starting on row
words and off them, with 8 and 16 planes a counter: counts and pass bits equal
the batched filter's on the same (read, bin) pairs."""
import numpy as np
import pytest

from tests.gpu_helpers import custom_workload, lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def big_rows():
    g = lib()
    rng = np.random.default_rng(5)
    B, O = 16, 1100
    n_bins = (1 << 21) + 70                       # 16384 rows of 256 KiB and more
    ref = rng.integers(0, 4, n_bins * B - 3).astype(np.uint8)
    idx = g.grim_build_bins(ref, 7, B, O)
    idx.transpose()
    yield g, ref, idx, B, O, n_bins
    del idx


@pytest.mark.parametrize("max_len", [120, 900])
def test_rows_past_4_gib(big_rows, max_len):
    import torch
    g, ref, idx, B, O, n_bins = big_rows
    rng = np.random.default_rng(max_len)
    sizes = [1, 31, 32, 33, 700, 1024, 2100, 4096, 4097, 9000] * 2
    lo, reads, cands = [], [], []
    for i, n in enumerate(sizes):
        at = int(rng.integers(0, n_bins - n)) if i else n_bins - n   # up to the last bin
        lo.append(at // 32 * 32 if i % 2 else at)
        L = max_len if i % 3 else int(rng.integers(7, max_len))
        p = min(at * B, ref.size - L)
        reads.append(ref[p:p + L])
        cands.append(np.arange(lo[-1], lo[-1] + n))
    w = custom_workload(ref, 7, B, O, reads, cands, [700] * len(reads))
    batch = g.Batch.from_workload(w, max_len=max_len)
    n = batch.n_pairs
    want, wbits = g.alloc_outputs(n)
    g.grim_filter_batch(idx, batch, want, wbits, g.alloc_workspace(idx, n))
    counts, bits = g.alloc_outputs(n)
    counts.fill_(-7)
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    win_lo = torch.tensor(lo, dtype=torch.int32, device="cuda")
    g.grim_filter_windows(idx, batch, win_lo, counts, bits, ws)
    assert g.grim_filter_status(ws) == (0, 0)
    assert torch.equal(counts[:n], want[:n])
    m = n // 32
    assert torch.equal(bits[:m], wbits[:m])
    assert int(want[:n].max()) >= 60              # the read's own bin is among them
