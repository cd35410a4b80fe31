"""Survivor lists around the block sizes of the list's three passes, against the
set bits of the mask (whole numbers: equal)."""
import numpy as np
import pytest

import grim_synth as gs
import oracle
from tests.gpu_helpers import lib

pytestmark = pytest.mark.gpu

BLOCK = 32768   # pairs of a count block; 128 blocks and more take whole-block workgroups


def _workload(k, cand_bin):
    off = gs.offsets_from_counts(k)
    n = k.size
    return dict(codes=np.zeros(n * 10, np.uint8), read_off=np.arange(n, dtype=np.uint64) * 10,
                read_len=np.full(n, 10, np.uint32), read_e=np.zeros(n, np.uint32), e_den=10000,
                cand_off=off, cand_bin=cand_bin), off


@pytest.mark.parametrize("n_pairs", [1, 31, 2047, 2048, 2049, BLOCK - 1, BLOCK, BLOCK + 33,
                                     127 * BLOCK, 127 * BLOCK + 1, 128 * BLOCK + 4097])
@pytest.mark.parametrize("density", [0.02, 1.0])
def test_block_edges(n_pairs, density):
    import torch
    g = lib()
    rng = np.random.default_rng(n_pairs)
    k = rng.integers(0, 2 * max(1, n_pairs // 3000) + 1, 4000)
    k[rng.random(k.size) < 0.3] = 0
    while k.sum() < n_pairs:
        k[rng.integers(0, k.size)] += int(n_pairs - k.sum() + 1) // 2 + 1
    k[np.searchsorted(np.cumsum(k), n_pairs):] = 0
    k[np.searchsorted(np.cumsum(k), k.sum())] += n_pairs - k.sum()
    w, off = _workload(k.astype(np.uint32), rng.integers(0, 1 << 30, n_pairs).astype(np.uint32))
    assert int(off[-1]) == n_pairs
    words = oracle.pack_bitmask((rng.random(n_pairs) < density).astype(np.uint8))
    want = oracle.survivors(words, n_pairs, off, w["cand_bin"])
    # a mask that starts 4 bytes into its buffer: no wider alignment is promised
    buf = torch.from_numpy(np.concatenate([[0], words, [0xFFFFFFFF]]).astype(np.uint32).view(np.int32)).cuda()
    batch = g.Batch.from_workload(w)
    sp, sr, sb, total = g.grim_compact_survivors(batch, buf[1:])
    assert total == want[0].size
    assert np.array_equal(sp.cpu().numpy().astype(np.uint64)[:total], want[0])
    assert np.array_equal(sr.cpu().numpy().view(np.uint32)[:total], want[1])
    assert np.array_equal(sb.cpu().numpy().view(np.uint32)[:total], want[2])


def test_more_blocks_than_one_scan_round():
    """Over 32768 count blocks (1.07e9 pairs), a few thousand of them set."""
    import torch
    g = lib()
    n = 32768 * BLOCK + 5 * BLOCK + 77
    rng = np.random.default_rng(4)
    at = np.unique(np.concatenate([rng.integers(0, n, 5000), [0, n - 1, 32768 * BLOCK - 1,
                                                              32768 * BLOCK, 32768 * BLOCK + 40]]))
    bits = torch.zeros((n + 31) // 32, dtype=torch.int32, device="cuda")
    word, bit = at // 32, (np.uint32(1) << (at % 32).astype(np.uint32))
    uniq = np.unique(word)
    vals = np.array([np.bitwise_or.reduce(bit[word == u]) for u in uniq], dtype=np.uint32)
    bits[torch.from_numpy(uniq).cuda()] = torch.from_numpy(vals.view(np.int32)).cuda()
    n_reads = 3000
    off = np.linspace(0, n, n_reads + 1).astype(np.uint64)
    w, _ = _workload(np.zeros(n_reads, np.uint32), np.zeros(1, np.uint32))
    batch = g.Batch.from_workload(dict(w, cand_off=off))
    cand = torch.arange(n, dtype=torch.int64, device="cuda").to(torch.int32)
    batch.c.cand_bin = cand.data_ptr()
    sp, sr, sb, total = g.grim_compact_survivors(batch, bits, capacity=at.size)
    assert total == at.size
    assert np.array_equal(sp.cpu().numpy(), at)
    assert np.array_equal(sr.cpu().numpy(), np.searchsorted(off, at, side="right") - 1)
    assert np.array_equal(sb.cpu().numpy().view(np.uint32), at.astype(np.uint32))
