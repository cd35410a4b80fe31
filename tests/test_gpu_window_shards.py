"""The bin-window kernel's split of the reads over workgroups: read counts around
its shards, and windows so uneven that shards run out at different times.
Whole numbers: equal to the oracle's."""
import numpy as np
import pytest

import grim_synth as gs
from tests.gpu_helpers import assert_same, lib, oracle_run
from tests.test_gpu_window import run_windows, window_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_reads", [1, 7, 63, 64, 65, 513, 9000])
@pytest.mark.parametrize("ordered", [False, True])
def test_uneven_windows(n_reads, ordered):
    g = lib()
    rng = np.random.default_rng(n_reads)
    ref = gs.reference(9, 900_000, 0.2, 20, 300, 0.85, 0.98)
    q, B, O = 5, 200, 105
    nb = -(-ref.size // B)
    lens = rng.integers(0, 120, n_reads)
    reads = [ref[a:a + L] for a, L in zip(rng.integers(0, ref.size - 200, n_reads), lens)]
    # the first eighth of the reads has nearly all of the pairs; sizes around
    # 32, 64 and 128 columns, empty windows among the others
    sizes = rng.choice([0, 1, 5, 33], n_reads)
    big = max(1, n_reads // 8)
    sizes[:big] = rng.choice([1024, 1025, 2047, 2048, 2049, 600], big)
    win_lo = rng.integers(0, nb - 2100, n_reads)
    win_lo[0] = win_lo[0] // 32 * 32
    w = window_workload(ref, q, B, O, reads, rng.integers(0, 1200, n_reads), win_lo, sizes)
    idx = g.grim_build_bins(ref, q, B, O)
    idx.transpose()
    order = "sorted" if ordered else None
    out = run_windows(g, idx, w, win_lo, order=order)
    assert out[2] == 0
    assert_same(out, oracle_run(w), f"{n_reads} reads")
