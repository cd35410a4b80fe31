"""The alignment check of long lists: pieces and bands in one launch, the scan of
all columns in another for the survivors it left, for every read-length class;
and batches whose spans are too long for pieces.  Distances are whole numbers and
equal the oracle's dynamic programme."""
import numpy as np
import pytest

from tests.test_gpu_verify_pieces import _check, _mutate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_len", [64, 128, 256, 512])
@pytest.mark.parametrize("tols", [(0, 300, 1100, 2500), (2500,), (300,), (300,) * 15 + (2500,),
                                  (300, 2500)])
def test_pieces_scan_and_both(max_len, tols):
    """Lists of over 1024 survivors a CU: chunks with pieces, without, with a few
    and half of each; tandem repeats whose bands find no room."""
    rng = np.random.default_rng(max_len + len(tols))
    parts = []
    for unit in (1, 2, 3, 7, 29, 61):
        x = np.tile(rng.integers(0, 4, unit).astype(np.uint8), 1500 // unit + 1)[:1500]
        at = rng.random(x.size) < 0.02
        x[at] = rng.integers(0, 4, int(at.sum()))
        parts += [x, rng.integers(0, 4, 500).astype(np.uint8)]
    ref = np.concatenate(parts)
    B, O = 200, max_len + 75
    nb = -(-ref.size // B)
    reads, es, bins = [], [], []
    for i in range(150):
        L = int(rng.integers(max(9, max_len // 4), max_len - 8)) if i else 0
        st = int(rng.integers(0, ref.size - L))
        reads.append(_mutate(rng, ref[st:st + L], int(rng.integers(0, 8)) if L else 0)[:max_len])
        es.append(int(rng.choice(tols)))
        bins.append([st // B, int(rng.integers(0, nb))])
    want, E = _check(ref, B, O, reads, es, bins, max_len, copies=950)   # 285,000
    assert (want <= E).any() and (want > E).any()


@pytest.mark.parametrize("copies", [1, 1200])
def test_spans_too_long_for_pieces(copies):
    rng = np.random.default_rng(4)
    ref = rng.integers(0, 4, 61_000).astype(np.uint8)
    B, O = 30_000, 130
    reads, es, bins = [], [], []
    for i in range(80):
        L = int(rng.integers(20, 60))
        st = int(rng.integers(0, ref.size - L))
        reads.append(_mutate(rng, ref[st:st + L], int(rng.integers(0, 4)))[:64])
        es.append(int(rng.choice([0, 500])))
        bins.append([st // B, 2, int(rng.integers(0, 3))])
    _check(ref, B, O, reads, es, bins, 64, copies=copies)
