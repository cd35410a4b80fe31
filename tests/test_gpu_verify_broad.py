"""The alignment check of long lists whose chunks hold more broad bands than the short
lists' 512, all that the long lists' 1,536 have room for, and more: every read has
`copies` copies in its span, `apart` bases from each other, so that its pieces hit that
far apart.  Distances are whole numbers and equal the oracle's dynamic programme."""
import numpy as np
import pytest

from tests.test_gpu_verify_pieces import _check, _mutate

pytestmark = pytest.mark.gpu


# bands of 128 diagonals less twice the 6 edits: 1, 1, 2 and 3 a survivor
@pytest.mark.parametrize("apart", [70, 110, 180, 300])
@pytest.mark.parametrize("share", [0.55, 1.0])
def test_broad_bands_of_a_chunk(apart, share):
    rng = np.random.default_rng(apart)
    B = 600
    ref, reads, bins = [], [], []
    for i in range(140):
        x = rng.integers(0, 4, B).astype(np.uint8)
        s = rng.integers(0, 4, 60).astype(np.uint8)
        x[40:100] = s
        if i < 140 * share:
            x[40 + apart:100 + apart] = s
        ref.append(x)
        reads.append(_mutate(rng, s, int(rng.integers(0, 5))))
        bins.append([i])
    reads = [r[:64] for r in reads]
    want, E = _check(np.concatenate(ref), B, 64, reads, [1000] * len(reads), bins, 64,
                     copies=2000)   # 280,000
    assert (want <= E).mean() > 0.9
