"""Launch shapes with fields left 0: which combinations are accepted, and that
those completed by the library count the same."""
import numpy as np
import pytest

import grim_synth as gs
from tests.gpu_helpers import assert_same, custom_workload, gpu_index, gpu_run, lib, oracle_run

pytestmark = pytest.mark.gpu

LANES, UNROLL = (1, 2, 4, 8, 16, 32, 64), (1, 2, 4, 8)
# field given alone -> values accepted
LANES_ALONE = {4: {1, 2}, 5: {2, 4, 8}, 6: {8, 16, 32}, 7: {32, 64}}
UNROLL_ALONE = {4: {2, 4, 8}, 5: {2, 4, 8}, 6: {1, 2}, 7: {1, 2, 4}}


@pytest.mark.parametrize("q", [4, 5, 6, 7])
def test_accepted_fields(q):
    g = lib()
    rng = np.random.default_rng(q)
    ref = gs.reference(5, 100_000)
    reads = [ref[a:a + 90] for a in rng.integers(0, ref.size - 90, 50)]
    w = custom_workload(ref, q, 200, 300, reads, rng.integers(0, 500, (50, 40)), [500] * 50)
    idx = gpu_index(w)
    want = oracle_run(w)
    pairs = {(t.lanes_per_cand, t.unroll) for t in g.grim_tuning_candidates(q)}
    for lanes in (0,) + LANES:
        for unroll in (0,) + UNROLL:
            tune = g.tuning(lanes, unroll)
            if lanes and unroll:
                ok = (lanes, unroll) in pairs
            elif lanes:
                ok = lanes in LANES_ALONE[q]
            else:
                ok = not unroll or unroll in UNROLL_ALONE[q]
            if not ok:
                with pytest.raises(g.GrimError) as e:
                    g.grim_workspace_size(idx, 2000, tune)
                assert e.value.code == g.GRIM_E_UNSUPPORTED, (lanes, unroll)
            elif not (lanes and unroll):
                out = gpu_run(idx, w, tune=tune)
                assert out[2] == 0
                assert_same(out, want, f"q={q} {lanes} {unroll}")
