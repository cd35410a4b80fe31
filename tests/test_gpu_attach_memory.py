"""Attaching a reference where the device has room for its packed copy alone: the
alignment check works from that, with the same distances."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import custom_workload, lib

pytestmark = pytest.mark.gpu


def test_no_room_for_bit_planes():
    import torch
    g = lib()
    G, B, O = 1_600_000_000, 1000, 200                    # 400 MB packed, 400 MB of planes
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    ref = torch.randint(0, 4, (G,), generator=gen, device="cuda", dtype=torch.uint8).cpu().numpy()
    torch.cuda.empty_cache()
    rng = np.random.default_rng(2)
    reads, es, bins = [], [], []
    for i in range(60):
        at = int(rng.integers(0, G - 130))
        read = ref[at:at + 100 + i % 30].copy()
        for p in rng.integers(0, read.size, i % 9):
            read[p] ^= 1
        reads.append(read)
        es.append(500)
        bins.append([at // B, int(rng.integers(0, G // B))])
    w = custom_workload(ref, 4, B, O, reads, [[] for _ in reads], es)
    idx = g.grim_build_bins(ref, 4, B, O)
    batch = g.Batch.from_workload(w, max_len=130)
    sr = np.repeat(np.arange(len(reads), dtype=np.uint32), 2)
    sb = np.array(bins, dtype=np.uint32).reshape(-1)
    want = oracle.verify(ref, B, O, w["codes"], w["read_off"], w["read_len"], w["read_e"],
                         w["e_den"], sr, sb)
    assert (want <= 5).any() and (want > 5).any()
    dsr, dsb = (torch.from_numpy(x.view(np.int32)).cuda() for x in (sr, sb))

    def check():
        dist, _ = g.grim_verify_survivors(idx, batch, dsr, dsb, sr.size)
        assert np.array_equal(dist.cpu().numpy(), want)

    torch.cuda.synchronize()
    # all memory but 620 MiB: taken until none is left, then given back
    hog = [torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")]
    try:
        while len(hog) < 4000:
            hog.append(torch.empty(62 << 20, dtype=torch.uint8, device="cuda"))
    except torch.cuda.OutOfMemoryError:
        pass
    assert 12 < len(hog) < 4000
    del hog[-10:]
    torch.cuda.empty_cache()
    idx.attach_reference(ref)
    del hog
    torch.cuda.empty_cache()
    check()
    idx.attach_reference(ref)                             # with room: pieces and bands
    check()
