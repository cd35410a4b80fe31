"""Timed cases of the library's device paths, through its Python entry points.

The cases are the steps a read mapper has the library do for a batch of reads,
with the reference's index already built: the batched filter (q = 4..7, from a
handful of reads to the 3.1 Gbp workload), the survivor list, the alignment
check, the bin-window form, device seeding, the whole chain for one batch, and
a served request.  Genome and read sizes, bin strides and overlaps, error
tolerances and candidate counts are those of grim_synth's workloads, of the
benchmark and of the GPU tests; inputs are made on the GPU from the seed.

listed()             the named cases
draw(rng)            one more case of the same ranges
prepare(case, seed)  inputs, index and buffers of a case
run(state)           one pass
work(case)           bytes a pass cannot do without
exact(case, seed)    counts and pass bits in plain torch, where that is cheap
"""
import math

import numpy as np
import torch

import paper_1711_01177_amd as grim

E_DEN = 10000
DEV = "cuda"


# ----------------------------------------------------------------------- cases
def _case(kind, name=None, **kw):
    c = dict(kind=kind, genome=100_000_000, repeat=0.1, q=5, stride=200, overlap=275, reads=1000,
             lens="100,150,250", tol="500,1000", cand="zipf", cand_max=4096)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one mapper thread's small batch: launches and latency are what it costs
        _case("filter", "filter_64_reads", genome=1_000_000, repeat=0.0, overlap=105, reads=64,
              lens="100", tol="500", cand="fixed", cand_max=64),
        # an ordinary batch on a chromosome-sized index, which the caches hold
        _case("filter", "filter_mid", reads=100_003),
        # the benchmark's 3.1 Gbp batch: random vectors of a 2 GB index
        _case("filter", "filter_genome_q5", genome=3_100_000_000, repeat=0.45, reads=4_000_000),
        # longer tokens, larger bins: 512-byte vectors, uniform candidate counts
        _case("filter", "filter_genome_q6", genome=3_100_000_000, repeat=0.45, q=6, stride=1000,
              overlap=263, reads=200_000, lens="250", tol="500", cand="uniform", cand_max=2048),
        # the longest tokens with long reads: 2 KiB vectors, many multiplicity planes
        _case("filter", "filter_q7_long_reads", q=7, stride=1000, overlap=2200, reads=20_001,
              lens="333,1000,2000", tol="500", cand="uniform", cand_max=512),
        # the survivor list of the benchmark's batch
        _case("survivors", "survivors_genome", genome=3_100_000_000, repeat=0.45, reads=4_000_000),
        # the alignment check of a batch's survivors
        _case("verify", "verify_mid", genome=400_000_000, repeat=0.45, reads=1_000_000),
        # 4096-bin windows on the mapper's 1024-bin grid, in the device's processing order
        _case("windows", "windows_genome", genome=3_100_000_000, repeat=0.45, reads=200_000,
              cand="fixed", cand_max=4096, grid=1024, ordered=True),
        # windows of any size starting anywhere, in index order
        _case("windows", "windows_ragged", reads=5_001, cand="uniform", cand_max=3000, grid=1,
              ordered=False),
        # k-mer seeding of a million reads
        _case("seed", "seed_mid", overlap=105, reads=1_000_000, lens="100", tol="500", cand_max=4096,
              k=12),
        # the whole chain for one batch: seeds, filter, survivors, alignment
        _case("chain", "chain_5000_reads", overlap=275, reads=5_000, k=12),
        # one request of a mapper to a running server, results back in host memory
        _case("serve", "serve_request", reads=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["filter", "filter", "filter", "survivors", "verify", "windows", "windows",
                       "seed", "chain", "serve"])
    c = _case(kind)
    c["lens"] = rng.choice(["100", "100,150,250", "250", "76,101,151"])
    c["tol"] = rng.choice(["500", "1000", "500,1000"])
    longest = max(int(x) for x in c["lens"].split(","))
    c["overlap"] = longest + longest // 10
    c["repeat"] = rng.choice([0.0, 0.1, 0.45])
    if kind == "filter":
        c["q"] = rng.choice([4, 5, 5, 5, 6, 6, 7])
        if c["q"] == 7 and rng.random() < 0.5:
            c["lens"], c["overlap"] = rng.choice([("500,1500", 1650), ("1000", 1100)])
        c["stride"] = {4: 100, 5: 200, 6: 1000, 7: 2000}[c["q"]] + rng.randrange(50)
        c["genome"] = _log(rng, 1e6, 3e9 if c["q"] > 4 else 1e9)
        c["cand"] = rng.choice(["zipf", "uniform", "fixed"])
        c["cand_max"] = _log(rng, 8, 4096 if c["cand"] == "zipf" else 1024)
        vb = 4 ** c["q"] // 8
        c["reads"] = _log(rng, 16, max(64, min(2e6, 4e10 / (vb + 8) / _mean_cand(c))))
    elif kind == "survivors":
        c["genome"], c["reads"] = _log(rng, 1e7, 1e9), _log(rng, 100, 1e6)
    elif kind == "verify":
        c["genome"], c["reads"] = _log(rng, 1e7, 2e8), _log(rng, 500, 6e5)
    elif kind == "windows":
        c["genome"] = _log(rng, 1e7, 3e9)
        c["cand"] = rng.choice(["uniform", "fixed"])
        c["cand_max"] = _log(rng, 64, 6000)
        c["reads"] = _log(rng, 64, 4e8 / _mean_cand(c) if c["cand_max"] > 2000 else 2e5)
        c["grid"] = rng.choice([1, 1, 32, 1024])
        c["ordered"] = rng.random() < 0.5
    elif kind == "seed":
        c["genome"], c["k"] = _log(rng, 2e7, 1e8), rng.choice([11, 12, 13])
        c["repeat"] = rng.choice([0.0, 0.1])
        c["reads"] = _log(rng, 100, 8e5)
    elif kind == "chain":
        c["genome"], c["k"], c["reads"] = _log(rng, 2e7, 1e8), 12, _log(rng, 100, 2e4)
        c["repeat"] = rng.choice([0.0, 0.1])
    else:
        c["genome"], c["reads"] = _log(rng, 1e6, 2e8), _log(rng, 8, 4096)
    return c


# ---------------------------------------------------------------------- inputs
class DeviceBatch:
    """A batch whose arrays are on the GPU already (as a mapper that seeds
    there has them)."""

    def __init__(self, rd, cand_off, cand_bin, n_pairs, max_len):
        self.words, self.read_off, self.read_len, self.read_e = rd
        self.cand_off, self.cand_bin = cand_off, cand_bin
        self.n_reads, self.n_pairs, self.max_len = int(self.read_len.numel()), int(n_pairs), max_len
        self.c = grim.grim_batch_t(
            self.words.data_ptr(), self.words.numel(), self.read_off.data_ptr(),
            self.read_len.data_ptr(), self.read_e.data_ptr(), E_DEN, max_len,
            cand_off.data_ptr() if cand_off is not None else None,
            cand_bin.data_ptr() if cand_bin is not None else None, self.n_reads, self.n_pairs)


class DeviceArray:
    """A device buffer the library owns, for torch.as_tensor."""

    def __init__(self, ptr, n, typestr, owner):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (int(n),), "typestr": typestr,
                                         "data": (int(ptr), False), "version": 2}


def _ints(text):
    return [int(x) for x in text.split(",")]


def _genome(case, g):
    """Base codes (uint8, GPU): uniform, with a share of the 300-base slots
    overwritten by copies of repeat families at 85-98 % identity."""
    G = case["genome"]
    codes = torch.randint(0, 4, (G,), generator=g, device=DEV, dtype=torch.uint8)
    if case["repeat"] and G >= 3000:
        n_fam = 100 if G <= 200_000_000 else 10_000
        fam = torch.randint(0, 4, (n_fam, 300), generator=g, device=DEV, dtype=torch.uint8)
        slots = codes[:G // 300 * 300].view(-1, 300)
        at = torch.nonzero(torch.rand(slots.shape[0], generator=g, device=DEV) < case["repeat"])[:, 0]
        for a in at.split(1 << 20):
            rep = fam[torch.randint(0, n_fam, a.shape, generator=g, device=DEV)]
            off = torch.rand(a.numel(), 1, generator=g, device=DEV) * 0.13 + 0.02
            mut = torch.rand(rep.shape, generator=g, device=DEV) < off
            slots[a] = (rep + mut * torch.randint(1, 4, rep.shape, generator=g, device=DEV,
                                                  dtype=torch.uint8)) & 3
    return codes


def _pack(codes):
    """2-bit words (int32, GPU): 16 bases a word, first base on top, one zero word after."""
    n = codes.numel()
    out = torch.zeros((n + 15) // 16 + 1, dtype=torch.int32, device=DEV)
    step = 1 << 28
    for a in range(0, n, step):
        x = codes[a:a + step]
        if x.numel() % 16:
            x = torch.cat([x, x.new_zeros(16 - x.numel() % 16)])
        x = x.view(-1, 16)
        w = out[a // 16:a // 16 + x.shape[0]]
        for j in range(16):
            w |= x[:, j].to(torch.int32) << (30 - 2 * j)
    return out


def _reads(case, codes, g):
    """Reads copied from random places with up to the tolerated share of edits
    (substitutions, insertions and deletions), packed back to back."""
    n, G = case["reads"], codes.numel()
    lens = torch.tensor(_ints(case["lens"]), device=DEV)
    tols = torch.tensor(_ints(case["tol"]), device=DEV)
    L = lens[torch.randint(0, len(lens), (n,), generator=g, device=DEV)]
    e = tols[torch.randint(0, len(tols), (n,), generator=g, device=DEV)]
    lmax = int(lens.max())
    z = (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (G - lmax * 1.2)).long()
    rate = torch.rand(n, generator=g, device=DEV) * e / E_DEN
    parts = []
    i = torch.arange(lmax, device=DEV)
    step = max(1, (1 << 26) // lmax)
    for a in range(0, n, step):
        s = slice(a, a + step)
        m = L[s].numel()
        hit = torch.rand(m, lmax, generator=g, device=DEV) < rate[s, None]
        what = torch.randint(0, 3, (m, lmax), generator=g, device=DEV, dtype=torch.int32) * hit
        ins, dele = hit & (what == 1), hit & (what == 2)
        shift = torch.cumsum(dele.int() - ins.int(), 1)
        src = (z[s, None] + i + shift).clamp_(0, G - 1)
        x = codes[src]
        x = (x + (hit & (what < 2)) * torch.randint(1, 4, x.shape, generator=g, device=DEV,
                                                    dtype=torch.uint8)) & 3
        parts.append(x[i < L[s, None]])
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(L, 0, out=off[1:])
    words = _pack(torch.cat(parts))
    return (words, off[:-1].contiguous(), L.int(), e.int()), z, lmax


def _zipf_table(k):
    w = torch.arange(1, k + 1, dtype=torch.float64) ** -1.2
    return torch.cumsum(w / w.sum(), 0)


def _mean_cand(case):
    k = case["cand_max"]
    if case["cand"] == "fixed":
        return float(k)
    if case["cand"] == "uniform":
        return (k + 1) / 2
    w = np.arange(1, k + 1, dtype=np.float64)
    return float((w ** -0.2).sum() / (w ** -1.2).sum())


def _offsets(case, g):
    """CSR offsets: the quantiles of the distribution of candidate counts (so
    that their sum is the case's own), in an order drawn from the seed."""
    n, k = case["reads"], case["cand_max"]
    at = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
    if case["cand"] == "fixed":
        c = torch.full((n,), k, dtype=torch.int64, device=DEV)
    elif case["cand"] == "uniform":
        c = 1 + (at * k).long()
    else:
        c = 1 + torch.searchsorted(_zipf_table(k).to(DEV), at)
        c.clamp_(max=k)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(c[torch.randperm(n, generator=g, device=DEV)], 0, out=off[1:])
    return off


def _n_bins(case):
    return -(-case["genome"] // case["stride"])


def _inputs(case, seed, need_codes=False):
    """Genome (packed words on the host, codes where a step takes those), reads
    and random candidates (the read's own bin first)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + 17)
    codes = _genome(case, g)
    rd, z, lmax = _reads(case, codes, g)
    words = _pack(codes).cpu().numpy().view(np.uint32)
    host = codes.cpu().numpy() if need_codes else None
    del codes
    return g, words, host, rd, z, lmax


def _random_candidates(case, g, z):
    off = _offsets(case, g)
    n_pairs = int(off[-1])
    bins = torch.randint(0, _n_bins(case), (n_pairs,), generator=g, device=DEV, dtype=torch.int32)
    bins[off[:-1]] = (z // case["stride"]).int()
    return off, bins, n_pairs


def _index(case, words):
    return grim.grim_build_bins(words, case["q"], case["stride"], case["overlap"], packed=True,
                                ref_len=case["genome"])


def _filtered(case, seed, need_codes=False):
    g, words, host, rd, z, lmax = _inputs(case, seed, need_codes)
    off, bins, n_pairs = _random_candidates(case, g, z)
    idx = _index(case, words)
    batch = DeviceBatch(rd, off, bins, n_pairs, lmax)
    counts, bits = grim.alloc_outputs(n_pairs)
    ws = grim.alloc_workspace(idx, n_pairs)
    return dict(case=case, idx=idx, batch=batch, counts=counts, bits=bits, ws=ws), host


def _n_verify(case):
    return max(1, int(0.012 * case["reads"] * _mean_cand(case)))


def _room(case):
    """Room for a batch's seeded candidates: over twice what random sequence
    and the repeat families give on average."""
    k, lens = case["k"], _ints(case["lens"])
    seeds = sum(x // k for x in lens) / len(lens)
    copies = case["repeat"] * case["genome"] / 300 / 100 * 0.2
    return int(case["reads"] * seeds * (case["genome"] / 4 ** k + case["repeat"] * copies) * 2.5) + 400_000


def prepare(case, seed):
    kind = case["kind"]
    if kind == "filter":
        return _filtered(case, seed)[0]
    if kind in ("survivors", "verify"):
        st, host = _filtered(case, seed, need_codes=kind == "verify")
        grim.grim_filter_batch(st["idx"], st["batch"], st["counts"], st["bits"], st["ws"])
        if kind == "survivors":
            n = int(st["batch"].n_pairs * 0.05) + 4096   # a mapper's list buffers, kept
            st["out"] = (torch.zeros(n, dtype=torch.int64, device=DEV),
                         torch.zeros(n, dtype=torch.int32, device=DEV),
                         torch.zeros(n, dtype=torch.int32, device=DEV),
                         torch.zeros(1, dtype=torch.int64, device=DEV))
            st["cws"] = torch.empty(grim.grim_survivors_workspace_size(st["batch"].n_pairs),
                                    dtype=torch.uint8, device=DEV)
        else:
            _, sr, sb, n = grim.grim_compact_survivors(st["batch"], st["bits"])
            want = _n_verify(case)   # a list of the case's own length: its start again where short
            at = torch.arange(want, device=DEV) % max(1, n)
            st["surv"] = (sr[at].contiguous(), sb[at].contiguous(), want)
            st["idx"].attach_reference(host)
        return st
    if kind == "windows":
        g, words, _, rd, z, lmax = _inputs(case, seed)
        off = _offsets(case, g)
        half = (off[1:] - off[:-1]) // 2
        lo = (z // case["stride"] - half).clamp_(min=0) // case["grid"] * case["grid"]
        idx = _index(case, words)
        idx.transpose()
        n_pairs = int(off[-1])
        batch = DeviceBatch(rd, off, None, n_pairs, lmax)
        counts, bits = grim.alloc_outputs(n_pairs)
        st = dict(case=case, idx=idx, batch=batch, win_lo=lo.int(), counts=counts, bits=bits,
                  ws=torch.empty(256, dtype=torch.uint8, device=DEV), order=None)
        if case["ordered"]:
            st["order"] = torch.empty(batch.n_reads, dtype=torch.int32, device=DEV)
            st["ows"] = torch.empty(grim.grim_window_order_workspace_size(idx, batch.n_reads),
                                    dtype=torch.uint8, device=DEV)
        return st
    if kind in ("seed", "chain"):
        g, words, host, rd, z, lmax = _inputs(case, seed, need_codes=True)
        st = dict(case=case, si=grim.SeedIndex(host, case["k"]),
                  batch=DeviceBatch(rd, None, None, 0, lmax))
        zeros = lambda n, d=torch.int32: torch.zeros(n, dtype=d, device=DEV)  # noqa: E731
        room = _room(case)
        if kind == "seed":   # the mapper's own lists: a candidate list's buffer is the library's
            st["off"], st["bin"] = zeros(case["reads"] + 1, torch.int64), zeros(room)
        else:
            st["idx"] = _index(case, words)
            st["idx"].attach_reference(host)
            st["counts"], st["bits"] = zeros(room), zeros(room // 32 + 1)
            st["ws"] = grim.alloc_workspace(st["idx"], room)
            st["out"] = (zeros(room, torch.int64), zeros(room), zeros(room), zeros(1, torch.int64))
            st["dist"], st["ok"] = zeros(room), zeros(room // 32 + 1)
        return st
    if kind == "serve":
        st, _ = _filtered(case, seed)
        b = st["batch"]
        u = lambda t, d: t.cpu().numpy().view(d)  # noqa: E731
        hb = grim.HostBatch(None, u(b.read_off, np.uint64), u(b.read_len, np.uint32),
                            u(b.read_e, np.uint32), E_DEN, u(b.cand_off, np.uint64),
                            u(b.cand_bin, np.uint32), max_len=b.max_len,
                            words=u(b.words, np.uint32), pinned=True)
        idx = st["idx"]
        server = grim.Server(idx, hbm_budget_bytes=128 << 20, max_tick_pairs=2 << 20, max_len=256)
        return dict(case=case, idx=idx, hb=hb, server=server)
    raise ValueError(kind)


def run(st):
    kind = st["case"]["kind"]
    if kind == "filter":
        grim.grim_filter_batch(st["idx"], st["batch"], st["counts"], st["bits"], st["ws"])
        return {"counts": st["counts"], "bits": st["bits"]}
    if kind == "survivors":
        sp, sr, sb, n = grim.grim_compact_survivors(st["batch"], st["bits"], out=st["out"],
                                                    workspace=st["cws"], read_total=False)
        return {"pair": sp, "read": sr, "bin": sb, "n": n}
    if kind == "verify":
        sr, sb, n = st["surv"]
        dist, ok = grim.grim_verify_survivors(st["idx"], st["batch"], sr, sb, n)
        return {"dist": dist, "ok": ok}
    if kind == "windows":
        if st["order"] is not None:
            grim.grim_window_order(st["idx"], st["win_lo"], order=st["order"], workspace=st["ows"])
        grim.grim_filter_windows(st["idx"], st["batch"], st["win_lo"], st["counts"], st["bits"],
                                 st["ws"], order=st["order"])
        return {"counts": st["counts"], "bits": st["bits"]}
    if kind == "seed":
        c = grim.grim_seed_candidates(st["si"], st["batch"], st["case"]["stride"])
        off = torch.as_tensor(DeviceArray(c.cand_off_ptr, c.n_reads + 1, "<i8", c), device=DEV)
        bins = torch.as_tensor(DeviceArray(c.cand_bin_ptr, c.n_pairs, "<i4", c), device=DEV)
        st["off"].copy_(off)
        st["bin"][:c.n_pairs].copy_(bins)
        return {"off": st["off"], "bin": st["bin"]}
    if kind == "chain":
        idx = st["idx"]
        c = grim.grim_seed_candidates(st["si"], st["batch"], st["case"]["stride"])
        if c.n_pairs > st["counts"].numel():
            raise RuntimeError("more candidates than the buffers hold")
        b = _with_candidates(st["batch"], c)
        grim.grim_filter_batch(idx, b, st["counts"], st["bits"], st["ws"])
        sp, sr, sb, n = grim.grim_compact_survivors(b, st["bits"], out=st["out"])
        dist, ok = grim.grim_verify_survivors(idx, b, sr, sb, n)
        st["dist"][:n].copy_(dist)
        st["ok"][:ok.numel()].copy_(ok)
        return {"counts": st["counts"], "bits": st["bits"], "pair": st["out"][0],
                "read": st["out"][1], "bin": st["out"][2], "dist": st["dist"], "ok": st["ok"]}
    t = st["server"].submit_inplace(st["hb"])
    rc, counts, bits, _ = st["server"].wait(t)
    if rc != grim.GRIM_OK:
        raise grim.GrimError(rc, "served request")
    return {"counts": counts, "bits": bits}


def _with_candidates(batch, c):
    b = DeviceBatch((batch.words, batch.read_off, batch.read_len, batch.read_e), None, None,
                    c.n_pairs, batch.max_len)
    b.cands = c
    b.c.cand_off, b.c.cand_bin = c.cand_off_ptr, c.cand_bin_ptr
    return b


# ------------------------------------------------------------------------ work
def work(case):
    """Bytes of a pass: each input once, each output once.  A bin vector that
    several pairs name counts once (an index is read whole at most)."""
    n, kind, vb = case["reads"], case["kind"], 4 ** case["q"] // 8
    lens = _ints(case["lens"])
    mean_len = sum(lens) / len(lens)
    read_bytes = n * (mean_len / 4 + 8 + 4 + 4 + 8)
    pairs = n * _mean_cand(case)
    index = _n_bins(case) * vb
    vectors = min(index, pairs * vb)
    span = (case["stride"] + case["overlap"]) / 4
    if kind in ("filter", "serve"):
        b = read_bytes + vectors + pairs * (4 + 4 + 1 / 8)
    elif kind == "survivors":
        s = 0.015 * pairs
        b = pairs / 8 + n * 8 + s * (4 + 16)
    elif kind == "verify":
        s = _n_verify(case)
        b = read_bytes + min(case["genome"] / 4, s * span) + s * (8 + 4 + 1 / 8)
    elif kind == "windows":
        b = read_bytes + 4 * n + vectors + pairs * (4 + 1 / 8)
    else:
        k = case["k"]
        seeds = n * sum(x // k for x in lens) / len(lens)
        hits = seeds * case["genome"] / 4 ** k
        # a seed's two offsets, every hit's position, every candidate written
        b = read_bytes + seeds * 16 + hits * 4 + hits * 4 + n * 8
        if kind == "chain":
            b += min(index, hits * vb) + hits * (4 + 4 + 1 / 8 + 1 / 8)
    return {"bytes": float(b), "flops": 0.0}


# ----------------------------------------------------------------------- exact
def exact(case, seed):
    """Counts and pass bits of the filter forms from a dense table of which
    token occurs in which bin; None where that table or the pairs are many."""
    kind, q = case["kind"], case["q"]
    pairs = case["reads"] * _mean_cand(case)
    lens = _ints(case["lens"])
    if kind not in ("filter", "windows", "serve") or _n_bins(case) * 4 ** q > 4e9 or \
            pairs * sum(lens) / len(lens) > 2e10:
        return None
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + 17)
    codes = _genome(case, g)
    (words, roff, L, e), z, lmax = _reads(case, codes, g)
    B, O, G, nb = case["stride"], case["overlap"], case["genome"], _n_bins(case)

    def tokens(c):
        t = torch.zeros(c.numel() - q + 1, dtype=torch.int32, device=DEV)
        for j in range(q):
            t = t * 4 + c[j:c.numel() - q + 1 + j].int()
        return t

    tok = tokens(codes)
    table = torch.zeros(nb, 4 ** q, dtype=torch.bool, device=DEV)
    p = torch.arange(tok.numel(), device=DEV)
    # start p lies in bin b when b * B <= p and p + q <= min(G, (b + 1) * B + O)
    for back in range((O + B - 1) // B + 1):
        b = p // B - back
        ok = (b >= 0) & (p + q <= (b + 1) * B + O)
        table[b[ok], tok[ok].long()] = True
    rc = torch.stack([(words >> (30 - 2 * j)) & 3 for j in range(16)], 1).reshape(-1)
    rtok = tokens(rc)
    if kind == "windows":
        off = _offsets(case, g)
        half = (off[1:] - off[:-1]) // 2
        lo = (z // B - half).clamp_(min=0) // case["grid"] * case["grid"]
        n_pairs = int(off[-1])
        rd = torch.repeat_interleave(torch.arange(case["reads"], device=DEV), off[1:] - off[:-1])
        bins = lo[rd] + torch.arange(n_pairs, device=DEV) - off[rd]
    else:
        off, bins, n_pairs = _random_candidates(case, g, z)
        rd = torch.repeat_interleave(torch.arange(case["reads"], device=DEV), off[1:] - off[:-1])
        bins = bins.long()
    counts = torch.empty(n_pairs, dtype=torch.int32, device=DEV)
    i = torch.arange(lmax - q + 1, device=DEV)
    L, e = L.long(), e.long()
    need = (L - q + 1).clamp(min=0) - q * ((e * L + E_DEN - 1) // E_DEN)
    for a in range(0, n_pairs, 1 << 19):
        r, b = rd[a:a + (1 << 19)], bins[a:a + (1 << 19)]
        inside = b < nb
        at = (roff[r, None] + i).clamp_(max=rtok.numel() - 1)
        seen = table[b.clamp(max=nb - 1)[:, None], rtok[at].long()] & (i < (L[r] - q + 1)[:, None])
        counts[a:a + r.numel()] = torch.where(inside, seen.sum(1), -1).int()
    ok = (counts >= need[rd]) & (bins < nb)
    ok = torch.cat([ok, ok.new_zeros(-n_pairs % 32)]).view(-1, 32).long()
    word = (ok << torch.arange(32, device=DEV)).sum(1)
    bits = torch.where(word >= 2 ** 31, word - 2 ** 32, word).int()
    if kind == "serve":
        return {"counts": counts.cpu().numpy(), "bits": bits.cpu().numpy().view(np.uint32)}
    return {"counts": counts, "bits": bits}
