"""The workloads whose speed is tracked: k-mer counts as a program calls them.

A case is one call of a public entry point of ``paper_2407_07718_amd.kc``:

* ``device``  -- ``DeviceCounter.count``: reads resident in HBM, workspace and outputs kept;
* ``bounded`` -- the same under ``kc_config.hbm_budget`` (the count runs in rounds);
* ``ext``     -- ``DeviceExtCounter.count``: pairs and every occurrence (read, position);
* ``batch``   -- ``DeviceBatch``: many small read sets per launch, results fetched per set;
* ``host``    -- ``kc_count``: host arrays in, host arrays out.

Results sit at the front of buffers whose sizes depend on the case alone; the rest stays zero.

Reads are drawn on the GPU from the recipes of ``synth.py`` (uniform genome with repeat
families, both strands, substitutions, indels, a few N), by ``seed`` alone.
"""
import math

import numpy as np
import torch

from paper_2407_07718_amd import kc, synth

ALL = 1 << 20   # an upper frequency bound that keeps every k-mer


def listed():
    return [
        # one amplicon-sized sample of 150 bp reads (the smoke workload's sizes): launches and latency
        dict(name="tiny_k31", kind="device", reads="short", bases=300_000, length=150, genome=100_000, sub=0.01,
             k=31, m=15, lo=2, hi=50, hist=65536),
        # a small bacterial sample with trimmed reads of 35 to 151 bp, no round sizes anywhere
        dict(name="ragged_k21", kind="device", reads="ragged", bases=6_000_011, length=151, genome=1_234_567, sub=0.005,
             k=21, m=11, lo=2, hi=50, hist=1000),
        # the short-read benchmark workload: 1 M x 150 bp, 30x of a 5 Mbp genome with repeats
        dict(name="short_k31", kind="device", reads="short", bases=150_000_000, length=150, genome=5_000_000, sub=0.005,
             k=31, m=17, lo=2, hi=1000, hist=65536),
        # the long-read benchmark workload (the headline): 1 Gbp, 20x of a 50 Mbp genome
        dict(name="long_k31", kind="device", reads="long", bases=1_000_000_000, length=15_000, genome=50_000_000,
             sub=0.001, k=31, m=21, lo=2, hi=200, hist=65536),
        # 128-bit keys on long reads (assembly k)
        dict(name="long_k51", kind="device", reads="long", bases=400_000_000, length=15_000, genome=20_000_000, sub=0.001,
             k=51, m=21, lo=2, hi=200, hist=65536),
        # the whole spectrum at low coverage: every k-mer reported, most of them seen once
        dict(name="all_k21", kind="device", reads="short", bases=60_000_000, length=150, genome=20_000_000, sub=0.005,
             k=21, m=11, lo=1, hi=ALL, hist=4096),
        # occurrence lists for an overlapper: short reads, and long reads with 128-bit keys
        dict(name="ext_short_k31", kind="ext", reads="short", bases=45_000_000, length=150, genome=1_500_000, sub=0.005,
             k=31, m=17, lo=2, hi=1000, hist=65536),
        dict(name="ext_long_k51", kind="ext", reads="long", bases=30_000_000, length=15_000, genome=1_500_000, sub=0.001,
             k=51, m=21, lo=2, hi=200, hist=65536),
        # a count beside other work on the GPU: a fifth of the one-pass workspace
        dict(name="bounded_k31", kind="bounded", reads="long", bases=200_000_000, length=15_000, genome=10_000_000,
             sub=0.001, k=31, m=21, lo=2, hi=200, hist=65536, per_base=10),
        # 48 small samples in one launch, as a screening pipeline has them
        dict(name="batch_48", kind="batch", reads="short", bases=500_000, length=150, genome=20_000, sub=0.005, k=31,
             m=17, lo=2, hi=50, hist=1024, sets=48),
        # one call on host arrays: copies and allocations included
        dict(name="host_k31", kind="host", reads="short", bases=20_000_000, length=150, genome=1_000_000, sub=0.005,
             k=31, m=17, lo=2, hi=1000, hist=65536),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["device"] * 6 + ["ext", "ext", "bounded", "batch", "host"])
    reads = rng.choice(["short", "ragged", "long"])
    k = rng.choice([17, 21, 25, 27, 31, 31, 33, 41, 51, 63])
    top = {"device": 600e6 if k <= 31 else 300e6, "ext": 60e6 if k <= 31 else 25e6, "bounded": 150e6, "batch": 1.5e6,
           "host": 30e6}[kind]
    bases = _log(rng, {"bounded": 2e7, "batch": 5e4}.get(kind, 2e5), top)
    lo = rng.choice([1, 2, 2, 2])
    c = dict(kind=kind, reads=reads, bases=bases, length={"short": rng.choice([100, 150, 250]), "ragged": 151,
                                                          "long": rng.choice([3001, 15_000])}[reads],
             genome=max(20_000, int(bases / rng.uniform(3, 40))), sub=rng.choice([0.001, 0.005, 0.01]), k=k,
             m=min(21, (k + 1) // 2 | 1), lo=lo, hi=ALL if lo == 1 else rng.choice([50, 200, 1000]),
             hist=rng.choice([256, 1000, 65536]))
    if kind == "bounded":
        c["per_base"] = 10 if k <= 31 else 18
        c["lo"], c["hi"] = 2, 200
    if kind == "batch":
        c["sets"] = rng.randint(5, 48)
        c["hist"] = 1024
    return c


# ---------------------------------------------------------------------------- inputs
def _lengths(case, g):
    bases, length = case["bases"], case["length"]
    if case["reads"] == "short":
        return np.full(max(1, bases // length), length, dtype=np.int64)
    if case["reads"] == "ragged":
        lens = g.integers(35, length + 1, size=bases // 60 + 2)
    else:
        lens = synth.lognormal_lengths(g, bases, float(length), length / 3.0, 64, case["genome"])
    cut = int(np.searchsorted(np.cumsum(lens), bases))
    lens = lens[: cut + 1].astype(np.int64)
    lens[-1] -= max(0, int(lens.sum()) - bases)
    return lens


def _read_set(case, seed):
    """(reads uint8, offsets int64) on the GPU; about case["bases"] bases."""
    g = np.random.Generator(np.random.PCG64(seed))
    genome = synth.uniform_genome(g, case["genome"])
    if case["genome"] >= 1_000_000:
        synth.add_repeat_families(g, genome, families=max(4, case["genome"] // 250_000))
    lens = np.minimum(_lengths(case, g), case["genome"])
    dev = torch.device("cuda")
    tg = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 1)
    genome = torch.from_numpy(genome).to(dev)
    ascii4 = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device=dev)
    indel = 0.0005 if case["reads"] == "long" else 0.0
    ends = np.cumsum(lens)
    pieces, kept = [], []
    i = 0
    while i < len(lens):   # about 2^26 bases at a time
        j = max(i + 1, int(np.searchsorted(ends, (ends[i - 1] if i else 0) + (1 << 26))))
        ln = torch.from_numpy(lens[i:j]).to(dev)
        n = int(lens[i:j].sum())
        start = (torch.rand(j - i, generator=tg, device=dev, dtype=torch.float64) * (case["genome"] - ln + 1)).long()
        rev = torch.rand(j - i, generator=tg, device=dev) < 0.5
        rid = torch.repeat_interleave(torch.arange(j - i, device=dev), ln, output_size=n)
        at = torch.arange(n, device=dev) - (torch.cumsum(ln, 0) - ln)[rid]
        back = rev[rid]
        at = torch.where(back, start[rid] + ln[rid] - 1 - at, start[rid] + at)
        seq = genome[at]
        seq = torch.where(back, 3 - seq, seq)
        hit = torch.rand(n, generator=tg, device=dev) < case["sub"]
        seq = torch.where(hit, (seq + torch.randint(1, 4, (n,), generator=tg, device=dev, dtype=torch.uint8)) & 3, seq)
        out = ascii4[seq.int()]
        out[torch.rand(n, generator=tg, device=dev) < 2e-5] = ord("N")
        if indel:   # half of the hits double a base, half drop it
            u = torch.rand(n, generator=tg, device=dev)
            rep = 1 + (u < indel / 2).long() - ((u >= indel / 2) & (u < indel)).long()
            out = torch.repeat_interleave(out, rep)
            ln = torch.zeros_like(ln).index_add_(0, rid, rep)
        pieces.append(out)
        kept.append(ln)
        i = j
    offsets = torch.zeros(len(lens) + 1, dtype=torch.int64, device=dev)
    torch.cumsum(torch.cat(kept), 0, out=offsets[1:])
    return torch.cat(pieces), offsets


def _set_case(case, i):
    """The i-th read set of a batch: sizes from a quarter to twice the case's."""
    f = 0.25 * 8.0 ** ((i * 0.6180339887498949) % 1.0)
    return dict(case, bases=int(case["bases"] * f), genome=max(5_000, int(case["genome"] * f)))


def _pairs(case):
    """Expected number of reported k-mers: the genome's, and errors made alike in lo reads."""
    n, g, k = case["bases"], case["genome"], case["k"]
    depth, e = n / g, n / g * case["sub"] / 3
    if case["lo"] == 1:
        return g * (1 - math.exp(-depth)) + 3 * k * g * (1 - math.exp(-e))
    return g * (1 - math.exp(-depth) * (1 + depth)) + 3 * k * g * (1 - math.exp(-e) * (1 + e))


def _caps(case):
    """Pairs and occurrences that a result has room for."""
    if case["kind"] == "batch":
        return sum(_caps(dict(_set_case(case, i), kind="host"))[0] for i in range(case["sets"])), 0
    top = case["bases"] + case["bases"] // 100 + 1000
    return min(top // case["lo"], int(1.3 * _pairs(case)) + 20_000), top


def prepare(case, seed):
    k, m, lo, hi, hist = (case[x] for x in ("k", "m", "lo", "hi", "hist"))
    pairs, occ = _caps(case)
    state = dict(case=case)
    if case["kind"] in ("batch", "host"):
        state.update(kmers=np.zeros((pairs, 1 if k <= 31 else 2), np.int64), counts=np.zeros(pairs, np.int32))
    if case["kind"] == "batch":
        sets = [_read_set(_set_case(case, i), seed * 1009 + i) for i in range(case["sets"])]
        torch.cuda.synchronize()
        state.update(sets=sets, plan=kc.DeviceBatch([(r, o, k, m, lo, hi, hist) for r, o in sets]))
        return state
    reads, offsets = _read_set(case, seed)
    n, n_reads = int(reads.numel()), int(offsets.numel()) - 1
    if case["kind"] == "host":
        state.update(reads=reads.cpu().numpy(), offsets=offsets.cpu().numpy().view(np.uint64))
        return state
    if case["kind"] == "ext":
        plan = kc.DeviceExtCounter(n, n_reads, k, lo, hi, hist, pair_capacity=pairs, occ_capacity=occ)
        for t in (plan.occ_off, plan.occ_read, plan.occ_pos):
            t.zero_()
    else:
        cfg = kc.make_config(hbm_budget=n * case["per_base"]) if case["kind"] == "bounded" else None
        plan = kc.DeviceCounter(n, n_reads, k, m, lo, hi, hist, cfg, pair_capacity=pairs)
    plan.kmers.zero_()
    plan.counts.zero_()
    state.update(reads=reads, offsets=offsets, plan=plan)
    return state


def _totals(t):
    return np.array([t["n_pairs"], t["n_windows"], t["n_distinct"], t["overflow_sum"], t["max_count"]], dtype=np.int64)


def run(state):
    case = state["case"]
    if case["kind"] in ("batch", "host"):
        if case["kind"] == "host":
            res = [kc.kc_count(state["reads"], state["offsets"], case["k"], case["m"], case["lo"], case["hi"], case["hist"])]
        else:
            state["plan"].run()
            res = [state["plan"].result(i) for i in range(case["sets"])]
        at = 0
        for r in res:
            state["kmers"][at:at + r.n_pairs] = r.kmers.view(np.int64)
            state["counts"][at:at + r.n_pairs] = r.counts.view(np.int32)
            at += r.n_pairs
        return dict(kmers=state["kmers"], counts=state["counts"], hist=np.stack([r.hist for r in res]).view(np.int64),
                    totals=np.stack([_totals(r.totals) for r in res]))
    plan = state["plan"]
    t = plan.count(state["reads"], state["offsets"])
    out = dict(kmers=plan.kmers, counts=plan.counts, hist=plan.hist, totals=_totals(t))
    if case["kind"] == "ext":
        out.update(occ_off=plan.occ_off, occ_read=plan.occ_read, occ_pos=plan.occ_pos)
    return out


def work(case):
    """Bytes of the reads and of the result: each read once, each pair (and occurrence) written once."""
    def of(c):
        n, k, pairs = c["bases"], c["k"], _pairs(c)
        windows = n * max(0.0, 1 - (k - 1) / c["length"])
        b = n + 8 * (n / c["length"] + 1) + pairs * (12 if k <= 31 else 20) + 8 * c["hist"]
        if c["kind"] == "ext":
            b += 8 * pairs + 8 * windows * (1.0 if c["lo"] == 1 else max(0.0, 1 - c["sub"] * k))
        return b
    sets = [_set_case(case, i) for i in range(case["sets"])] if case["kind"] == "batch" else [case]
    return {"bytes": float(sum(of(c) for c in sets)), "flops": 0.0}


# ---------------------------------------------------------------------------- the definition
def _windows(codes, a):
    """Values of the windows of `a` bases, first base most significant, and of their complements read
    backwards (64 bits; a <= 32)."""
    n = codes.numel()
    if a == 0:
        z = torch.zeros_like(codes)
        return z, z
    if a == 1:
        return codes, 3 - codes
    h = a // 2
    f, r = _windows(codes, h)
    if a % 2 == 0:
        f2, r2 = f[h:], r[h:]
    else:
        f2, r2 = _windows(codes, h + 1)
        f2, r2 = f2[h:], r2[h:]
    w = n - a + 1
    return (f[:w] << (2 * (a - h))) | f2[:w], (r2[:w] << (2 * h)) | r[:w]


def _count(case, reads, offsets):
    k, lo, hi, hist = case["k"], case["lo"], case["hi"], case["hist"]
    dev, n = reads.device, int(reads.numel())
    up = reads & 0xDF
    bad = ~((up == 65) | (up == 67) | (up == 71) | (up == 84))
    codes = (((up >> 1) ^ (up >> 2)) & 3).long()
    lens = offsets[1:] - offsets[:-1]
    rid = torch.repeat_interleave(torch.arange(lens.numel(), device=dev), lens, output_size=n)
    nbad = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(bad.long(), 0)])
    w = n - k + 1
    pos = torch.nonzero((rid[:w] == rid[k - 1:]) & (nbad[:w] == nbad[k:])).flatten()
    sign = -(1 << 63)
    if k <= 31:
        f, r = _windows(codes, k)
        words = [torch.minimum(f, r)[pos]]
    else:
        h = k - 32
        fh, rh = _windows(codes, h)
        fl, rl = _windows(codes, 32)
        fl, rl, fh, rh = fl[h:][:w][pos], rl[:w][pos], fh[:w][pos], rh[32:][:w][pos]
        less = (fh < rh) | ((fh == rh) & ((fl ^ sign) < (rl ^ sign)))
        words = [torch.where(less, fl, rl), torch.where(less, fh, rh)]
    order = None
    for i, x in enumerate(words):   # least significant word first, each pass stable
        y = (x ^ sign) if len(words) == 2 and i == 0 else x
        o = torch.sort(y if order is None else y[order], stable=True)[1]
        order = o if order is None else order[o]
    words, pos = [x[order] for x in words], pos[order]
    head = torch.ones(pos.numel(), dtype=torch.bool, device=dev)
    head[1:] = (words[0][1:] != words[0][:-1]) if len(words) == 1 else \
        ((words[0][1:] != words[0][:-1]) | (words[1][1:] != words[1][:-1]))
    first = torch.nonzero(head).flatten()
    cnt = torch.diff(first, append=torch.tensor([pos.numel()], device=dev))
    keep = (cnt >= lo) & (cnt <= hi)
    over = cnt[cnt >= hist - 1]
    out = dict(kmers=torch.stack([x[first[keep]] for x in words], 1), counts=cnt[keep].int(),
               hist=torch.bincount(cnt.clamp(max=hist - 1), minlength=hist),
               totals=[int(keep.sum()), int(pos.numel()), int(first.numel()), int(over.sum()),
                       int(cnt.max()) if cnt.numel() else 0])
    if case["kind"] == "ext":
        c = cnt[keep]
        off = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(c, 0)])
        p = pos[torch.repeat_interleave(keep, cnt)]
        out.update(occ_off=off, occ_read=rid[p].int(), occ_pos=(p - offsets[rid[p]]).int())
    return out


def exact(case, seed):
    """The result by the definition, in plain torch (None where that takes too long)."""
    if case["bases"] > 200_000_000:
        return None
    many = case["kind"] in ("batch", "host")
    sets = [(_set_case(case, i), seed * 1009 + i) for i in range(case["sets"])] if case["kind"] == "batch" else [(case, seed)]
    res = [_count(c, *_read_set(c, s)) for c, s in sets]
    pairs, occ = _caps(case)

    def room(name, n):
        x = torch.cat([r[name] for r in res])
        return torch.cat([x, x.new_zeros((n - x.shape[0],) + x.shape[1:])])

    out = dict(kmers=room("kmers", pairs), counts=room("counts", pairs),
               hist=torch.stack([r["hist"] for r in res]) if many else res[0]["hist"],
               totals=torch.tensor([r["totals"] for r in res] if many else res[0]["totals"]))
    if case["kind"] == "ext":
        out.update(occ_off=room("occ_off", pairs + 1), occ_read=room("occ_read", occ), occ_pos=room("occ_pos", occ))
    return out
