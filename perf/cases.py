"""The work that users of the classifier have it do, as cases that can be timed.

listed() holds one case for each way the library is used, from a handful of reads on a
small database to ten million on a large one; draw() gives more cases of the same ranges.
Databases and reads follow the workloads of the synth module (bacterial-size random genomes,
near-identical strains, short reads with a sequencing error model, a share of long reads),
drawn on the GPU so that the large ones take seconds.

Keys of a case:
  kind        classify, pairs, contain, abundance, index or serve
  db          random (n_genomes x genome_len, a GC content of its own each) or strains
              (n_genomes genomes in families of `family`, 1-5% apart)
  n_reads, len_lo, len_hi    short reads, lengths uniform in [len_lo, len_hi]
  n_long      reads of 1,000 to 10,000 bases among them, at 2% substitutions and 3% indels
  p_n         share of read bases that are N
  k, w, min_hits, top_n, E, permille   the query; permille = 1: E permille of the length
  mode        per_stage, fused or graph;  filter, strands   as in the query
  host        results are taken to the host, as by a program that prints them
  requests    serve: requests in flight, their sizes spread evenly up to n_reads
"""
import ctypes as C
import math

import numpy as np
import torch

import paper_2311_02029_amd as mt

MODES = {"per_stage": mt.MT_MODE_PER_STAGE, "fused": mt.MT_MODE_FUSED, "graph": mt.MT_MODE_FUSED_GRAPH}
FILTERS = {"obstacle": mt.MT_FILTER_OBSTACLE, "hamming": mt.MT_FILTER_HAMMING, "base_count": mt.MT_FILTER_BASE_COUNT,
           "qgram": mt.MT_FILTER_QGRAM, "shd": mt.MT_FILTER_SHD}
DEFAULTS = dict(kind="classify", db="random", n_genomes=200, genome_len=2_500_000, family=1, n_reads=1_000_000,
                len_lo=150, len_hi=150, n_long=0, p_n=0.0, k=21, w=11, min_hits=3, top_n=3, E=7, permille=0,
                mode="fused", filter="obstacle", strands=1, host=0, requests=0)
MAX_REQUESTS = 5  # a served result is 12 arrays


def _case(**kw):
    return dict(DEFAULTS, **kw)


def listed():
    small = dict(n_genomes=10, genome_len=100_000, k=15, w=10)
    strains = dict(db="strains", n_genomes=2000, genome_len=2_000_000, family=5)
    return [
        # a few reads against a small database, read back at once: launches and latency
        _case(name="classify_16_reads", n_reads=16, host=1, **small),
        # the usual first run: ten thousand reads of 150 bp on 1 Mbp, read back
        _case(name="classify_10k_reads", n_reads=10_000, host=1, p_n=0.001, **small),
        # a sequencing batch: a million reads of 150 bp on a 500 Mbp database
        _case(name="classify_1m_reads"),
        # the largest batch: ten million reads on 4 Gbp of near-identical strains (the headline benchmark)
        _case(name="classify_strains_10m", n_reads=10_000_000, **strains),
        # mixed read lengths, 5% of them long reads whose E grows with the length (the uneven workload)
        _case(name="classify_uneven_2m", n_reads=1_900_000, len_lo=75, len_hi=300, n_long=100_000, E=50, permille=1),
        # reads of unknown orientation: both strands of every genome
        _case(name="classify_strands", strands=2),
        # another of the five filters, in the per-stage form that all of them run in: 100 bp reads, SHD, E = 5%
        _case(name="classify_shd", n_reads=250_000, len_lo=100, len_hi=100, mode="per_stage", filter="shd", E=5),
        # the filter alone on (read, location) pairs from elsewhere, half of them wrong locations
        _case(name="filter_pairs", kind="pairs", n_reads=500_000, E=7),
        # stage 1: which genomes of the database does a sample hold (hit counts, then the subset)
        _case(name="containment", kind="contain"),
        # stage 3: relative abundances from a classification, 2,000 strains
        _case(name="abundance", kind="abundance", n_reads=1_000_000, db="strains", n_genomes=2000, genome_len=100_000,
              family=5),
        # the database is loaded: the seed index over 500 Mbp, and the first reads classified with it
        _case(name="index_500mbp", kind="index", n_reads=20_000),
        # a service: five requests in flight, up to fifty thousand reads each, from host memory and back to it
        _case(name="serve_5_requests", kind="serve", n_reads=50_000, len_lo=100, len_hi=250, E=50, permille=1,
              requests=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the whole range, odd ones among them."""
    kind = rng.choice(["classify", "classify", "classify", "classify", "pairs", "contain", "abundance", "index", "serve"])
    c = _case(kind=kind)
    if rng.random() < 0.4:
        c["db"], c["family"] = "strains", rng.choice([2, 3, 5, 8, 20])
    c["n_genomes"] = _log_int(rng, 1, 200) * c["family"] if c["family"] > 1 else _log_int(rng, 2, 1000)
    c["genome_len"] = max(1000, min(_log_int(rng, 20_000, 5_000_000), 500_000_000 // c["n_genomes"]))
    c["k"], c["w"] = rng.choice([(21, 11), (21, 11), (15, 10), (17, 8), (28, 18), (31, 16)])
    if c["k"] == 15 and c["n_genomes"] * c["genome_len"] > 50_000_000:
        c["k"], c["w"] = 21, 11
    c["n_reads"] = _log_int(rng, 1, 2_000_000)
    lens = rng.choice(["one", "one", "range"])
    c["len_lo"] = rng.randint(50, 300)
    c["len_hi"] = c["len_lo"] if lens == "one" else rng.randint(c["len_lo"], 300)
    c["p_n"] = rng.choice([0.0, 0.0, 0.001, 0.01])
    c["E"], c["permille"] = rng.choice([(0, 0), (3, 0), (7, 0), (7, 0), (15, 0), (50, 1), (50, 1), (100, 1)])
    c["top_n"] = rng.choice([1, 3, 3, 3, 5, 0])
    c["min_hits"] = rng.choice([1, 2, 3, 3, 3]) if c["top_n"] else 3
    c["host"] = int(c["n_reads"] <= 20_000)
    if kind == "classify":
        c["mode"] = rng.choice(["fused", "fused", "fused", "graph", "per_stage"])
        c["strands"] = rng.choice([1, 1, 2])
        if rng.random() < 0.25:
            c["filter"], c["mode"] = rng.choice(["hamming", "base_count", "qgram", "shd"]), "per_stage"
        if rng.random() < 0.25 and c["filter"] == "obstacle":
            c["n_long"] = min(20_000, c["n_reads"] // rng.choice([3, 10, 20]) + 1)
            c["E"], c["permille"], c["top_n"] = 50, 1, rng.choice([1, 3])
    elif kind == "pairs":
        c["filter"] = rng.choice(["obstacle", "obstacle", "hamming", "base_count", "qgram", "shd"])
    elif kind == "index":
        c["n_reads"], c["host"] = min(c["n_reads"], 20_000), 0
    elif kind == "serve":
        c["n_reads"], c["requests"], c["host"] = min(c["n_reads"], 50_000), rng.randint(1, MAX_REQUESTS), 0
    return c


# ------------------------------------------------------------------ inputs --

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)


def _to_ascii(codes):
    """A, C, G, T of the codes 0 to 3."""
    return codes * 2 + (codes >= 2).to(torch.uint8) * 2 + (codes == 3).to(torch.uint8) * 11 + 65


def _genomes(case, g):
    """The database as codes 0..3 (uint8, back to back) with per-genome GC content, or in families of strains."""
    n, length, fam = case["n_genomes"], case["genome_len"], case["family"]
    codes = torch.empty(n * length, dtype=torch.uint8, device="cuda")
    per = max(1, (1 << 27) // length)  # genomes at a time
    if case["db"] == "random":
        gc = torch.rand(n, generator=g, device="cuda") * 0.4 + 0.3
        for a in range(0, n, per):
            b = min(n, a + per)
            u = torch.rand((b - a, length), generator=g, device="cuda")
            x = gc[a:b, None]
            out = (u >= (1 - x) / 2).to(torch.uint8) + (u >= 0.5).to(torch.uint8) + (u >= (1 + x) / 2).to(torch.uint8)
            codes[a * length:b * length] = out.view(-1)
        return codes
    for f in range(0, n, fam):
        root = torch.randint(0, 4, (length,), generator=g, device="cuda", dtype=torch.uint8)
        for a in range(f, min(n, f + fam), per):
            b = min(n, f + fam, a + per)
            p = torch.rand((b - a, 1), generator=g, device="cuda") * 0.04 + 0.01
            hit = torch.rand((b - a, length), generator=g, device="cuda") < p
            other = torch.randint(1, 4, (b - a, length), generator=g, device="cuda", dtype=torch.uint8)
            codes[a * length:b * length] = ((root + other * hit) & 3).view(-1)
    return codes


def _database(codes, case):
    """The database as the library takes it: ASCII bytes and offsets on the device."""
    n, length = case["n_genomes"], case["genome_len"]
    seq = torch.empty_like(codes)
    for a in range(0, len(codes), 1 << 28):
        seq[a:a + (1 << 28)] = _to_ascii(codes[a:a + (1 << 28)])
    offs = torch.arange(n + 1, device="cuda", dtype=torch.int64) * length
    return mt.DeviceSeqs(seq, offs, n, n * length)


def _lengths(case, g):
    n, nl = case["n_reads"], case["n_long"]
    lens = torch.randint(case["len_lo"], case["len_hi"] + 1, (n,), generator=g, device="cuda")
    if nl:
        lens = torch.cat([lens, torch.randint(1000, 10_001, (nl,), generator=g, device="cuda")])
        lens = lens[torch.randperm(n + nl, generator=g, device="cuda")]
    return lens.clamp(max=int(case["genome_len"] * 0.9))


def _reads(codes, case, lens, g, flip):
    """Reads of the given lengths: a uniform genome and start, and per base an insertion, a
    deletion before it, a substitution or a copy.  Returns the reads and their (genome, start)."""
    n, length = len(lens), case["genome_len"]
    offs = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=offs[1:])
    total = int(offs[-1])
    seq = torch.empty(max(total, 1), dtype=torch.uint8, device="cuda")
    is_long = lens >= 1000
    p_sub = torch.rand(n, generator=g, device="cuda") * 0.009 + 0.001
    p_indel = torch.rand(n, generator=g, device="cuda") * 0.0009 + 0.0001
    p_sub, p_indel = torch.where(is_long, 0.02, p_sub), torch.where(is_long, 0.03, p_indel)
    genome = torch.randint(0, case["n_genomes"], (n,), generator=g, device="cuda")
    where = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    start = torch.empty(n, dtype=torch.int64, device="cuda")
    ends = offs.cpu().numpy()
    a = 0
    while a < n:
        b = max(a + 1, int(np.searchsorted(ends, ends[a] + (1 << 26), side="right")) - 1)
        o, m = offs[a:b] - offs[a], lens[a:b]
        rd = torch.repeat_interleave(torch.arange(b - a, device="cuda"), m)
        u = torch.rand(len(rd), generator=g, device="cuda")
        pi = p_indel[a:b][rd] * 0.5
        ins, dele = u < pi, (u >= pi) & (u < 2 * pi)
        sub = (u >= 2 * pi) & (u < 2 * pi + p_sub[a:b][rd])
        step = 1 + dele.to(torch.int32) - ins.to(torch.int32)  # reference bases up to and with this one
        cum = torch.cumsum(step, 0, dtype=torch.int64)
        before = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), cum])
        span = before[o + m] - before[o] + 1
        st = (where[a:b] * (length - span + 1).clamp(min=1)).to(torch.int64)
        start[a:b] = st
        pos = (genome[a:b] * length + st - before[o])[rd] + cum - 1
        base = codes[pos.clamp_(0, len(codes) - 1)]
        other = torch.randint(1, 4, (len(rd),), generator=g, device="cuda", dtype=torch.uint8)
        base = torch.where(ins, other, (base + other * sub) & 3)
        if flip:  # every other read, on average, from the other strand
            fl = (torch.rand(b - a, generator=g, device="cuda") < 0.5)[rd]
            at = torch.arange(len(rd), device="cuda")
            base = torch.where(fl, 3 - base[torch.where(fl, (2 * o + m - 1)[rd] - at, at)], base)
        text = _to_ascii(base)
        if case["p_n"]:
            text[torch.rand(len(rd), generator=g, device="cuda") < case["p_n"]] = ord("N")
        seq[ends[a]:ends[b]] = text
        a = b
    return mt.DeviceSeqs(seq, offs, n, total), genome, start


class _HostReads:
    """A sequence set in host memory, as a service receives it."""

    def __init__(self, seq, offsets):
        self.seq, self.offsets = seq, offsets


def prepare(case, seed):
    g = _generator(seed)
    codes = _genomes(case, g)
    db = _database(codes, case)
    st = {"case": case, "query": dict(min_hits=case["min_hits"], top_n=case["top_n"], e_value=case["E"],
                                      e_mode=mt.MT_E_CEIL_PERMILLE if case["permille"] else mt.MT_E_FIXED)}
    if case["kind"] == "serve":
        st["requests"] = []
        for i in range(case["requests"]):
            n = max(1, case["n_reads"] * (i + 1) // case["requests"])
            m = case["len_lo"] + (case["len_hi"] - case["len_lo"]) * i // max(1, case["requests"] - 1)
            lens = torch.full((n,), min(m, int(case["genome_len"] * 0.9)), device="cuda", dtype=torch.int64)
            r = _reads(codes, case, lens, g, False)[0]
            st["requests"].append(_HostReads(r.seq.cpu().numpy(), r.offsets.cpu().numpy().view(np.uint64)))
        st["index"] = mt.Index(db, case["k"], case["w"])
        st["server"] = mt.Server(st["index"])
        st["room"] = [_room(case, len(r.offsets) - 1, True) for r in st["requests"]]
        return st
    st["reads"], genome, start = _reads(codes, case, _lengths(case, g), g, case["strands"] == 2)
    if case["kind"] == "index":
        st["db"], st["room"] = db, _room(case, case["n_reads"], True)
        return st
    st["index"] = mt.Index(db, case["k"], case["w"])
    if case["kind"] == "classify":
        st["room"] = _room(case, st["reads"].n, case["host"])
    elif case["kind"] == "contain":
        st["room"] = torch.full((case["n_genomes"],), -1, dtype=torch.int32, device="cuda")
    elif case["kind"] == "pairs":
        # each read with where it comes from, some indels off, and with a place that it does not come from
        n = len(genome)
        off = torch.randint(-2, 3, (n,), generator=g, device="cuda")
        wrong = torch.randint(0, case["n_genomes"], (n,), generator=g, device="cuda")
        at = torch.randint(0, case["genome_len"], (n,), generator=g, device="cuda")
        lens = torch.diff(st["reads"].offsets)
        E = (lens * case["E"] + 999) // 1000 if case["permille"] else torch.full_like(lens, case["E"])
        st["pairs"] = dict(
            pair_read=torch.arange(n, device="cuda", dtype=torch.int32).repeat_interleave(2),
            pair_genome=torch.stack([genome, wrong], 1).view(-1).to(torch.int32),
            pair_diag=torch.stack([start + off, at], 1).view(-1).contiguous(),
            pair_E=E.repeat_interleave(2).to(torch.int16))
    elif case["kind"] == "abundance":
        st["result"] = st["index"].classify(st["reads"], mode=MODES["fused"], **st["query"])
    return st


# ------------------------------------------------------------------- a pass --

# A result's arrays with a length that the reads decide, and those of the database's or the read set's.
CANDS = {"genome": ("<i4", torch.int32), "diag": ("<i8", torch.int64), "hits": ("<i4", torch.int32),
         "approx": ("<i2", torch.int16), "accept": ("|u1", torch.uint8), "strand": ("|u1", torch.uint8)}


def _candidate_room(case, n):
    """More candidates than n reads of the case have."""
    return n * (case["top_n"] or 2 * case["family"] + 2) + 256


def _room(case, n, host):
    """The program's own arrays for the candidates of n reads, which outlive the result."""
    room = _candidate_room(case, n)
    if host:
        return {name: np.zeros(room, np.dtype(t)) for name, (t, _) in CANDS.items()}
    return {name: torch.zeros(room, dtype=t, device="cuda") for name, (_, t) in CANDS.items()
            if name != "strand" or case["strands"] == 2}


def _to_host(result, room):
    """Every output of a result on the host, the candidates in the program's arrays."""
    out = result.to_host()
    for name in CANDS:
        room[name][:len(out[name])] = out[name]
        out[name] = room[name]
    return out


class _DeviceArray:
    """A result's device array, without a copy; keeps the result alive."""

    def __init__(self, result, ptr, n, typestr):
        self.result = result
        self.__cuda_array_interface__ = dict(shape=(n,), typestr=typestr, data=(ptr, False), version=2, strides=None)


def _on_device(result, room):
    """Every output of a result as device tensors (unsigned arrays as the signed type of their
    width), the candidates in the program's arrays."""
    lib, h = result.lib, result.h
    n, nc, nt = C.c_uint64(), C.c_uint64(), C.c_uint32()
    p = [C.c_void_p() for _ in range(12)]
    refs = [C.byref(x) for x in p]
    lib.mt_result_reads(h, C.byref(n), *refs[:3])
    lib.mt_result_cands(h, C.byref(nc), *refs[3:8])
    lib.mt_result_strands(h, refs[8])
    lib.mt_result_taxa(h, C.byref(nt), *refs[9:])
    n, nc, nt = n.value, nc.value, nt.value
    fixed = (("cand_offsets", n + 1, "<i8", p[0]), ("read_accepted", n, "|u1", p[1]), ("read_E", n, "<i2", p[2]),
             ("unique", nt, "<i8", p[9]), ("multi", nt, "<i8", p[10]), ("unmapped", 1, "<i8", p[11]))
    out = {name: torch.as_tensor(_DeviceArray(result, x.value, count, t), device="cuda") for name, count, t, x in fixed}
    for x, name in zip(p[3:9], room):
        if nc:
            view = torch.as_tensor(_DeviceArray(result, x.value, nc, CANDS[name][0]), device="cuda")
            room[name][:nc].copy_(view)
        out[name] = room[name]
    return out


def run(state):
    case, q = state["case"], state["query"]
    kind = case["kind"]
    if kind == "classify":
        r = state["index"].classify(state["reads"], mode=MODES[case["mode"]], filter_kind=FILTERS[case["filter"]],
                                    strands=case["strands"], **q)
        return (_to_host if case["host"] else _on_device)(r, state["room"])
    if kind == "pairs":
        return state["index"].filter_pairs(state["reads"], **state["pairs"], kind=FILTERS[case["filter"]])
    if kind == "contain":
        hits = state["index"].containment(state["reads"])
        kept, most = mt.select_genomes(hits)
        state["room"][:len(kept)] = kept
        return hits, state["room"], len(kept), most
    if kind == "abundance":
        return state["index"].abundance(state["result"])
    if kind == "index":
        ix = mt.Index(state["db"], case["k"], case["w"])
        info = ix.info()
        first = _to_host(ix.classify(state["reads"], mode=MODES["fused"], **q), state["room"])
        return [info["n_minimizers"], info["n_keys"], info["n_multi_occ"], first]
    ids = [state["server"].submit(r, **q) for r in state["requests"]]
    return [_to_host(state["server"].wait(i), room) for i, room in zip(ids, state["room"])]


# --------------------------------------------------------------------- work --

def work(case):
    """Bytes: the reads once, a 16-byte index entry per seed, the reference of each pair once, and
    the outputs.  Operations: the obstacle rows of each pair (6 a mismatch word of 32 bits)."""
    c = case
    seeds = 2.0 / (c["w"] + 1)  # minimizers a base
    ref = c["n_genomes"] * c["genome_len"]
    long_bases = c["n_long"] * 5500.0
    if c["kind"] == "index":
        # the genomes read; bit planes and a table of two 16-byte slots a seed written
        return {"bytes": ref + ref * 0.375 + ref * seeds * 32, "flops": ref * 8.0}
    n = c["n_reads"]
    mean = (c["len_lo"] + c["len_hi"]) / 2
    if c["kind"] == "serve":
        n = n * (c["requests"] + 1) / 2
    elif c["kind"] == "abundance":
        pairs = n * min(c["family"], c["top_n"] or c["family"])
        return {"bytes": 8.0 * (n + 1) + 8.0 * pairs + 16.0 * c["n_genomes"], "flops": 4.0 * pairs}
    bases = (n * mean + long_bases) * c["strands"]
    if c["kind"] == "pairs":
        n_pairs, seeded = 2.0 * n, 0.0
    elif c["kind"] == "contain":
        n_pairs, seeded = 0.0, bases * seeds
    else:
        n_pairs = (n + c["n_long"]) * float(min(c["family"], c["top_n"] or c["family"]))
        seeded = bases * seeds
    E = mean * c["E"] / 1000 if c["permille"] else c["E"]
    E_long = 5500.0 * c["E"] / 1000 if c["permille"] else c["E"]
    share = n / max(1, n + c["n_long"])
    rows = share * (2 * E + 1) * mean / 32 + (1 - share) * (2 * E_long + 1) * 5500 / 32
    window = share * (mean + 2 * E) + (1 - share) * (5500 + 2 * E_long)
    bytes_ = bases / c["strands"] + 8.0 * n + 16.0 * seeded + n_pairs * (window / 4 + 19) + 11.0 * n
    return {"bytes": bytes_, "flops": 10.0 * bases * (c["kind"] != "pairs") + 6.0 * rows * n_pairs}


def exact(case, seed):
    """Every output is a whole number or a byte, compared as it is, but the abundances, which
    are quotients of two of the whole numbers returned beside them."""
    return None
