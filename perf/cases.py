"""The workloads that this library's speed is judged on.

Each case is one whole call a user's program makes through the public entry
points, with the plan, context, server or batch that such a program keeps made
beforehand.  The families and their ranges:

  one     one pattern over a text in device memory (``Plan.count`` and
          ``Plan.collect`` into buffers the program keeps), from a
          few KiB, where launches and the total's readback are all there is,
          to several GiB, where the text's read is; both hash modes, DNA,
          letter and byte alphabets, patterns of 4 to 64 bytes
  many    a pattern set over word text (same calls): hits are dense, the
          table test, the verification and the sort by pattern count; both
          modes, fixed and mixed pattern lengths
  dict    a dictionary of thousands of patterns over word text: more ids than
          one sort pass covers
  call    the one-line ``search(text, patterns)``, which builds and drops its
          plan inside the call
  batch   uneven independent instances in one ``BatchPlan``
  serve   requests merged by a ``Server`` over resident corpora, results
          fetched to the host
  host    a text in pageable host memory through ``Plan.search_host``
  paper   the one-thread-per-offset procedure and its positions

Texts are drawn on the device from the seed alone.  Positions are left in a
buffer of a fixed size that the program keeps, so that its unused end is as
``prepare`` made it.
"""
import math
import os

import numpy as np
import torch

import paper_1810_01051_amd as rk

DEV = "cuda:0"
TUNED = os.path.join(os.path.dirname(os.path.abspath(rk.__file__)), "autotune_gfx950.json")
TPB = (32, 64, 128, 256, 512, 1024)
MIB = 1 << 20
CHUNK = 1 << 26


def listed():
    return [
        # the latency case: a short text, one short pattern, a hundred hits
        {"name": "one_small", "family": "one", "n": MIB, "alphabet": 26, "m": 8, "plants": 100, "mode": "screen"},
        # the headline scan: one long pattern over a large DNA text
        {"name": "one_large", "family": "one", "n": 4096 * MIB, "alphabet": 4, "m": 32, "plants": 10000,
         "mode": "screen"},
        # the same with every window's 61-bit hash tested, on a ragged length
        {"name": "one_exact", "family": "one", "n": 1024 * MIB + 4321, "alphabet": 4, "m": 32, "plants": 2500,
         "mode": "exact"},
        # a short pattern over DNA: a hit every 256 bytes by chance
        {"name": "one_short", "family": "one", "n": 256 * MIB + 77, "alphabet": 4, "m": 4, "plants": 0,
         "mode": "screen"},
        # a thousand patterns over word text, a hit every 32 bytes
        {"name": "many_screen", "family": "many", "n": 1024 * MIB, "k": 1024, "mmin": 16, "mmax": 16,
         "mode": "screen"},
        # a smaller set of mixed lengths, every length class with a hash stream of its own
        {"name": "many_exact", "family": "many", "n": 200 * MIB + 9, "k": 300, "mmin": 12, "mmax": 64,
         "mode": "exact"},
        # a dictionary: more patterns than one digit of the sort covers
        {"name": "dict", "family": "dict", "n": 64 * MIB + 1001, "k": 6000, "mmin": 12, "mmax": 40, "mode": "screen"},
        # the one-line call on a text of some MiB
        {"name": "call", "family": "call", "n": 8 * MIB + 13, "k": 24, "mmin": 4, "mmax": 64, "mode": "auto"},
        # a thousand uneven instances, 4 KiB to 16 MiB, in one batch
        {"name": "batch", "family": "batch", "count": 1024, "nmax": 16 * MIB, "kmax": 32, "mode": "screen"},
        # requests against resident corpora, as a client sees them
        {"name": "serve", "family": "serve", "corpora": 4, "n": 16 * MIB, "requests": 24, "kmax": 64,
         "mode": "screen"},
        # a text in host memory, longer than one piece
        {"name": "host", "family": "host", "n": 400 * MIB + 5, "m": 32, "plants": 1000, "piece": 256 * MIB,
         "mode": "screen"},
        # the one-thread-per-offset procedure on a 320 MB DNA text
        {"name": "paper", "family": "paper", "n": 320000000, "m": 25, "tpb": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = rng.choice(["one", "one", "many", "many", "dict", "call", "batch", "serve", "host", "paper"])
    mode = rng.choice(["screen", "exact"])
    if f == "one":
        n = _log(rng, 4096, 4096 * MIB)
        m = rng.randint(4, 64)
        return {"family": f, "n": n, "alphabet": rng.choice([4, 26, 256]), "m": m,
                "plants": min(rng.randint(0, 10000), n // (8 * m)), "mode": mode}
    if f == "many":
        m = rng.randint(12, 64)
        return {"family": f, "n": _log(rng, MIB, 1024 * MIB), "k": _log(rng, 16, 1024), "mmin": rng.choice([12, m]),
                "mmax": m, "mode": mode}
    if f == "dict":
        return {"family": f, "n": _log(rng, MIB, 64 * MIB), "k": rng.randint(2049, 8192), "mmin": 12,
                "mmax": rng.randint(13, 64), "mode": mode}
    if f == "call":
        return {"family": f, "n": _log(rng, 4096, 64 * MIB), "k": rng.randint(1, 64), "mmin": 4,
                "mmax": rng.randint(5, 64), "mode": rng.choice(["auto", "exact"])}
    if f == "batch":
        return {"family": f, "count": _log(rng, 16, 1024), "nmax": _log(rng, 65536, 16 * MIB),
                "kmax": rng.randint(1, 32), "mode": mode}
    if f == "serve":
        return {"family": f, "corpora": rng.randint(1, 4), "n": _log(rng, MIB, 16 * MIB),
                "requests": rng.randint(2, 24), "kmax": rng.randint(1, 64), "mode": mode}
    if f == "host":
        n = _log(rng, MIB, 400 * MIB)
        return {"family": f, "n": n, "m": rng.randint(20, 64), "plants": min(1000, n // 1024),
                "piece": rng.choice([64, 256]) * MIB, "mode": mode}
    return {"family": f, "n": _log(rng, 1000000, 320000000), "m": rng.choice([7, 25, 50, rng.randint(4, 200)]),
            "tpb": rng.choice(TPB)}


# ------------------------------------------------------------------- inputs
def _alphabet(a):
    if a == 4:
        return np.frombuffer(b"ACGT", np.uint8)
    if a == 26:
        return np.arange(97, 123, dtype=np.uint8)
    return np.arange(256, dtype=np.uint8)


def _iid(gen, n, a):
    """n bytes drawn uniformly from the alphabet of a letters, on the device."""
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    table = torch.from_numpy(_alphabet(a).copy()).to(DEV)
    for s in range(0, n, CHUNK):
        c = out[s:s + CHUNK]
        c.random_(0, a, generator=gen)
        if a == 4:
            c.copy_(table[c.long()])
        elif a == 26:
            c.add_(97)
    return out


def _plant(g, text, pattern, plants):
    """Copies of the pattern at distinct multiples of 2 m, on the device."""
    m = len(pattern)
    slots = text.numel() // (2 * m)
    if plants and slots >= plants:
        at = torch.from_numpy(np.sort(g.choice(slots, size=plants, replace=False)) * (2 * m)).to(DEV)
        p = torch.from_numpy(np.frombuffer(pattern, np.uint8).copy()).to(DEV)
        text[(at[:, None] + torch.arange(m, device=DEV)[None, :]).reshape(-1)] = p.repeat(plants)


def _words(g, gen, n, words=50000):
    """Word text: lengths 3..12 over 'a'..'z', ranks from a finite Zipf(1.1), single spaces."""
    lens = g.integers(3, 13, size=words)
    wl = torch.from_numpy(lens + 1).to(DEV)
    start = torch.cumsum(wl, 0) - wl
    blob = torch.from_numpy(g.integers(97, 123, size=int(lens.sum()) + words, dtype=np.uint8)).to(DEV)
    blob[start + wl - 1] = 32
    cdf = torch.cumsum(torch.arange(1, words + 1, device=DEV, dtype=torch.float64) ** -1.1, 0)
    cdf /= cdf[-1].clone()
    out = torch.empty(n, dtype=torch.uint8, device=DEV)
    filled = 0
    step = min(1 << 22, n // 4 + 16)
    while filled < n:
        r = torch.searchsorted(cdf, torch.rand(step, generator=gen, device=DEV, dtype=torch.float64)).clamp_(max=words - 1)
        ends = torch.cumsum(wl[r], 0)
        take = min(int(ends[-1]), n - filled)
        shift = start[r] - (ends - wl[r])
        src = torch.repeat_interleave(shift, wl[r])[:take] + torch.arange(take, device=DEV)
        out[filled:filled + take] = blob[src]
        filled += take
    return out


def _pattern_set(g, text, k, mmin, mmax):
    """k patterns of mmin..mmax bytes, half copied from the text, half random letters."""
    ms = g.integers(mmin, mmax + 1, size=k)
    at = (g.random(k) * (text.numel() - mmax)).astype(np.int64)
    rows = torch.from_numpy(at).to(DEV)[:, None] + torch.arange(mmax, device=DEV)[None, :]
    rows = text[rows].cpu().numpy()
    rnd = g.integers(97, 123, size=(k, mmax), dtype=np.uint8)
    return [(rows if j % 2 == 0 else rnd)[j, :ms[j]].tobytes() for j in range(k)]


def _context():
    ctx = rk.Context(0)
    ctx.autotune_load(TUNED)
    return ctx


def _one_pattern(g, case):
    a = _alphabet(case.get("alphabet", 4))
    return a[g.integers(0, len(a), size=case["m"])].tobytes()


def prepare(case, seed):
    f = case["family"]
    g = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    st = {"family": f, "case": dict(case)}
    if f in ("one", "host", "paper"):
        text = _iid(gen, case["n"], case.get("alphabet", 4))
        pat = _one_pattern(g, case)
        _plant(g, text, pat, case.get("plants", min(1000, case["n"] // (8 * case["m"]))))
        st["patterns"] = [pat]
        st["text"] = text.cpu().numpy() if f == "host" else text
    elif f in ("many", "dict", "call"):
        st["text"] = _words(g, gen, case["n"])
        st["patterns"] = _pattern_set(g, st["text"], case["k"], case["mmin"], case["mmax"])
    k = len(st.get("patterns", ()))
    if f in ("one", "many", "dict"):
        st["out"] = (torch.zeros(k + 1, dtype=torch.int64, device=DEV), _positions(case))
    elif f in ("call", "paper"):
        st["out"] = _positions(case)
    if f == "call":  # the call makes its own plan on the default context
        return st
    st["ctx"] = _context()
    if f in ("one", "many", "dict", "host"):
        st["plan"] = rk.Plan(st["ctx"], st["patterns"], case["mode"])
    elif f == "batch":
        st.update(_batch(g, gen, case, st["ctx"]))
    elif f == "serve":
        st.update(_serve(g, gen, case, st["ctx"]))
    return st


def _positions(case):
    """The program's buffer for the positions: more than the case ever has."""
    n, k = case["n"], case.get("k", 1)
    if case["family"] in ("one", "paper"):
        hits = n * float(case.get("alphabet", 4)) ** -case["m"]
        cap = case.get("plants", 1000) + 1.25 * hits + 10000
    else:
        cap = n * k / 2 * (2e-2 if case["family"] == "call" else 6e-4) + 65536
    return torch.zeros(int(cap), dtype=torch.int64, device=DEV)


def _batch(g, gen, case, ctx):
    """Instances of log-uniform length, 4, 26 or 256 letters, 1..kmax patterns
    of 4..64 bytes, every other one planted up to 8 times.  Lengths and
    pattern counts are the case's, the bytes the seed's."""
    texts, sets = [], []
    dst, src = [], []
    gs = np.random.Generator(np.random.PCG64(case["count"]))
    ns = [_log_np(gs, 4096, case["nmax"]) for _ in range(case["count"])]
    ks = [int(gs.integers(1, case["kmax"] + 1)) for _ in range(case["count"])]
    starts = np.concatenate([[0], np.cumsum([(n + 255) // 256 * 256 for n in ns])])
    buf = torch.empty(int(starts[-1]), dtype=torch.uint8, device=DEV)
    for i, n in enumerate(ns):
        base = int(starts[i])
        a = int(g.choice([4, 26, 256]))
        text = buf[base:base + n]
        text.random_(0, a, generator=gen)
        al = _alphabet(a)
        if a == 4:
            text.copy_(torch.from_numpy(al.copy()).to(DEV)[text.long()])
        elif a == 26:
            text.add_(97)
        pats = [al[g.integers(0, a, size=int(m))] for m in g.integers(4, 65, size=ks[i])]
        planted = pats[::2]
        slots = g.permutation(n // 64)[:8 * len(planted)]
        for j, s in enumerate(slots.tolist()):
            p = planted[j % len(planted)]
            dst.append(base + 64 * s + np.arange(len(p)))
            src.append(p)
        texts.append(text)
        sets.append([p.tobytes() for p in pats])
    buf[torch.from_numpy(np.concatenate(dst)).to(DEV)] = torch.from_numpy(np.concatenate(src)).to(DEV)
    out = torch.zeros(sum(ns) // 64 + 8 * sum(ks) + 65536, dtype=torch.int64, device=DEV)
    return {"texts": texts, "sets": sets, "plan": rk.BatchPlan(ctx, texts, sets, case["mode"]), "out": out}


def _log_np(g, lo, hi):
    return int(math.exp(g.uniform(math.log(lo), math.log(hi))))


def _serve(g, gen, case, ctx):
    """Resident corpora of word text and the requests of one burst, each of
    1..kmax patterns of 4..64 bytes."""
    srv = rk.Server(ctx, arena_bytes=2 << 30, mode=case["mode"])
    texts = [_words(g, gen, case["n"]) for _ in range(case["corpora"])]
    cids = [srv.add_corpus(t) for t in texts]
    reqs = []
    for _ in range(case["requests"]):
        c = int(g.integers(0, case["corpora"]))
        reqs.append((cids[c], _pattern_set(g, texts[c], int(g.integers(1, case["kmax"] + 1)), 4, 64)))
    torch.cuda.synchronize()
    cap = int(case["requests"] * case["kmax"] * case["n"] * 1.5e-3) + 65536
    return {"texts": texts, "server": srv, "requests": reqs, "counts": np.zeros((case["requests"], case["kmax"]), np.int64),
            "out": np.zeros(cap, np.int64)}


# --------------------------------------------------------------------- runs
def run(st):
    f = st["family"]
    if f in ("one", "many", "dict"):
        total = st["plan"].count(st["text"])
        st["plan"].collect(st["text"], total, out=st["out"])
        return st["out"]
    if f == "host":
        return st["plan"].search_host(st["text"], st["case"]["piece"])
    if f == "serve":
        return _burst(st)
    if f == "paper":
        first = st["ctx"].paper_search(st["text"], st["patterns"][0], st["case"]["tpb"])
        positions = st["ctx"].paper_positions(first)
    elif f == "call":
        first, positions = rk.search(st["text"], st["patterns"], mode=st["case"]["mode"])
    else:
        first, positions = st["plan"].search()
    st["out"][:positions.numel()] = positions
    return first, st["out"]


def _burst(st):
    """Submits the burst, then takes every result in turn into the client's buffer."""
    srv, at = st["server"], 0
    rids = [srv.submit(c, p) for c, p in st["requests"]]
    for i, rid in enumerate(rids):
        r = srv.wait(rid)
        offs, pos = r["offsets"], r["positions"]
        st["counts"][i, :len(offs) - 1] = offs[1:] - offs[:-1]
        st["out"][at:at + len(pos)] = pos
        at += len(pos)
        srv.release(rid)
    return st["counts"], st["out"]


# --------------------------------------------------------------------- work
def work(case):
    """Bytes: the text read once, the positions (8 bytes each) and offsets
    written once; operations: one 8-bit multiply-add per text byte and hash
    stream.  Hit counts of the word texts are expectations of the generator
    (a copied pattern of 16 bytes recurs every 16,000 bytes, a shorter one
    more often)."""
    f = case["family"]
    if f == "batch":
        ln = math.log(case["nmax"] / 4096.0)
        n = case["count"] * ((case["nmax"] - 4096) / ln if ln > 0 else 4096)
        k = case["count"] * (case["kmax"] + 1) / 2
        return {"bytes": int(n + 8 * (4 * k + k + 1)), "flops": int(2 * n)}
    if f == "serve":
        n = case["corpora"] * case["n"]
        k = case["requests"] * (case["kmax"] + 1) / 2
        return {"bytes": int(n + 8 * (k + case["n"] * k * 1.1e-4)), "flops": int(2 * n)}
    n = case["n"]
    if f == "paper":
        return {"bytes": int(2 * n + 8 * min(1000, n // (8 * case["m"]))), "flops": int(2 * n * min(case["m"], 32))}
    if f in ("one", "host"):
        hits = case["plants"] + n * float(case.get("alphabet", 4)) ** -case["m"]
        return {"bytes": int(n + 8 * (hits + 2)), "flops": int(2 * n)}
    per = 6.1e-5 if case["mmin"] >= 16 else 1.0e-4
    return {"bytes": int(n + 8 * (case["k"] + 1 + n * case["k"] / 2 * per)), "flops": int(2 * n)}


# -------------------------------------------------------------------- exact
def exact(case, seed):
    """The occurrences by plain byte search on the host, for the cases that
    are small enough; every output of these workloads is a whole number or a
    byte."""
    if case["family"] not in ("one", "call") or case["n"] * case.get("k", 1) > 64 * MIB:
        return None
    st = prepare(case, seed)
    text = st["text"].cpu().numpy().tobytes()
    offsets, positions = [0], []
    for p in st["patterns"]:
        at = text.find(p)
        while at >= 0:
            positions.append(at)
            at = text.find(p, at + 1)
        offsets.append(len(positions))
    out = torch.zeros(_positions(case).shape, dtype=torch.int64)
    out[:len(positions)] = torch.tensor(positions, dtype=torch.int64)
    return torch.tensor(offsets, dtype=torch.int64), out
