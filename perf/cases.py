"""Timed workloads of the library, through its public entry points.

A case is a dict of sizes and parameters.  ``prepare`` draws its strings on the
GPU from a seed (clusters of mutated copies of random strings, the recipe of
``synthdata``), ``run`` makes one call as a user's program does.  Lengths are
uniform in [lo, hi], or log-uniform where hi is at least four times lo.
"""
import math

import numpy as np
import torch

import paper_1702_00093_amd as ej


def listed():
    return [
        # One query against a resident index of short reads: serving latency.
        dict(name="query_one", kind="query", n=20000, copies=10, lo=900, hi=1100, letters=4,
             edit_lo=0.05, edit_hi=0.05, nq=1, r=32, z=8, m=20, L=64),
        # Saturated serving: a batch of long-read queries, thresholds of 2, 5 and 10%.
        dict(name="query_batch", kind="query", n=100000, copies=10, lo=4500, hi=5500, letters=4,
             edit_lo=0.05, edit_hi=0.05, nq=4096, r=32, z=8, m=20, L=64),
        # Building the serving index from strings in HBM, and a first small batch on it.
        dict(name="index_build", kind="build", n=60000, copies=10, lo=4500, hi=5500, letters=4,
             edit_lo=0.05, edit_hi=0.05, nq=64, r=32, z=8, m=20, L=64),
        # A small set held by a host program (a few clusters to clean up): host arrays in,
        # host arrays out, launch and synchronisation latency.
        dict(name="join_small_host", kind="join", form="host", n=203, copies=8, lo=300, hi=500,
             letters=4, edit_lo=0.03, edit_hi=0.03, K=25, r=7, z=16, m=8, L=64, exact_len=0),
        # The 2,000-string DNA set, joined again and again in place (graph replay).
        dict(name="join_tiny_graph", kind="join", form="graph", n=2000, copies=10, lo=900, hi=1100,
             letters=4, edit_lo=0.03, edit_hi=0.03, K=50, r=7, z=16, m=8, L=64, exact_len=0),
        # The benchmark's workload: 20,000 genome reads of about 5,000 letters, K=500,
        # left in HBM.
        dict(name="join_medium", kind="join", form="device", n=20000, copies=10, lo=4500, hi=5500,
             letters=4, edit_lo=0.04, edit_hi=0.04, K=500, r=32, z=16, m=18, L=64, exact_len=0),
        # Uneven lengths over a factor of 40, K=400.
        dict(name="join_uneven", kind="join", form="device", n=60000, copies=4, lo=500, hi=20000,
             letters=4, edit_lo=0.0, edit_hi=0.08, K=400, r=32, z=16, m=16, L=64, exact_len=0),
        # Protein-like strings (25 letters, skewed), the stated parameters of that set: very many
        # candidates among the strings not much longer than K.
        dict(name="join_protein", kind="join", form="device", n=200001, copies=4, lo=50, hi=4000,
             letters=25, edit_lo=0.02, edit_hi=0.15, K=100, r=5, z=10, m=32, L=1101, exact_len=0,
             results=50000000),
        # The join made exact among short strings: the exhaustive pass's many candidates.
        dict(name="join_short_pass", kind="join", form="device", n=9000, copies=3, lo=400, hi=6000,
             letters=4, edit_lo=0.0, edit_hi=0.08, K=200, r=16, z=16, m=12, L=64, exact_len=900),
        # EmbedJoin+ on genome reads with shifted starts, walks over the average length.
        dict(name="plus_shifted", kind="plus", n=30000, copies=10, lo=4500, hi=5500, letters=4,
             edit_lo=0.003, edit_hi=0.003, shift=60, K=100, delta=50, T=2, r=6, z=16, m=8, L=0),
        # Grouping by length in place of truncation: many front ends on small sets.
        dict(name="grouped_uneven", kind="grouped", n=8000, copies=4, lo=500, hi=12000, letters=4,
             edit_lo=0.0, edit_hi=0.06, K=400, r=8, z=16, m=16, L=0, results=2000000),
        # Verification alone on a caller's pairs (half similar, half not), 25 letters, with a
        # threshold per pair.
        dict(name="verify_pairs", kind="verify", n=4001, copies=5, lo=100, hi=1500, letters=25,
             edit_lo=0.01, edit_hi=0.12, pairs=30011, K=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; the text of a case stays under about 300 MB."""
    kind = rng.choice(["query", "query", "build", "join", "join", "join", "join", "plus",
                       "grouped", "verify", "verify"])
    lo = _log_int(rng, 60, 4500)
    hi = int(lo * rng.choice([1.2, 1.5, 5, 20])) + 1
    if kind == "grouped":
        lo, hi = min(lo, 1000), min(hi, 12000)
    hi = max(lo, min(hi, 20000))
    mean = (lo + hi) / 2 if hi < 4 * lo else (hi - lo) / math.log(hi / lo)
    letters = rng.choice([4, 4, 4, 20, 25])
    top = {"query": 100000, "build": 60000, "join": 60000, "plus": 30000, "grouped": 6000,
           "verify": 8000}[kind]
    n = _log_int(rng, 50, max(51, min(top, int(3e8 / mean))))
    e = rng.uniform(0.002, 0.06)
    c = dict(kind=kind, n=n, copies=rng.randint(2, 12), lo=lo, hi=hi, letters=letters,
             edit_lo=0.0 if rng.random() < 0.5 else e, edit_hi=e)
    K = max(1, min(600, int(mean * rng.uniform(0.01, 0.12))))
    lsh = dict(r=rng.randint(3, 32), z=rng.choice([7, 8, 16]),
               m=rng.randint(14, 24) if letters == 4 else rng.randint(8, 16),
               L=rng.choice([64, 64, 200]))
    if kind in ("query", "build"):
        c.update(nq=_log_int(rng, 1, 4096 if kind == "query" else 64), **lsh)
        c.update(nq=max(1, min(c["nq"], int(2e7 / mean))))
    elif kind == "verify":
        pairs = min(_log_int(rng, 10, 60000), int(6e10 / (mean * max(K, 32))))
        c.update(pairs=max(1, pairs), K=rng.choice([0, K]))
    else:
        c.update(K=K, **lsh)
        if kind == "join":
            c.update(form=rng.choice(["host", "device", "device", "graph"]), exact_len=0)
            if n < 8000 and rng.random() < 0.25:
                c.update(exact_len=int(mean * rng.uniform(0.3, 0.8)), form="device")
        elif kind == "plus":
            c.update(shift=rng.randint(0, 60), K=min(K, 150), T=rng.choice([0, 2]))
            c.update(delta=rng.choice([0, 50, 25]), r=min(c["r"], 8))
        else:
            c.update(r=min(c["r"], 8), L=0, K=max(K, hi // 40))
    return c


# ------------------------------------------------------------------ inputs --

def _letters(count, letters, gen):
    """`count` letter codes: uniform, or Zipf(1.1) for the wide alphabets."""
    if letters <= 4:
        return torch.randint(0, letters, (count,), generator=gen, device="cuda",
                             dtype=torch.uint8)
    p = torch.arange(1, letters + 1, device="cuda", dtype=torch.float32) ** -1.1
    cdf = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(count, generator=gen, device="cuda")
    return torch.searchsorted(cdf, u).clamp_(max=letters - 1).to(torch.uint8)


def _lengths(count, lo, hi, gen):
    u = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64)
    if hi >= 4 * lo:
        return (lo * (hi / lo) ** u).round().long()
    return (lo + u * (hi - lo)).round().long()


def _starts(length):
    off = torch.zeros(length.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=off[1:])
    return off


def _mutated(text, start, length, rate, letters, gen):
    """Copies of text[start[i] : start[i] + length[i]], each letter edited with
    probability rate[i] (substitution, deletion or insertion alike)."""
    off = _starts(length)
    total = int(off[-1])
    sid = torch.repeat_interleave(torch.arange(length.numel(), device="cuda"), length,
                                  output_size=total)
    src = torch.arange(total, device="cuda") + (start - off[:-1])[sid]
    u = torch.rand(total, generator=gen, device="cuda") / rate.float()[sid].clamp_(min=1e-9)
    del sid
    gone, more, other = u < 1 / 3, (u >= 1 / 3) & (u < 2 / 3), (u >= 2 / 3) & (u < 1)
    del u
    code = text[src]
    del src
    fresh = _letters(total, letters, gen)
    code = torch.where(other & (fresh != code), fresh,
                       torch.where(other, (code + 1) % letters, code))
    end = torch.cumsum(1 + more.int() - gone.int(), 0)
    new_off = torch.zeros_like(off)
    has = off[1:] > 0
    new_off[1:][has] = end[off[1:][has] - 1]
    out = torch.empty(int(new_off[-1]), dtype=torch.uint8, device="cuda")
    keep = ~gone
    out[end[keep] - 1] = code[keep]
    out[end[more] - 2] = fresh[more]
    return out, new_off


def _strings(case, gen):
    """Letter codes and offsets of the case's strings, and each one's cluster."""
    n, shift = case["n"], case.get("shift", 0)
    nb = max(1, n // case["copies"])
    if case["letters"] > 4 and case["lo"] == 50:
        z = torch.randn(nb, generator=gen, device="cuda", dtype=torch.float64)
        blen = (400 * torch.exp(0.8 * z)).round().long().clamp_(case["lo"], case["hi"])
    else:
        blen = _lengths(nb, case["lo"], case["hi"], gen)
    boff = _starts(blen + shift)
    base = _letters(int(boff[-1]), case["letters"], gen)
    owner = torch.randint(0, nb, (n,), generator=gen, device="cuda")
    rate = case["edit_lo"] + (case["edit_hi"] - case["edit_lo"]) * torch.rand(
        n, generator=gen, device="cuda", dtype=torch.float64)
    start = boff[owner] + torch.randint(0, shift + 1, (n,), generator=gen, device="cuda")
    codes, off = _mutated(base, start, blen[owner], rate, case["letters"], gen)
    return codes, off, owner


def _bytes_of(codes, letters):
    table = b"ACGT" if letters <= 4 else b"ACDEFGHIKLMNPQRSTVWYBZXJU"[:letters]
    return torch.tensor(list(table), dtype=torch.uint8, device="cuda")[codes.long()]


def _queries(case, codes, off, gen):
    """70% re-mutated members, 30% fresh strings; thresholds of 2, 5 or 10% (host arrays)."""
    nq, n = case["nq"], case["n"]
    src = torch.randint(0, n, (nq,), generator=gen, device="cuda")
    fresh = torch.rand(nq, generator=gen, device="cuda") < 0.3
    flen = _lengths(nq, max(1, case["lo"] // 4), case["hi"] * 2, gen).clamp_(max=20000)
    foff = _starts(flen)
    text = torch.cat([codes, _letters(int(foff[-1]), case["letters"], gen)])
    start = torch.where(fresh, codes.numel() + foff[:-1], off[src])
    length = torch.where(fresh, flen, off[src + 1] - off[src])
    rate = torch.where(fresh, 0.0, 0.05).double()
    q, qoff = _mutated(text, start, length, rate, case["letters"], gen)
    frac = torch.tensor([0.02, 0.05, 0.10], device="cuda", dtype=torch.float64)[
        torch.randint(0, 3, (nq,), generator=gen, device="cuda")]
    Kq = (frac * (qoff[1:] - qoff[:-1])).floor().long()
    return (_bytes_of(q, case["letters"]).cpu().numpy(), qoff.cpu().numpy().astype(np.uint64),
            Kq.cpu().numpy().astype(np.uint32))


def _pairs(case, off, owner, gen):
    """Pairs of neighbours in cluster order (similar) and of random strings, and
    thresholds of 2 to 15% of the longer one (case K = 0) or None."""
    n, count = case["n"], case["pairs"]
    order = torch.argsort(owner, stable=True)
    at = torch.randint(0, n - 1, (count,), generator=gen, device="cuda")
    a, b = order[at], order[at + 1]
    b = torch.where(torch.rand(count, generator=gen, device="cuda") < 0.5, b,
                    torch.randint(0, n, (count,), generator=gen, device="cuda"))
    Kq = None
    if case["K"] == 0:
        length = off[1:] - off[:-1]
        frac = 0.02 + 0.13 * torch.rand(count, generator=gen, device="cuda")
        Kq = (frac * torch.maximum(length[a], length[b])).floor().int().clamp_(max=2046)
    return (a << 32) | b, Kq


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ctx = ej.context(0)
    codes, off, owner = _strings(case, gen)
    s = dict(case=case, ctx=ctx, chars=_bytes_of(codes, case["letters"]), offsets=off)
    kind = case["kind"]
    if kind in ("query", "build"):
        s["queries"] = _queries(case, codes, off, gen)
        if kind == "query":
            torch.cuda.synchronize()
            s["index"] = _index(s)
            del s["chars"], s["offsets"]
    elif kind == "verify":
        s["pairs"], s["Kq"] = _pairs(case, off, owner, gen)
    elif case.get("form") == "host":
        s["chars"], s["offsets"] = s["chars"].cpu().numpy(), off.cpu().numpy().astype(np.uint64)
    _buffers(s)
    torch.cuda.synchronize()
    return s


# -------------------------------------------------------------------- calls --

def _index(s):
    c = s["case"]
    return ej.Index(s["ctx"], s["chars"], s["offsets"], r=c["r"], z=c["z"], m=c["m"], seed=0,
                    L=c["L"])


def _shorts(case):
    """Expected number of strings that the exhaustive pass takes."""
    S, lo, hi = case.get("exact_len", 0), case["lo"], case["hi"]
    if S <= lo:
        return 0.0
    S = min(S, hi)
    return case["n"] * (math.log(S / lo) / math.log(hi / lo) if hi >= 4 * lo
                        else (S - lo) / max(1, hi - lo))


def _buffers(s):
    """Result arrays of the caller's, sized for the case: a call's results go to their
    front, -1 stands behind them."""
    c = s["case"]
    if c["kind"] == "verify":
        return
    if c["kind"] in ("query", "build"):
        cap = 4096 + 4 * c["copies"] * c["nq"]
        s["ids"], s["dist"] = np.full(cap, -1, np.int64), np.full(cap, -1, np.int32)
        return
    n = c["n"]
    cap = 65536 + 2 * n * c["copies"] + int(0.75 * _shorts(c) ** 2) + c.get("results", 0)
    cap = min(cap, n * (n - 1) // 2)
    if c.get("form") == "host":
        s["pairs"], s["dist"] = np.full((cap, 2), -1, np.int64), np.full(cap, -1, np.int32)
    else:
        s["pairs"] = torch.full((cap, 2), -1, dtype=torch.int32, device="cuda")
        s["dist"] = torch.full((cap,), -1, dtype=torch.int32, device="cuda")


def _into(s, names, found):
    """The results in the caller's arrays (as they are, should they not fit)."""
    count = found[0].shape[0]
    if count > s[names[0]].shape[0]:
        return dict(zip(names, found), count=count)
    for name, x in zip(names, found):
        s[name][:count] = x
    return dict({name: s[name] for name in names}, count=count)


def _answer(s, res):
    out = _into(s, ("ids", "dist"), (res.ids, res.dist))
    return dict(out, offsets=res.offsets.astype(np.int64), candidates=res.n_candidates)


def _joined(s, res):
    found = (res.pairs, res.dist) if s["case"].get("form") == "host" else \
        (res.pairs_device, res.dist_device)
    return dict(_into(s, ("pairs", "dist"), found), candidates=res.n_candidates, raw=res.n_raw)


def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "query":
        return _answer(s, s["index"].query(*s["queries"]))
    if kind == "build":
        index = _index(s)
        out = _answer(s, index.query(*s["queries"]))
        index.close()
        return out
    if kind == "verify":
        return ctx.verify(s["chars"], s["offsets"], s["pairs"], c["K"], d_Kq=s["Kq"])
    args = (s["chars"], s["offsets"], c["K"], c["r"], c["z"], c["m"])
    if kind == "plus":
        return _joined(s, ctx.join_plus(*args, delta=c["delta"], T=c["T"], L=c["L"],
                                        flags=ej.FLAG_DEVICE_OUT))
    if kind == "grouped":
        return _joined(s, ctx.join_grouped(*args, L=c["L"], flags=ej.FLAG_DEVICE_OUT))
    flags = {"host": 0, "device": ej.FLAG_DEVICE_OUT,
             "graph": ej.FLAG_DEVICE_OUT | ej.FLAG_GRAPH}[c["form"]]
    return _joined(s, ctx.join(*args, L=c["L"], flags=flags, exact_len=c["exact_len"]))


# ------------------------------------------------------------------- bounds --

def work(case):
    """Strings read once and results written once; verification's recurrence
    (10 operations per 32 cells of the K+1 band and column) over the planted
    pairs, and the walks' 3 operations per step."""
    lo, hi = case["lo"], case["hi"]
    mean = (lo + hi) / 2 if hi < 4 * lo else (hi - lo) / math.log(hi / lo)
    if case["letters"] > 4 and lo == 50:
        mean = 540
    n, kind = case["n"], case["kind"]

    def band(K):
        return mean * 10 * ((K + 32) // 32)

    planted = n * case["copies"] / 2
    if kind == "verify":
        K = case["K"] or 0.085 * mean
        return dict(bytes=n * mean + 12 * case["pairs"], flops=case["pairs"] / 2 * band(int(K)))
    steps = case["L"] or mean
    if kind in ("query", "build"):
        nq = case["nq"]
        found = 0.7 * nq * case["copies"]
        text = (n * mean if kind == "build" else found * mean) + nq * mean
        walks = nq + (n if kind == "build" else 0)
        return dict(bytes=text + 8 * found + 12 * nq,
                    flops=found * band(int(0.057 * mean)) + walks * case["r"] * steps * 3)
    shorts = _shorts(case) ** 2 / 2
    if shorts:
        shorts *= min(1.0, 2 * case["K"] / max(1, min(case["exact_len"], hi) - lo))
    if kind == "plus":
        steps *= math.ceil(case["K"] / (case["delta"] or max(1, int(mean ** 0.5))))
    if kind == "grouped":
        steps = 6 * mean
    return dict(bytes=n * (mean + 8) + 12 * planted,
                flops=planted * band(case["K"]) + shorts * band(case["K"]) / mean * lo
                + n * case["r"] * steps * 3)


def exact(case, seed):
    """Distances of the verification cases by the full dynamic program, cell by
    cell along anti-diagonals.  A join's and a query's candidates depend on the
    library's random streams, so they have no value apart from it."""
    if case["kind"] != "verify" or case["pairs"] * float(case["hi"]) ** 2 > 1.5e11:
        return None
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    codes, off, owner = _strings(case, gen)
    pairs, Kq = _pairs(case, off, owner, gen)
    length = off[1:] - off[:-1]
    a, b = pairs >> 32, pairs & 0xFFFFFFFF
    la, lb = length[a], length[b]
    W = int(torch.maximum(la.max(), lb.max()))
    col = torch.arange(W, device="cuda")

    def rows(ids, ln, pad):
        at = (off[ids][:, None] + col).clamp_(max=max(0, codes.numel() - 1))
        return torch.where(col < ln[:, None], codes[at], pad)

    A, B = rows(a, la, 254), rows(b, lb, 255).flip(1)
    big = 1 << 20
    two = torch.full((A.shape[0], W + 1), big, dtype=torch.int32, device="cuda")
    one = two.clone()
    one[:, 0] = 0                       # anti-diagonal 0: cell (0, 0)
    out = torch.where(la + lb == 0, 0, big).int()
    end = la + lb
    for d in range(1, int(end.max()) + 1):
        i0, i1 = max(0, d - W), min(W, d)
        cur = torch.full_like(one, big)
        cur[:, i0:i1 + 1] = one[:, i0:i1 + 1] + 1
        j0 = max(1, i0)
        cur[:, j0:i1 + 1] = torch.minimum(cur[:, j0:i1 + 1], one[:, j0 - 1:i1] + 1)
        lo_i, hi_i = max(1, d - W), min(W, d - 1)
        if lo_i <= hi_i:
            # row i reads A[i - 1] against column j = d - i, letter B[j - 1]
            s = W - d
            miss = A[:, lo_i - 1:hi_i] != B[:, s + lo_i:s + hi_i + 1]
            cur[:, lo_i:hi_i + 1] = torch.minimum(cur[:, lo_i:hi_i + 1],
                                                  two[:, lo_i - 1:hi_i] + miss)
        at = torch.nonzero(end == d).flatten()
        out[at] = cur[at, la[at]]
        two, one = one, cur
    limit = Kq if Kq is not None else case["K"]
    return torch.minimum(out, torch.as_tensor(limit, device="cuda", dtype=torch.int32) + 1)
