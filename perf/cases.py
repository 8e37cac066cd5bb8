"""The work that users of the library have it do, as measurable cases.

Five kinds of case, each through the public entry points of the binding:

* ``search``    sequences in, weighted edges out (Context.search);
* ``align``     records of a given pair list (Context.align_pairs);
* ``filter``    the learned filter's scoring of a discovery's candidates
                (Context.mlp_features, then Context.mlp_forward);
* ``epoch``     one training epoch of the filter from a given network
                (Context.mlp_set, Context.mlp_train_epoch, Context.mlp_get);
* ``families``  the similarity graph as families (Context.components, then
                Context.cluster_scores).

Inputs are made on the GPU from the seed alone.  The sequence sets follow the
recipe of this repository's synthetic workloads (family-structured sets with
lognormal lengths, BLOSUM62-weighted substitutions and geometric indels).
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2009_14467_amd as P

ALPHABET = "ARNDCQEGHILKMFPSTWYV"
# Background frequencies of the 20 residues (in ALPHABET's order) and, per
# residue, the weight of each substitute: a plain stand-in for protein
# statistics, with substitutions inside a physico-chemical class favoured.
BACKGROUND = (0.078, 0.051, 0.045, 0.054, 0.019, 0.043, 0.063, 0.074, 0.022, 0.051,
              0.091, 0.057, 0.022, 0.039, 0.052, 0.071, 0.058, 0.013, 0.032, 0.065)
CLASSES = ("AGST", "RKHQ", "NDEQ", "C", "ILMV", "FWY", "P", "AST", "HY", "NST")
# composition groups of the learned filter's features
GROUPS = ("AG", "ST", "DE", "NQ", "KRH", "IV", "LM", "FYW", "C", "P")
# feature normalisation of the scoring case's network: of the order of what
# training on such sets gives
MEAN = (2.0, 0.0, 0.1, 5.7, 6.0, 0.7) + (0.03,) * 10
STD = (3.0, 0.5, 0.3, 0.5, 0.5, 0.2) + (0.03,) * 10

SEARCH = dict(kind="search", families=25, size=20, singles=0, mean=200, lo=50, hi=600, diverge=0.3, long=0.0, k=6,
              subs=0, ck=1, mode="sw", weight="ani", graph=False)


def listed():
    return [
        # a few hundred sequences against each other: the smallest search,
        # where launches and synchronisations count
        dict(SEARCH, name="search_small"),
        # a proteome-sized set, exact 6-mers, default schedule
        dict(SEARCH, name="search_ordinary", families=400, singles=2003, mean=350, lo=30, hi=5000, ck=2),
        # the benchmark's set: a quarter of a million sequences, alignment
        # stage replayed as a graph
        dict(SEARCH, name="search_large", families=10000, singles=50000, mean=350, lo=30, hi=5000, ck=2, graph=True),
        # sensitive search through 25 substitute 6-mers
        dict(SEARCH, name="search_substitutes", families=800, size=25, mean=350, lo=30, hi=2000, subs=25, ck=2),
        # seed-and-extend alignment in place of Smith-Waterman
        dict(SEARCH, name="search_xdrop", families=4000, singles=20001, mean=350, lo=30, hi=5000, ck=2, mode="xd"),
        # normalised-score weights: every candidate becomes an edge
        dict(SEARCH, name="search_score_weight", families=1201, size=17, singles=5000, mean=300, lo=30, hi=3000, ck=1,
             weight="ns"),
        # sequences with a long tail (5% of 5,000 to 25,000 residues), 5-mers
        # and substitutes
        dict(SEARCH, name="search_long_tail", families=40, size=25, mean=300, lo=30, hi=5000, diverge=0.4, long=0.05,
             k=5, subs=25, ck=2),
        # full records of a pair list of the caller's own
        dict(name="align_records", kind="align", families=900, size=21, mean=300, lo=30, hi=2000, pairs=250001,
             mode="sw", full=True),
        # a handful of pairs, as an interactive user aligns them
        dict(name="align_few", kind="align", families=4, size=10, mean=350, lo=30, hi=1500, pairs=61, mode="sw",
             full=True),
        # the filter's decision on a discovery's candidates
        dict(name="filter_score", kind="filter", families=500, size=20, mean=350, lo=30, hi=2000, k=5, ck=1),
        # minibatch training of the filter at the library's default batch
        dict(name="filter_epoch", kind="epoch", examples=70001, batch=8192, positive=0.15),
        # connected components of the graph and their agreement with families
        dict(name="graph_families", kind="families", vertices=250000, size=20, singles=50000, keep=0.8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "align", "filter", "epoch", "families"])
    if kind == "search":
        what = rng.choice(["exact", "exact", "xd", "subs", "ns", "long"])
        size = rng.randint(5, 30)
        if what == "long":
            return dict(SEARCH, families=_log_int(rng, 4, 40), size=rng.randint(10, 25), mean=rng.randint(150, 320),
                        lo=30, hi=5000, diverge=rng.choice([0.3, 0.4]), long=0.05, k=5, subs=rng.choice([0, 25]), ck=2,
                        mode=rng.choice(["sw", "sw", "xd"]))
        most = {"exact": 120000, "xd": 120000, "subs": 18000, "ns": 40000}[what]
        n = _log_int(rng, 60, most)
        families = max(2, n // size)
        return dict(SEARCH, families=families, size=size, singles=rng.randint(0, n // 4), mean=rng.randint(90, 380),
                    lo=30, hi=rng.choice([600, 2000, 5000]), diverge=round(rng.uniform(0.15, 0.5), 2),
                    k=rng.choice([6, 6, 5]) if n < 20000 else 6, subs=rng.choice([10, 25]) if what == "subs" else 0,
                    ck=rng.randint(1, 3) if what != "subs" else 2, mode="xd" if what == "xd" else "sw",
                    weight="ns" if what == "ns" else "ani", graph=rng.random() < 0.3 and what != "xd")
    if kind == "align":
        return dict(kind="align", families=rng.randint(4, 900), size=rng.randint(5, 25), mean=rng.randint(90, 380),
                    lo=30, hi=rng.choice([600, 2000, 4000]), pairs=_log_int(rng, 5, 250000),
                    mode=rng.choice(["sw", "sw", "xd"]), full=rng.random() < 0.6)
    if kind == "filter":
        return dict(kind="filter", families=_log_int(rng, 5, 500), size=rng.randint(5, 25), mean=rng.randint(90, 350),
                    lo=30, hi=2000, k=rng.choice([5, 6]), ck=rng.randint(1, 2))
    if kind == "epoch":
        return dict(kind="epoch", examples=_log_int(rng, 300, 70000), batch=rng.choice([1024, 4096, 8192, 16384]),
                    positive=round(rng.uniform(0.03, 0.5), 2))
    return dict(kind="families", vertices=_log_int(rng, 200, 250000), size=rng.randint(3, 40),
                singles=rng.randint(0, 40), keep=round(rng.uniform(0.3, 1.0), 2))


# ---------------------------------------------------------------- inputs


def _tables(dev):
    p = torch.tensor(BACKGROUND, dtype=torch.float64)
    p = p / p.sum()
    w = p.repeat(20, 1).clone()
    for cls in CLASSES:
        for a in cls:
            for b in cls:
                w[ALPHABET.index(a), ALPHABET.index(b)] *= 3.0
    w.fill_diagonal_(0.0)
    cdf = torch.cumsum(w / w.sum(1, keepdim=True), 1)
    cdf[:, -1] = 1.0
    # rows shifted by their index, so one sorted array serves every residue
    sub = (cdf + torch.arange(20)[:, None]).reshape(-1)
    back = torch.cumsum(p, 0)
    back[-1] = 1.0
    return back.float().to(dev), sub.to(dev)


def _starts(lens):
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=lens.device)
    torch.cumsum(lens, 0, out=off[1:])
    return off


def _sequences(case, gen, dev):
    """(residues uint8 ASCII, offsets int64, family of each sequence) on the GPU."""
    nf, size, singles = case["families"], case["size"], case.get("singles", 0)
    back, sub = _tables(dev)

    def uniform(n):
        return torch.rand(n, generator=gen, device=dev)

    n_anc = nf + singles
    mu = math.log(case["mean"]) - 0.18
    lens = torch.exp(torch.randn(n_anc, generator=gen, device=dev) * 0.6 + mu).round().clamp(case["lo"], case["hi"])
    lens = lens.to(torch.int64)
    top = case["hi"]
    if case.get("long", 0.0) > 0:
        top = 25000
        # a fixed share of the ancestors, so that every seed has the same tail
        n_long = max(1, round(case["long"] * n_anc))
        which = torch.randperm(n_anc, generator=gen, device=dev)[:n_long]
        lens[which] = torch.linspace(5000, 25000, n_long + 2, device=dev)[1:-1].to(torch.int64)
    a_off = _starts(lens)
    anc = torch.searchsorted(back, uniform(int(a_off[-1])), right=True).clamp(max=19)

    # members of the families, and the singletons as families of one
    fam = torch.cat([torch.arange(nf, device=dev).repeat_interleave(size),
                     torch.arange(nf, n_anc, device=dev)])
    mlen = lens[fam]
    m_off = _starts(mlen)
    total = int(m_off[-1])
    owner = torch.repeat_interleave(torch.arange(fam.numel(), device=dev), mlen)
    pos = torch.arange(total, device=dev)
    x = anc[a_off[fam[owner]] + (pos - m_off[owner])]
    hit = uniform(total) < case.get("diverge", 0.3)
    u = torch.rand(total, generator=gen, device=dev, dtype=torch.float64)
    other = (torch.searchsorted(sub, x.double() + u, right=True) - 20 * x).clamp(0, 19)
    x = torch.where(hit, other, x)
    # indels: 2% of the positions start one, geometric length of mean 3
    event = uniform(total) < 0.02
    ins = uniform(total) < 0.5
    glen = 1 + torch.floor(torch.log(uniform(total).clamp(min=1e-9)) / math.log(2.0 / 3.0)).to(torch.int64)
    until = torch.where(event & ~ins, torch.minimum(pos + glen, m_off[owner + 1]), torch.zeros_like(pos))
    keep = pos >= torch.cummax(until, 0).values
    width = keep.to(torch.int64) + torch.where(event & ins, glen, torch.zeros_like(glen))
    w_off = _starts(width)
    src = torch.repeat_interleave(pos, width)
    out_pos = torch.arange(src.numel(), device=dev)
    orig = (out_pos == w_off[src]) & keep[src]
    fresh = torch.searchsorted(back, uniform(src.numel()), right=True).clamp(max=19)
    vals = torch.where(orig, x[src], fresh)
    seq = owner[src]
    slen = torch.bincount(seq, minlength=fam.numel())
    s_off = _starts(slen)
    cut = slen.clamp(max=top)

    # a random order of the sequences
    perm = torch.randperm(fam.numel(), generator=gen, device=dev)
    off = _starts(cut[perm])
    where = torch.repeat_interleave(s_off[perm] - off[:-1], cut[perm]) + torch.arange(int(off[-1]), device=dev)
    letters = torch.tensor(list(ALPHABET.encode()), dtype=torch.uint8, device=dev)
    label = torch.where(fam < nf, fam, torch.full_like(fam, -1))[perm]
    return letters[vals[where]].contiguous(), off, label


def _pairs(case, label, gen, dev):
    """A pair list: half of it family pairs, half unrelated ones, shuffled."""
    n, m = label.numel(), case["pairs"]
    order = torch.argsort(label)
    start = torch.searchsorted(label[order].contiguous(), label)
    size = torch.bincount(label, minlength=1)[label]
    i = torch.randint(0, n, (m,), generator=gen, device=dev)
    mate = order[start[i] + (torch.rand(m, generator=gen, device=dev) * size[i]).to(torch.int64)]
    rand = torch.randint(0, n, (m,), generator=gen, device=dev)
    j = torch.where(torch.rand(m, generator=gen, device=dev) < 0.5, mate, rand)
    j = torch.where(j == i, (i + 1) % n, j)
    return i.to(torch.int32), j.to(torch.int32)


def _network(rng):
    parts = [rng.normal(0, math.sqrt(2 / 16), 128 * 16), rng.normal(0, 0.1, 128),
             rng.normal(0, math.sqrt(2 / 128), 128 * 128), rng.normal(0, 0.1, 128),
             rng.normal(0, math.sqrt(1 / 128), 128), rng.normal(0, 0.1, 1)]
    return np.concatenate(parts).astype(np.float32)


def _examples(case, gen, dev):
    """Raw features and labels shaped like a collection's."""
    n = case["examples"]
    y = torch.rand(n, generator=gen, device=dev) < case["positive"]
    r = torch.randn(n, 16, generator=gen, device=dev)
    la = torch.exp(r[:, 3] * 0.5 + 5.6)
    lb = la * torch.exp(r[:, 4].abs() * torch.where(y, 0.05, 0.6))
    cols = [torch.where(y, 2 + (r[:, 0].abs() * 9).floor(), 2 + (r[:, 0].abs() * 0.6).floor()),
            r[:, 1] * torch.where(y, 0.04, 0.5), r[:, 2].abs() * torch.where(y, 0.02, 0.4), torch.log(la),
            torch.log(lb), la / lb]
    cols += [r[:, 6 + g].abs() * torch.where(y, 0.012, 0.03) for g in range(10)]
    X = torch.stack(cols, 1).float().contiguous()
    order = torch.randperm(n, generator=gen, device=dev).to(torch.int32)
    return X, y.to(torch.uint8), order


def _graph(case, gen, dev):
    """Sorted edges as the search writes them (i and j set), and the families."""
    n, size = case["vertices"], case["size"]
    in_fam = max(0, n - case["singles"])
    fam = torch.full((n,), -1, dtype=torch.int64, device=dev)
    perm = torch.randperm(n, generator=gen, device=dev)
    fam[perm[:in_fam]] = torch.arange(in_fam, device=dev) // size
    a, b = torch.triu_indices(size, size, 1, device=dev)
    base = torch.arange(0, in_fam, size, device=dev)[:, None]
    u, v = (base + a).reshape(-1), (base + b).reshape(-1)
    ok = (v < in_fam) & (torch.rand(u.numel(), generator=gen, device=dev) < case["keep"])
    u, v = perm[u[ok]], perm[v[ok]]
    # a few edges between families, which merge some of them
    extra = max(1, n // 500)
    x, z = (torch.randint(0, n, (extra,), generator=gen, device=dev) for _ in range(2))
    u, v = torch.cat([u, x[x != z]]), torch.cat([v, z[x != z]])
    key = torch.unique(torch.minimum(u, v) * n + torch.maximum(u, v))
    edges = torch.zeros(key.numel(), 12, dtype=torch.int32, device=dev)
    edges[:, 0] = (key // n).to(torch.int32)
    edges[:, 1] = (key % n).to(torch.int32)
    return edges, fam.to(torch.int32)


def _params(case):
    return P.Params(k=case["k"], n_subs=case.get("subs", 0), ck_min=case["ck"], align_mode=case.get("mode", "sw"),
                    weight_mode=case.get("weight", "ani"), graph_mode=case.get("graph", False))


def _chance_pairs(case):
    """About how many unrelated pairs share a k-mer (an effective alphabet of 17 residues)."""
    n = case["families"] * case["size"] + case.get("singles", 0)
    return 0.5 * (n * case["mean"]) ** 2 / 17.0 ** case["k"]


def _family_pairs(case):
    return case["families"] * case["size"] * (case["size"] - 1) // 2


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    kind = case["kind"]
    state = {"kind": kind}
    if kind in ("search", "align", "filter"):
        state["res"], state["off"], label = _sequences(case, gen, dev)
    if kind == "search":
        state["ctx"] = P.Context(_params(case))
        # the program's own table, which the edges of each search go into
        rows = _family_pairs(case) * 2 + 4096 + (int(4 * _chance_pairs(case)) if case["weight"] == "ns" else 0)
        state["edges"] = np.zeros(rows, dtype=P.EDGE_DTYPE)
    elif kind == "align":
        state["ctx"] = P.Context(P.Params(align_mode=case["mode"], full_records=case["full"]))
        state["i"], state["j"] = _pairs(case, label, gen, dev)
        if case["mode"] == "xd":
            # one seed near the middle of the shorter sequence of each pair
            i, j = state["i"].long(), state["j"].long()
            lens = state["off"][1:] - state["off"][:-1]
            p = torch.minimum(lens[i], lens[j]) // 2 - 3
            state["seed1"] = ((p << 16) | p).to(torch.int32)
    elif kind == "filter":
        ctx = state["ctx"] = P.Context(_params(case))
        ctx.mlp_set(_network(np.random.default_rng(int(seed))), MEAN, STD)
        state["candidates"] = ctx.discover(state["res"], state["off"])
        # tables for the candidates' features and logits
        rows = _family_pairs(case) + 4096 + int(3 * _chance_pairs(case))
        state["X"] = torch.zeros(rows, 16, device=dev)
        state["logits"] = torch.zeros(rows, device=dev)
    elif kind == "epoch":
        state["ctx"] = P.Context()
        state["X"], state["y"], state["order"] = _examples(case, gen, dev)
        state["net"] = _network(np.random.default_rng(int(seed)))
        state["batch"] = case["batch"]
        state["weight"] = (1 - case["positive"]) / case["positive"]
    else:
        state["ctx"] = P.Context()
        edges, state["family"] = _graph(case, gen, dev)
        state["edges"] = edges.view(torch.uint8).reshape(-1)
        state["n"] = case["vertices"]
    return state


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "search":
        found = ctx.search(state["res"], state["off"])
        state["edges"][: found.size] = found
        # 48-byte edges as 12 words each: positions, counts and the weights' bits
        return {"count": found.size, "edges": state["edges"].view(np.int32)}
    if kind == "align":
        return ctx.align_pairs(state["res"], state["off"], state["i"], state["j"], state.get("seed1")).view(torch.int32)
    if kind == "filter":
        n = state["candidates"]
        X = ctx.mlp_features(state["res"], state["off"], n)
        state["X"][:n] = X
        state["logits"][:n] = ctx.mlp_forward(X)
        return {"count": n, "features": state["X"], "logits": state["logits"]}
    if kind == "epoch":
        ctx.mlp_set(state["net"], MEAN, STD)
        loss = ctx.mlp_train_epoch(state["X"], state["y"], state["order"], state["batch"], 1e-3, state["weight"])
        return {"loss": loss, "params": ctx.mlp_get()["params"]}
    label = ctx.components(state["edges"], state["n"])
    precision, recall = ctx.cluster_scores(label, state["family"])
    return {"label": label, "precision": precision, "recall": recall}


# ---------------------------------------------------------------- what a pass cannot do without


def work(case):
    kind = case["kind"]
    if kind in ("search", "align", "filter"):
        n = case["families"] * case["size"] + case.get("singles", 0)
        residues = n * case["mean"]
        if case.get("long", 0.0) > 0:
            residues += n * case["long"] * 15000
        # mean of a product of two members' lengths (lognormal, sigma 0.6)
        cells = case["mean"] ** 2 * math.exp(0.36)
        if case.get("long", 0.0) > 0:
            cells += case["long"] * 15000.0 ** 2
        family_pairs = _family_pairs(case)
    if kind == "search":
        # the sequences in, the family pairs' edges out; their DP cells at 11
        # operations each, in x-drop those of a band of about 22 rows
        if case["mode"] == "xd":
            cells = 22.0 * case["mean"]
        return {"bytes": residues + 8.0 * n + 48.0 * family_pairs, "flops": 11.0 * cells * family_pairs}
    if kind == "align":
        if case["mode"] == "xd":
            cells = 22.0 * case["mean"]
        return {"bytes": residues + 8.0 * n + 56.0 * case["pairs"], "flops": 11.0 * cells * case["pairs"]}
    if kind == "filter":
        # chance matches of k-mers dominate the candidates
        pairs = family_pairs + _chance_pairs(case) / (1 if case["ck"] == 1 else 50)
        return {"bytes": residues + 8.0 * n + pairs * (20 + 64 + 64 + 4), "flops": 2.0 * 18560 * pairs}
    if kind == "epoch":
        return {"bytes": case["examples"] * 69.0 + 18817 * 4 * 2, "flops": 6.0 * 18560 * case["examples"]}
    m = case["keep"] * (case["vertices"] - min(case["vertices"], case["singles"])) * (case["size"] - 1) / 2
    return {"bytes": 48.0 * m + 3 * 4.0 * case["vertices"], "flops": 0.0}


# ---------------------------------------------------------------- 64-bit values


def _exact_candidates(case, res, off):
    """Exact k-mer candidates in plain torch: (lo, hi, count, seed1, seed2) sorted by (lo, hi)."""
    dev, k = res.device, case["k"]
    code = torch.zeros(256, dtype=torch.int64, device=dev)
    for c, a in enumerate(ALPHABET):
        code[ord(a)] = c
    x = code[res.long()]
    n, m = off.numel() - 1, x.numel()
    seq = torch.repeat_interleave(torch.arange(n, device=dev), off[1:] - off[:-1])
    g = torch.arange(m, device=dev)
    g = g[g + k <= off[seq + 1]]
    kid = torch.zeros_like(g)
    for t in range(k):
        kid = kid * 20 + x[g + t]
    # first occurrence of each (k-mer, sequence): g is ascending, the sort stable
    key, perm = torch.sort(kid * n + seq[g], stable=True)
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    g, key = g[perm][first], key[first]
    kid, s = key // n, key % n
    pos = g - off[s]
    # all pairs inside a k-mer's group: entry e meets the later ones of its group
    _, cnt = torch.unique_consecutive(kid, return_counts=True)
    end = torch.repeat_interleave(torch.cumsum(cnt, 0), cnt)
    e = torch.arange(kid.numel(), device=dev)
    later = end - e - 1
    a = torch.repeat_interleave(e, later)
    b = a + 1 + torch.arange(a.numel(), device=dev) - torch.repeat_interleave(_starts(later)[:-1], later)
    pair = s[a] * n + s[b]  # sequences ascend inside a group
    seed = (pos[a] << 16) | pos[b]
    o = torch.argsort(seed, stable=True)
    o = o[torch.argsort(pair[o], stable=True)]
    pair, seed = pair[o], seed[o]
    up, count = torch.unique_consecutive(pair, return_counts=True)
    at = torch.cumsum(count, 0) - count
    s1 = seed[at]
    s2 = torch.where(count > 1, seed[(at + 1).clamp(max=seed.numel() - 1)], torch.full_like(s1, -1))
    ok = count >= case["ck"]
    return (up // n)[ok], (up % n)[ok], count[ok], s1[ok], s2[ok]


def _exact_features(case, res, off):
    lo, hi, count, s1, s2 = _exact_candidates(case, res, off)
    n, dev = off.numel() - 1, res.device
    lens = off[1:] - off[:-1]
    seq = torch.repeat_interleave(torch.arange(n, device=dev), lens)
    group = torch.full((256,), 10, dtype=torch.int64, device=dev)
    for q, members in enumerate(GROUPS):
        for a in members:
            group[ord(a)] = q
    comp = torch.bincount(seq * 11 + group[res.long()], minlength=11 * n).reshape(n, 11)[:, :10].double()
    comp = comp / lens.clamp(min=1)[:, None]
    swap = lens[hi] < lens[lo]
    a, b = torch.where(swap, hi, lo), torch.where(swap, lo, hi)
    la, lb = lens[a].double(), lens[b].double()

    def diagonal(s):
        d = ((s & 0xFFFF) - (s >> 16)).double()
        return torch.where(swap, -d, d)

    d1, d2 = diagonal(s1), diagonal(s2)
    two = s2 >= 0
    cols = [count.double(), d1 / lb, torch.where(two, (d2 - d1).abs() / lb, torch.zeros_like(lb)), la.log(), lb.log(),
            la / lb]
    return torch.cat([torch.stack(cols, 1), (comp[a] - comp[b]).abs()], 1)


def _split(theta):
    W1, b1, W2, b2, w3, b3 = torch.split(theta, [2048, 128, 16384, 128, 128, 1])
    return W1.reshape(128, 16), b1, W2.reshape(128, 128), b2, w3, b3


def _logits(theta, Z):
    W1, b1, W2, b2, w3, b3 = _split(theta)
    return torch.relu(torch.relu(Z @ W1.T + b1) @ W2.T + b2) @ w3 + b3


def exact(case, seed):
    kind = case["kind"]
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    if kind in ("search", "align"):
        return None  # whole numbers only
    net = _network(np.random.default_rng(int(seed)))
    mean = torch.tensor(MEAN, dtype=torch.float32, device=dev).double()
    std = torch.tensor(STD, dtype=torch.float32, device=dev).double()
    if kind == "filter":
        res, off, _ = _sequences(case, gen, dev)
        F = _exact_features(case, res, off)
        theta = torch.from_numpy(net).double().to(dev)
        y = torch.cat([_logits(theta, (f - mean) / std) for f in F.split(1 << 18)])
        rows = _family_pairs(case) + 4096 + int(3 * _chance_pairs(case)) - y.numel()
        pad = torch.nn.functional.pad
        return {"count": None, "features": pad(F, (0, 0, 0, rows)), "logits": pad(y, (0, rows))}
    if kind == "epoch":
        X, y, order = _examples(case, gen, dev)
        theta = torch.from_numpy(net).double().to(dev)
        weight = (1 - case["positive"]) / case["positive"]
        m, v, losses = torch.zeros_like(theta), torch.zeros_like(theta), []
        for step, idx in enumerate(order.long().split(case["batch"]), 1):
            t = theta.clone().requires_grad_(True)
            z = _logits(t, (X[idx].double() - mean) / std)
            lab = y[idx].double()
            sp = torch.nn.functional.softplus
            loss = (weight * lab * sp(-z) + (1 - lab) * sp(z)).mean()
            (g,) = torch.autograd.grad(loss, t)
            losses.append(float(loss))
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            theta = theta - 1e-3 * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
        return {"loss": float(np.mean(losses)), "params": theta.cpu().numpy()}
    edges, fam = _graph(case, gen, dev)
    n = case["vertices"]
    i, j = edges[:, 0].long(), edges[:, 1].long()
    lab = torch.arange(n, device=dev)
    while True:  # smallest label among neighbours, then pointer jumping
        new = lab.scatter_reduce(0, i, lab[j], "amin").scatter_reduce(0, j, lab[i], "amin")
        new = new[new]
        if torch.equal(new, lab):
            break
        lab = new
    own = torch.where(fam >= 0, fam.long(), n + torch.arange(n, device=dev))
    up, cnt = torch.unique(lab * (2 * n) + own, return_counts=True)
    best_c = torch.zeros(n, dtype=torch.int64, device=dev).scatter_reduce(0, up // (2 * n), cnt, "amax")
    best_f = torch.zeros(2 * n, dtype=torch.int64, device=dev).scatter_reduce(0, up % (2 * n), cnt, "amax")
    return {"label": None, "precision": float(best_c.sum()) / n, "recall": float(best_f.sum()) / n}
