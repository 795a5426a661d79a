"""Work that a program using this library has it do, timed case by case.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU (on
the host for the host-pointer entry) from a seed, ``run`` is one call of the
public entry points as a program makes it, ``exact`` the same result by plain
dense or sorting arithmetic where that is affordable. Inputs are built with
torch alone (R-MAT, Chung-Lu and Erdos-Renyi digraphs; the recipes of
``paper_1209_6308_amd.graphs`` with another generator of random numbers).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1209_6308_amd import triad


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # A query on a small communication graph: the census of one host's
        # neighbourhood, called from an interactive loop. Latency and launches.
        dict(name="census_small", kind="census", model="rmat", n=1024, ef=8, recip=0.0),
        # The same in a serving loop that may not allocate (ragged size).
        dict(name="census_noalloc", kind="noalloc", model="rmat", n=13001, ef=8, recip=0.1),
        # An ordinary network of the size of the US patents (2^20 vertices,
        # 16 arcs a vertex, a tenth of the pairs mutual).
        dict(name="census_patents", kind="census", model="rmat", n=1 << 20, ef=16, recip=0.1),
        # A large social network, the size of Orkut (2^24 vertices, 268 M arcs,
        # degrees above 10^5): the benchmark workload.
        dict(name="census_social", kind="census", model="rmat", n=1 << 24, ef=16, recip=0.0),
        # A power-law network of exponent 2.1 whose vertex ids say nothing
        # about degrees (2^22 vertices, 24 arcs a vertex, hubs of 2^17).
        dict(name="census_powerlaw", kind="census", model="chunglu", n=1 << 22, ef=24, recip=0.0),
        # The 64-state census (a triple's vertices told apart by id).
        dict(name="labelled", kind="labelled", model="rmat", n=1 << 20, ef=16, recip=0.1),
        # A graph that lives in host memory, through the host-pointer entry:
        # host checks, the copy, the census (ragged size).
        dict(name="census_host", kind="host", model="rmat", n=200003, ef=16, recip=0.1),
        # A null-model ensemble censused again and again from a kept plan:
        # 4,096 graphs of 64 to 8,192 vertices, mean degree 4 to 32.
        dict(name="ensemble", kind="ensemble", graphs=4096, nmax=8192),
        # A significance profile: a new small ensemble, planned, censused and
        # reduced to z-scores in one go.
        dict(name="profile", kind="profile", graphs=256, nmax=1024),
        # The CSR built from the raw arcs of the large network (duplicates and
        # self-loops among them).
        dict(name="build_social", kind="build", model="rmat", n=1 << 24, ef=16),
        # A large network followed through time: 100,000 arc updates between
        # two censuses, with the CSR after them (ragged size).
        dict(name="update_large", kind="update", model="rmat", n=3500003, ef=16, recip=0.0, updates=100000),
        # Traffic monitoring: a small graph, a short interval's updates.
        dict(name="update_window", kind="update", model="rmat", n=3001, ef=8, recip=0.1, updates=601),
    ]


def _log_int(rng, lo, hi):
    """Whole number in [lo, hi], uniform over the logarithm, mostly odd."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, x | 1 if rng.random() < 0.7 else x))


def draw(rng):
    kind = rng.choice(["census", "census", "census", "noalloc", "labelled", "host", "ensemble", "profile", "build",
                       "update"])
    if kind == "ensemble":
        return dict(kind=kind, graphs=_log_int(rng, 16, 4096), nmax=_log_int(rng, 256, 8192))
    if kind == "profile":
        return dict(kind=kind, graphs=_log_int(rng, 16, 1024), nmax=_log_int(rng, 128, 1024))
    top = {"census": 1 << 22, "noalloc": 60000, "labelled": 1 << 21, "host": 1 << 20, "build": 1 << 23,
           "update": 3500003}[kind]
    n = _log_int(rng, 500, top)
    ef = rng.randint(4, 8) if kind == "noalloc" else rng.randint(4, 20)
    case = dict(kind=kind, model=rng.choice(["rmat", "chunglu"]) if n >= 4096 else "rmat", n=n, ef=ef)
    if kind != "build":
        case["recip"] = rng.choice([0.0, 0.1, round(rng.uniform(0.0, 0.3), 3)])
    if kind == "update":
        case["updates"] = _log_int(rng, 50, max(100, min(200000, n * ef // 20)))
    return case


# ------------------------------------------------------------------ the inputs

def _gen(seed, salt, device):
    g = torch.Generator(device=device)
    g.manual_seed((seed * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _rmat(n, m, seed):
    """R-MAT arcs (.57, .19, .19, .05), ids from n on dropped (high ids are rare)."""
    dev = _device()
    g = _gen(seed, 1, dev)
    scale = max(1, (n - 1).bit_length())
    src = torch.zeros(m, dtype=torch.int32, device=dev)
    dst = torch.zeros(m, dtype=torch.int32, device=dev)
    r = torch.empty(m, dtype=torch.float32, device=dev)
    for _ in range(scale):
        r.uniform_(generator=g)
        s = r >= 0.76
        d = ((r >= 0.57) & ~s) | (r >= 0.95)
        src.mul_(2).add_(s)
        dst.mul_(2).add_(d)
    if n != 1 << scale:
        keep = (src < n) & (dst < n)
        src, dst = src[keep], dst[keep]
    return src, dst


def _power_cdf(n, mean, top, gamma):
    """Running sum (whole numbers) of the weights top * ((i + i0) / i0)^(-1 / (gamma - 1)),
    i0 such that they have the given mean (by their integral)."""
    p = 1.0 - 1.0 / (gamma - 1.0)
    lo, hi = 1e-3, 4.0 * n
    for _ in range(60):
        i0 = math.sqrt(lo * hi)
        if top * i0 * (((n + i0) / i0) ** p - 1.0) / (n * p) < mean:
            lo = i0
        else:
            hi = i0
    i = torch.arange(n, dtype=torch.float64, device=_device())
    w = ((i + lo) / lo) ** (p - 1.0) * float(1 << 36)
    return torch.cumsum(w.to(torch.int64).clamp_(min=1), 0)


def _pick(cdf, m, g):
    r = torch.rand(m, dtype=torch.float64, device=cdf.device, generator=g) * int(cdf[-1])
    return torch.searchsorted(cdf, r.to(torch.int64), right=True).clamp_(max=cdf.numel() - 1)


def _chunglu(n, m, seed):
    """Chung-Lu arcs, exponent 2.1: sources by weight, targets by weight under a random permutation."""
    dev = _device()
    g = _gen(seed, 2, dev)
    cdf = _power_cdf(n, m / n, n / 16.0, 2.1)
    perm = torch.randperm(n, device=dev, generator=g)
    src = _pick(cdf, m, g).to(torch.int32)
    dst = perm[_pick(cdf, m, g)].to(torch.int32)
    return src, dst


def _arcs(case, seed):
    m = case["n"] * case["ef"]
    return _rmat(case["n"], m, seed) if case["model"] == "rmat" else _chunglu(case["n"], m, seed)


def _mix(key, seed):
    """A scrambled 64-bit number of each 64-bit key (one to one)."""
    x = key * -7046029254386353131 + (seed + 1) * 7919
    x = x ^ (x >> 29)
    x = x * 4600416091520132537
    return x ^ (x >> 32)


def _coin(key, seed):
    """A number in [0, 1) from each 64-bit key."""
    return (_mix(key, seed) & 0xFFFFFF).to(torch.float64) / float(1 << 24)


def _sym_pairs(base, row, col, width):
    """Sorted keys row << width | col of the symmetric closure of the arcs row -> base + col
    (self-loops and duplicates dropped; col < 2^width is the target's id within its
    graph, whose first row is base) and each entry's direction bits."""
    keep = row != base + col
    row, col = row[keep], col[keep]
    if torch.is_tensor(base):
        base = base[keep]
    key = torch.cat([((row << width) | col) << 1, (((base + col) << width) | (row - base)) << 1 | 1])
    del row, col, base, keep
    key = torch.sort(key).values
    head = torch.ones(key.numel(), dtype=torch.bool, device=key.device)
    torch.ne(key[1:], key[:-1], out=head[1:])
    key = key[head]
    pair, flag = key >> 1, (key & 1).to(torch.uint8) + 1
    del key, head
    same = pair[1:] == pair[:-1]
    flag[:-1][same] = 3
    head = torch.ones(pair.numel(), dtype=torch.bool, device=pair.device)
    torch.logical_not(same, out=head[1:])
    return pair[head], flag[head]


def _finish(pair, flag, rows, width):
    row = pair >> width
    off = torch.zeros(rows + 1, dtype=torch.int64, device=pair.device)
    torch.cumsum(torch.bincount(row, minlength=rows), 0, out=off[1:])
    nbr = (pair & ((1 << width) - 1)).to(torch.int32)
    k = flag.numel()
    f = torch.zeros((k + 3) // 4 * 4, dtype=torch.uint8, device=flag.device)
    f[:k] = flag
    f = f.view(-1, 4)
    return off, nbr, f[:, 0] | (f[:, 1] << 2) | (f[:, 2] << 4) | (f[:, 3] << 6)


def _csr_of(n, src, dst, recip=0.0, seed=0):
    width = max(1, (n - 1).bit_length())
    pair, flag = _sym_pairs(0, src.to(torch.int64), dst.to(torch.int64), width)
    if recip > 0:
        row, col = pair >> width, pair & ((1 << width) - 1)
        flag[_coin((torch.minimum(row, col) << width) | torch.maximum(row, col), seed) < recip] = 3
    return _finish(pair, flag, n, width)


def _unit(lo, hi, x):
    return min(1.0, max(0.0, (x - lo) / (hi - lo)))


def _even(case, src, dst, seed):
    """The arcs without some of their pairs, so that a model, n and ef give one number of
    edges whatever the seed (a random share of the pairs, duplicates and all, goes)."""
    n = case["n"]
    want = int(n * case["ef"] * (0.375 + 0.425 * _unit(10, 20, math.log2(n))))
    width = max(1, (n - 1).bit_length())
    s, d = src.to(torch.int64), dst.to(torch.int64)
    key = _mix((torch.minimum(s, d) << width) | torch.maximum(s, d), seed)
    loop = s == d
    del s, d
    rank = torch.sort(key[~loop]).values
    head = torch.ones(rank.numel(), dtype=torch.bool, device=rank.device)
    torch.ne(rank[1:], rank[:-1], out=head[1:])
    rank = rank[head]
    if rank.numel() <= want:
        return src, dst
    keep = (key < rank[want]) | loop
    return src[keep], dst[keep]


def _csr(case, seed):
    src, dst = _arcs(case, seed)
    if case["kind"] == "update":
        src, dst = _even(case, src, dst, seed)
    return _csr_of(case["n"], src, dst, case["recip"], seed)


def _sizes(case, seed):
    """Sizes of an ensemble's members: vertices, arcs, reciprocity."""
    r = np.random.RandomState((seed * 7 + 3) & 0x7FFFFFFF)
    n = r.randint(64, case["nmax"] + 1, case["graphs"])
    return n, (n * np.minimum(r.uniform(4, 32, n.size), n / 4)).astype(np.int64), r.uniform(0, 0.3, n.size)


def _batch(case, seed):
    """Concatenated CSR of Erdos-Renyi (even) and Chung-Lu (odd) members."""
    dev = _device()
    g = _gen(seed, 3, dev)
    n, m, recip = _sizes(case, seed)
    vbase = torch.from_numpy(np.concatenate([[0], np.cumsum(n)])).to(dev)
    nt, mt, rt = (torch.from_numpy(a).to(dev) for a in (n.astype(np.int64), m, recip))
    member = torch.repeat_interleave(torch.arange(n.size, device=dev), mt)
    nm = nt[member].to(torch.float64)
    u, v = (torch.rand(member.numel(), dtype=torch.float64, device=dev, generator=g) for _ in range(2))
    # a power of a uniform number: density of a power law of exponent 2.5 over the ranks
    bent = (member & 1).to(torch.float64) * 2.0 + 1.0
    src = (u ** bent * nm).to(torch.int64)
    dst = (v ** bent * nm).to(torch.int64)
    dst = torch.where(member % 2 == 1, (dst * 48271 + 11) % nt[member], dst)
    base = vbase[member]
    width = max(1, (case["nmax"] - 1).bit_length())
    pair, flag = _sym_pairs(base, base + src, dst, width)
    del u, v, src, dst, base, nm, bent, member
    row, col = pair >> width, pair & ((1 << width) - 1)
    who = torch.repeat_interleave(torch.arange(n.size, device=dev), nt)[row]
    loc = row - vbase[who]
    key = (torch.minimum(loc, col) << width | torch.maximum(loc, col)) * n.size + who
    flag[_coin(key, seed) < rt[who]] = 3
    del row, col, loc, key, who
    return (vbase,) + _finish(pair, flag, int(vbase[-1]), width)


def _distinct(key, k, seed):
    """k of the distinct keys, in a random order."""
    key = torch.unique(key)
    return key[torch.argsort(_mix(key, seed + 77))[:k]]


def _updates(case, seed, off, nbr, flg):
    """Arc updates: just under half delete one-way arcs (drawn by entry, so by degree), as
    many insert arcs between random unconnected vertices, the rest reverse one-way arcs."""
    dev = off.device
    g = _gen(seed, 4, dev)
    k, n = case["updates"], case["n"]
    width = max(1, (n - 1).bit_length())
    kr = k // 10
    kd = (k - kr) // 2
    ki = k - kr - kd
    at = torch.randint(0, nbr.numel(), (4 * (kd + kr),), device=dev, generator=g)
    f = flg[at >> 2].to(torch.int64) >> 2 * (at & 3) & 3
    at, f = at[f != 3], f[f != 3]
    row, col = torch.searchsorted(off, at, right=True) - 1, nbr[at].to(torch.int64)
    src, dst = torch.where(f == 1, row, col), torch.where(f == 1, col, row)
    old = _distinct(src << width | dst, kd + kr, seed)
    a = torch.randint(0, n, (4 * ki,), device=dev, generator=g)
    b = (a + torch.randint(1, n, (4 * ki,), device=dev, generator=g)) % n
    lo, hi = torch.minimum(a, b), torch.maximum(a, b)
    rows = torch.repeat_interleave(torch.arange(n, device=dev), off[1:] - off[:-1])
    pair = (rows << width) | nbr
    key = lo << width | hi
    there = pair[torch.searchsorted(pair, key).clamp_(max=pair.numel() - 1)] == key
    new = _distinct(key[~there], ki, seed)
    del rows, pair
    mask = (1 << width) - 1
    src = torch.cat([old >> width, new >> width])
    dst = torch.cat([old & mask, new & mask])
    turn = torch.zeros(src.numel(), dtype=torch.bool, device=dev)
    turn[kd:old.numel()] = True  # the arc back
    turn[old.numel():] = (_mix(new, seed) & 1) == 1
    src, dst = torch.where(turn, dst, src), torch.where(turn, src, dst)
    ins = torch.ones(src.numel(), dtype=torch.uint8, device=dev)
    ins[:kd] = 0
    p = torch.randperm(src.numel(), device=dev, generator=g)
    return src[p].to(torch.int32), dst[p].to(torch.int32), ins[p]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "ensemble":
        vb, off, nbr, flg = _batch(case, seed)
        return dict(kind=kind, plan=triad.BatchPlan(case["graphs"], off.numel() - 1, nbr.numel(), vb, off, nbr, flg))
    if kind == "profile":
        vb, off, nbr, flg = _batch(case, seed)
        real = [int(x) for x in np.random.RandomState(seed & 0x7FFFFFFF).randint(0, 1 << 20, 16)]
        return dict(kind=kind, graphs=case["graphs"], batch=(vb, off, nbr, flg), real=real)
    if kind == "build":
        src, dst = _even(case, *_arcs(case, seed), seed)
        return dict(kind=kind, n=case["n"], src=src, dst=dst)
    off, nbr, flg = _csr(case, seed)
    if kind == "host":
        return dict(kind=kind, n=case["n"], csr=tuple(t.cpu().numpy() for t in (off, nbr, flg)))
    s = dict(kind=kind, n=case["n"], csr=(off, nbr, flg))
    if kind == "update":
        s["updates"] = _updates(case, seed, off, nbr, flg)
        s["census"] = triad.triad_census_device(case["n"], nbr.numel(), off, nbr, flg)[0]
    else:
        s["out"] = torch.zeros(65 if kind == "labelled" else 17, dtype=torch.int64, device=off.device)
    return s


# --------------------------------------------------------------------- a pass

def run(s):
    kind = s["kind"]
    if kind == "ensemble":
        s["plan"].launch()
        return s["plan"].d_out
    if kind == "profile":
        vb, off, nbr, flg = s["batch"]
        plan = triad.BatchPlan(s["graphs"], off.numel() - 1, nbr.numel(), vb, off, nbr, flg)
        plan.launch()
        plan.status()
        z, sp = triad.significance_profile(plan.d_out, s["real"])
        plan.close()
        return plan.d_out, np.array(z), np.array(sp)
    if kind == "build":
        return triad.csr_from_arcs(s["n"], s["src"], s["dst"])
    if kind == "host":
        return triad.triad_census(s["n"], *s["csr"])
    off, nbr, flg = s["csr"]
    if kind == "update":
        return triad.census_update(s["n"], nbr.numel(), off, nbr, flg, s["census"], *s["updates"])
    if kind == "noalloc":
        triad.triad_census_device_noalloc(s["n"], nbr.numel(), off, nbr, flg, s["out"])
    elif kind == "labelled":
        triad.labelled_census_device(s["n"], nbr.numel(), off, nbr, flg, d_out=s["out"])
    else:
        triad.triad_census_device(s["n"], nbr.numel(), off, nbr, flg, d_out=s["out"])
    return s["out"]


def work(case):
    """Bytes: the graph (8 B a row, 4 1/4 B an entry, two entries an edge) read
    once, what the call writes written once. Operations: one an entry read."""
    kind = case["kind"]
    if kind in ("ensemble", "profile"):
        rows = case["graphs"] * (64 + case["nmax"]) / 2
        nnz = 2 * 18 * rows
        return {"bytes": 8 * rows + 4.25 * nnz + 136 * case["graphs"], "flops": nnz}
    rows, nnz = case["n"], 2.0 * case["n"] * case["ef"]
    graph = 8 * rows + 4.25 * nnz
    if kind == "build":
        return {"bytes": 8.0 * case["n"] * case["ef"] + graph, "flops": nnz}
    if kind == "update":
        return {"bytes": 2 * graph + 9 * case["updates"], "flops": nnz}
    return {"bytes": graph + 136, "flops": nnz}


# ---------------------------------------------------------------- exact values

# (mutual pairs, asymmetric pairs) and degrees name the 16 classes: the class
# of a state f_ab | f_ac << 2 | f_bc << 4 (f: bit0 = forward, bit1 = backward)
def _class_of(code):
    f = [code & 3, code >> 2 & 3, code >> 4]
    ends = [(0, 1), (0, 2), (1, 2)]
    out, inn = [0] * 3, [0] * 3
    for x, (a, b) in zip(f, ends):
        out[a] += x & 1
        inn[b] += x & 1
        out[b] += x >> 1
        inn[a] += x >> 1
    mut, asym = f.count(3), f.count(1) + f.count(2)
    names = {(0, 0): 0, (0, 1): 1, (1, 0): 2, (2, 0): 10, (2, 1): 14, (3, 0): 15}
    if (mut, asym) in names:
        return names[mut, asym]
    if (mut, asym) == (0, 2):
        return 3 if 2 in out else 4 if 2 in inn else 5
    if (mut, asym) == (1, 1):
        return 6 if 2 in inn else 7
    if (mut, asym) == (0, 3):
        return 8 if 2 in out else 9
    lone = [i for i in range(3) if f[[2, 1, 0][i]] == 3][0]  # the vertex outside the mutual pair
    return 11 if out[lone] == 2 else 12 if inn[lone] == 2 else 13


def _states(n, off, nbr, flg):
    """Triples a < b < c in each of the 64 states, by dense products in float64 (exact: below 2^53)."""
    flag = torch.stack([flg >> s & 3 for s in (0, 2, 4, 6)], 1).view(-1)[:nbr.numel()]
    row = torch.repeat_interleave(torch.arange(n, device=off.device), off[1:] - off[:-1])
    A = torch.zeros((n, n), dtype=torch.uint8, device=off.device)
    A[row, nbr.to(torch.int64)] = flag
    P = [torch.triu((A == f).to(torch.float64), 1) for f in range(4)]
    out = torch.zeros(64, dtype=torch.int64, device=off.device)
    for ab in range(4):
        for bc in range(4):
            C = P[ab] @ P[bc]
            for ac in range(4):
                out[ab | ac << 2 | bc << 4] = (C * P[ac]).sum().to(torch.int64)
    return out


def _classes(states):
    out = torch.zeros(16, dtype=torch.int64, device=states.device)
    return out.index_add_(0, torch.tensor([_class_of(c) for c in range(64)], device=states.device), states)


def _zscores(counts, real):
    """z-scores and unit profile with whole-number moments about the first member."""
    c = np.array(counts.cpu(), dtype=object)
    z = np.zeros(16)
    for t in range(16):
        d = [int(x) - int(c[0, t]) for x in c[:, t]]
        k, s1, s2 = len(d), sum(d), sum(x * x for x in d)
        var = k * s2 - s1 * s1  # k (k - 1) sd^2
        if var:
            num = k * (int(real[t]) - int(c[0, t])) - s1
            z[t] = num / math.sqrt(k * var / (k - 1)) if var < 1 << 1000 else 0.0
    sp = z.copy()
    sp[:3] = 0
    norm = math.sqrt(float((sp * sp).sum()))
    return z, sp / norm if norm else sp * 0


DENSE = 4096  # the largest graph that `_states` takes


def exact(case, seed):
    kind = case["kind"]
    if kind == "profile":
        if case["graphs"] > 512:
            return None
        s = prepare(case, seed)
        vb, off, nbr, flg = s["batch"]
        flag = torch.stack([flg >> k & 3 for k in (0, 2, 4, 6)], 1).view(-1)[:nbr.numel()]
        got, v = [], vb.tolist()
        for g in range(case["graphs"]):
            o = off[v[g]:v[g + 1] + 1]
            a, b = int(o[0]), int(o[-1])
            f = torch.zeros((b - a + 3) // 4 * 4, dtype=torch.uint8, device=flag.device)
            f[:b - a] = flag[a:b]
            f = f.view(-1, 4)
            got.append(_classes(_states(v[g + 1] - v[g], o - a, nbr[a:b],
                                        f[:, 0] | (f[:, 1] << 2) | (f[:, 2] << 4) | (f[:, 3] << 6))))
        counts = torch.stack(got)
        z, sp = _zscores(counts, s["real"])
        return counts, z, sp
    if kind == "build":
        return _csr_of(case["n"], *_even(case, *_arcs(case, seed), seed))
    if kind in ("ensemble", "update") or case["n"] > DENSE:
        return None
    states = _states(case["n"], *_csr(case, seed))
    zero = torch.zeros(1, dtype=torch.int64, device=states.device)
    if kind == "labelled":
        return torch.cat([states, zero])
    if kind == "host":
        return _classes(states).tolist()
    return torch.cat([_classes(states), zero])
