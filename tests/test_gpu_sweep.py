"""The triangle-listing census (the default call) where its kernels change
path: tile and table edges, rows that cross tiles, list lengths around the
sorted sizes, ranks past the workgroup tables. Against the oracle, closed forms
of disjoint cliques, and the merge kernel (which an explicit chunk selects).
Every count is a whole number: equality."""
from math import comb

import numpy as np
import pytest

import oracle
from paper_1209_6308_amd import graphs, triad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no HIP device")
    return t


def _census(n, d, **kw):
    return triad.triad_census_device(n, int(d[1].numel()), *d, **kw)[0]


@pytest.mark.parametrize("edges", [1, 2, 2047, 2048, 2049, 4096, 6145])
def test_tile_edges(torch, edges):
    """A hub and a path: 2 * edges entries around multiples of the 4,096-entry
    tile, the hub's row ending in, at and past tile boundaries, first or last."""
    rng = np.random.default_rng(edges)
    for hub_first in (True, False):
        n = edges + 2
        hub = 0 if hub_first else n - 1
        k = max(1, edges * 2 // 3)
        leaf = (np.arange(k) + 1) % n if hub_first else np.arange(k)
        rest = edges - k
        s = np.concatenate([np.full(k, hub), (np.arange(rest) + 1) % (n - 1)]).astype(np.int32)
        t = np.concatenate([leaf, (np.arange(rest) + 2) % (n - 1)]).astype(np.int32)
        flip = rng.random(edges) < 0.4
        g = graphs.build_csr(n, np.where(flip, t, s), np.where(flip, s, t), recip_p=0.3, recip_seed=3)
        assert _census(n, triad.to_device(g)) == oracle.census(g)


@pytest.mark.parametrize("n", [16383, 16384, 16385, 65536, 65537])
def test_table_edges(torch, n):
    """Around the largest graph whose tables are indexed by id, and around the
    ranks of the workgroup tables; ids at both ends carry the dense part."""
    rng = np.random.default_rng(n)
    core = np.concatenate([np.arange(150), np.arange(n - 150, n)])
    s = np.concatenate([rng.choice(core, 30000), rng.integers(0, n, 60000)]).astype(np.int32)
    t = np.concatenate([rng.choice(core, 30000), rng.choice(core, 60000)]).astype(np.int32)
    g = graphs.build_csr(n, s, t, recip_p=0.2, recip_seed=1)
    d = triad.to_device(g)
    got = _census(n, d)
    assert got == oracle.census_mt(g)
    assert got == _census(n, d, chunk=32768)


def _cliques(torch, sizes, mutual):
    """Disjoint cliques: complete, or transitive (arcs to the higher id)."""
    off, nbr, flg, base = [], [], [], 0
    for k in sizes:
        i = torch.arange(k, device="cuda", dtype=torch.int32)
        y = i[None, :].expand(k, k)[~torch.eye(k, dtype=torch.bool, device="cuda")].view(k, k - 1)
        up = y > i[:, None]
        nbr.append((y + base).reshape(-1))
        flg.append((torch.where(up, 1, 2) if not mutual else torch.full_like(y, 3)).to(torch.uint8).reshape(-1))
        off.append(torch.full((k,), k - 1, dtype=torch.int64, device="cuda"))
        base += k
    deg = torch.cat(off)
    offs = torch.zeros(base + 1, dtype=torch.int64, device="cuda")
    offs[1:] = torch.cumsum(deg, 0)
    f = torch.cat(flg)
    f = torch.nn.functional.pad(f, (0, -f.numel() % 4)).view(-1, 4)
    return base, (offs, torch.cat(nbr), f[:, 0] | (f[:, 1] << 2) | (f[:, 2] << 4) | (f[:, 3] << 6))


@pytest.mark.parametrize("mutual", [True, False])
@pytest.mark.parametrize("sizes", [
    [64, 65, 66, 67, 256, 257, 258, 514, 515] + [3] * 6000,  # lists around 64, 256 and 512 entries
    [4097, 4098, 200] + [2] * 5000,                          # lists past the sorted length (4,096)
    [600] * 130,                                             # 78,000 ranks, lists of up to 599
    [40] * 3000 + [300] * 10,
])
def test_cliques(torch, sizes, mutual):
    n, d = _cliques(torch, sizes, mutual)
    c = [0] * 16
    c[15 if mutual else 8] = sum(comb(k, 3) for k in sizes)
    c[2 if mutual else 1] = sum(comb(k, 2) * (n - k) for k in sizes)
    c[0] = comb(n, 3) - sum(c)
    assert _census(n, d) == c


@pytest.mark.parametrize("case", [("rmat", 15, 12), ("rmat", 17, 8), ("chung_lu", 90001, 20), ("chung_lu", 300007, 9)])
def test_against_the_merge(torch, case):
    kind, a, b = case
    g = graphs.rmat(a, b, seed=4, recip_p=0.25) if kind == "rmat" else graphs.chung_lu(a, 2.1, float(b), a / 16.0, seed=2)
    d = triad.to_device(g)
    want = _census(g.n, d, chunk=32768)
    for _ in range(2):  # ranks of equal degrees fall differently from run to run
        assert _census(g.n, d) == want
    assert _census(g.n, d, validate=1) == want


@pytest.mark.parametrize("n,k", [(20000, 2700), (600000, 2700), (900000, 1300)])
def test_packed_lists(torch, n, k):
    """A complete core of k vertices with arcs of all kinds (lists of every
    length up to its size, in blocks of 8 and groups of 64 entries) among
    sparse ones: packed by few and by many vertices at a time, and, with fewer
    entries, not packed."""
    rng = np.random.default_rng(n)
    core = rng.permutation(n)[:k]
    i, j = np.triu_indices(k, 1)
    kind = rng.integers(0, 3, i.size)
    s = np.concatenate([core[i[kind != 1]], core[j[kind != 0]], rng.integers(0, n, 100000)])
    t = np.concatenate([core[j[kind != 1]], core[i[kind != 0]], rng.choice(core, 100000)])
    g = graphs.build_csr(n, s.astype(np.int32), t.astype(np.int32))
    d = triad.to_device(g)
    want = _census(n, d, chunk=32768)
    assert _census(n, d) == want
    assert _census(n, d, validate=1) == want


@pytest.mark.parametrize("n", [900, 40000])
def test_one_sided_csr_is_refused(torch, n):
    """Entries above and below the diagonal that do not pair up."""
    off = np.zeros(n + 1, np.int64)
    off[1:] = 2
    off[n // 2:] = 4
    nbr = np.array([3, 5, 7, n - 1], np.int32)
    flg = np.array([0b01010101], np.uint8)
    d = [torch.from_numpy(a).cuda() for a in (off, nbr, flg)]
    for kw in ({}, {"validate": 1}, {"chunk": 32768}):
        with pytest.raises(triad.TriadError) as e:
            triad.triad_census_device(n, 4, *d, **kw)
        assert e.value.status == triad.EASYM


def test_batch_members_of_all_sizes(torch):
    """Members around a tile and beyond the id-indexed tables (hash tables of
    N+, filled in parts where it is longer than 512), empty and tiny ones
    between them; the same members without the large one (id-indexed tables)."""
    rng = np.random.default_rng(8)

    def core(n, k, m):  # k vertices densely connected, m arcs into them
        c = rng.choice(n, k, replace=False)
        s = np.concatenate([rng.choice(c, k * k), rng.integers(0, n, m)])
        t = np.concatenate([rng.choice(c, k * k), rng.choice(c, m)])
        return graphs.build_csr(n, s.astype(np.int32), t.astype(np.int32), recip_p=0.2, recip_seed=2)

    none = np.zeros(0, np.int32)
    small = [graphs.rmat(6, 4, seed=s) for s in range(40)] + [graphs.build_csr(3, none, none), core(2500, 60, 9000),
             graphs.from_arcs(2, [(1, 0)]), core(16384, 200, 20000), graphs.build_csr(0, none, none), core(70, 30, 200)]
    for members in (small, small[:20] + [core(20011, 900, 40000)] + small[20:]):
        B = graphs.concat_csrs(members)
        d = triad.batch_to_device(B)
        want = [oracle.census_mt(g) if g.n > 1000 else oracle.census(g) for g in members]
        nv = int(B.vbase[-1])
        assert triad.triad_census_batch(B.G, nv, B.nnz, *d) == want
        assert triad.triad_census_batch(B.G, nv, B.nnz, *d, short_tasks=-1) == want
        plan = triad.BatchPlan(B.G, nv, B.nnz, *d, waves_per_group=1, grid_groups=7, kernel_variant=2)
        for _ in range(3):
            plan.launch()
            assert plan.result() == want
        plan.close()


def _lab(n, d, **kw):
    return triad.labelled_census_device(n, int(d[1].numel()), *d, **kw)[0]


@pytest.mark.parametrize("edges", [1, 2047, 2049, 6145, 20000])
def test_labelled_rows_across_tiles(torch, edges):
    """Rows of one hub over several tiles, the hub's id at either end or in the
    middle (its entries then lie below and above it), all flags mixed."""
    rng = np.random.default_rng(edges + 1)
    n = edges + 3
    for hub in (0, n // 2, n - 1):
        leaf = rng.permutation(np.delete(np.arange(n), hub))[:edges * 3 // 4 + 1]
        extra = rng.integers(0, n, (2, edges // 4 + 1))
        s = np.concatenate([np.full(leaf.size, hub), extra[0]]).astype(np.int32)
        t = np.concatenate([leaf, extra[1]]).astype(np.int32)
        flip = rng.random(s.size) < 0.5
        g = graphs.build_csr(n, np.where(flip, t, s), np.where(flip, s, t), recip_p=0.3, recip_seed=3)
        assert _lab(n, triad.to_device(g)) == oracle.labelled_census(g)


@pytest.mark.parametrize("case", [("rmat", 9, 12), ("rmat", 14, 10), ("rmat", 15, 12), ("chung_lu", 90001, 20)])
def test_labelled_against_the_merge(torch, case):
    kind, a, b = case
    g = graphs.rmat(a, b, seed=4, recip_p=0.25) if kind == "rmat" else graphs.chung_lu(a, 2.1, float(b), a / 16.0, seed=2)
    d = triad.to_device(g)
    assert _lab(g.n, d) == _lab(g.n, d, chunk=32768)


@pytest.mark.parametrize("sizes", [[64, 257, 514, 3, 3, 700], [4100, 30] + [2] * 13000, [600] * 120])
def test_labelled_cliques(torch, sizes):
    n, d = _cliques(torch, sizes, False)  # transitive: every triple a < b < c has arcs a->b, a->c, b->c
    c = _lab(n, d)
    want = sum(comb(k, 3) for k in sizes)
    assert c[21] == want
    assert sum(c) == comb(n, 3)
    assert all(c[s] == 0 for s in range(64) if s not in (0, 1, 4, 16, 21))


def _updated(n, s, d, ops):
    """Arcs after the operations (source, target, insert), in order."""
    arcs = set(zip(s.tolist(), d.tolist()))
    for a, b, i in ops:
        (arcs.add if i else arcs.discard)((a, b))
    a = np.array(sorted(arcs), np.int32).reshape(-1, 2)
    return a[:, 0], a[:, 1]


def _check_update(torch, n, s, d, ops):
    g = graphs.build_csr(n, s, d)
    s, d = g.arcs()
    t = [torch.tensor([o[i] for o in ops], dtype=torch.uint8 if i == 2 else torch.int32, device="cuda") for i in range(3)]
    dev = triad.to_device(g)
    got, new, changed = triad.census_update(n, g.nnz, *dev, oracle.census_mt(g), *t)
    want = graphs.build_csr(n, *_updated(n, s, d, ops))
    assert got == oracle.census_mt(want)
    for x, y in zip(new, (want.offsets, want.nbrs, want.flags)):
        assert np.array_equal(x.cpu().numpy(), y)
    none = triad.census_update(n, g.nnz, *dev, oracle.census_mt(g), *t, new_csr=False)
    assert none[0] == got and none[1] is None and none[2] == changed


@pytest.mark.parametrize("k", [1, 31, 32, 33, 2047, 2048, 2049, 5000])
def test_update_batch_sizes(torch, k):
    """Around the batches that one workgroup sorts; repeated operations on few
    vertices, so that runs of operations and shared changed rows occur."""
    rng = np.random.default_rng(k)
    n = 700
    s, d = rng.integers(0, n, 6000), rng.integers(0, n, 6000)
    keep = s != d
    ops = []
    while len(ops) < k:
        a, b = (int(x) for x in rng.integers(0, n if len(ops) % 3 else 40, 2))
        if a != b:
            ops.append((a, b, int(rng.random() < 0.5)))
    _check_update(torch, n, s[keep].astype(np.int32), d[keep].astype(np.int32), ops)


def test_update_long_rows(torch):
    """Two rows of 5,000 shared neighbours (their pair is searched in parts) that
    change, and a row that gains and loses thousands of neighbours in a few
    tiles of the new CSR (more changes than a tile stages)."""
    rng = np.random.default_rng(3)
    n = 9000
    leaf = rng.permutation(np.arange(3, n))
    s = np.concatenate([np.full(6000, 0), np.full(6000, 1), np.full(3000, 2), rng.integers(3, n, 4000)])
    d = np.concatenate([leaf[:6000], leaf[1000:7000], leaf[:3000], rng.integers(3, n, 4000)])
    keep = s != d
    ops = [(0, 1, 1), (1, 0, 1)] + [(2, int(x), 0) for x in leaf[:2500]] + [(int(x), 2, 1) for x in leaf[3000:8000]]
    ops += [(0, int(x), 0) for x in leaf[:40]] + [(int(x), 1, 1) for x in leaf[1000:1040]]
    order = rng.permutation(len(ops))
    _check_update(torch, n, s[keep].astype(np.int32), d[keep].astype(np.int32), [ops[i] for i in order])
    _check_update(torch, n, s[keep].astype(np.int32), d[keep].astype(np.int32), ops[:2])


@pytest.mark.parametrize("scale", [8, 15])
def test_host_entry_finds_what_the_host_check_finds(torch, scale):
    """Faulty host arrays, one and several faults at a time, at both levels of
    validation: the host-pointer entry returns the status of triad_validate_host."""
    g = graphs.rmat(scale, 6, seed=2, recip_p=0.2)
    rows = np.flatnonzero(np.diff(g.offsets) >= 3)
    rng = np.random.default_rng(scale)

    def unsorted(off, nb, fl, r):
        b = off[r]
        nb[b], nb[b + 1] = nb[b + 1], nb[b]

    def loop(off, nb, fl, r):
        nb[off[r]:off[r + 1]] = np.sort(np.concatenate([[r], nb[off[r]:off[r + 1]][1:]]))

    def wild(off, nb, fl, r):
        nb[off[r] + 1] = g.n + 7 if r % 2 else -3

    def noflag(off, nb, fl, r):
        fl[off[r] >> 2] = 0

    def onesided(off, nb, fl, r):
        fl[off[r] >> 2] ^= 1 << (2 * (off[r] & 3)) if (fl[off[r] >> 2] >> (2 * (off[r] & 3)) & 3) != 1 else 3 << (2 * (off[r] & 3))

    def offsets(off, nb, fl, r):
        off[r] = off[r + 1] + 1

    faults = [unsorted, loop, wild, noflag, onesided, offsets]
    for i, f in enumerate(faults):
        for h in [None] + faults[i:]:
            off, nb, fl = g.offsets.copy(), g.nbrs.copy(), g.flags.copy()
            f(off, nb, fl, int(rng.choice(rows)))
            if h is not None:
                h(off, nb, fl, int(rng.choice(rows)))
            for level in (0, 1):
                want = triad.triad_validate_host(g.n, off, nb, fl, level)
                if want == triad.OK:  # level 0 does not look at symmetry; the census refuses uneven sides
                    continue
                with pytest.raises(triad.TriadError) as e:
                    triad.triad_census(g.n, off, nb, fl, validate=level)
                assert e.value.status == want, (f.__name__, h and h.__name__, level)
    assert triad.triad_census(g.n, g.offsets, g.nbrs, g.flags, validate=1) == oracle.census_mt(g)


@pytest.mark.parametrize("sizes", [
    [2] * 9000, [3] * 7000, [2, 3, 4, 5] * 4000,  # many rows of an in-list of one or two
    [16, 17, 18, 19] * 300,                       # N+ around 16 entries: 16 or 8 rows at once
    [31, 32, 33, 34, 35] * 150,                   # around 32, in-lists up to the workgroups'
    [64, 65, 66, 128, 129, 130] * 60,             # around 64 and 128: four, two rows, one
    [1, 2, 40, 3, 100, 2, 300, 17] * 60,          # all mixed
], ids=lambda s: "%dx%d" % (len(s), s[0]))
def test_rows_taken_together(torch, sizes):
    """Vertices with short in-lists, as many of which share a wavefront as their
    lists towards higher degrees allow."""
    n, d = _cliques(torch, sizes, False)
    want = [0] * 16
    want[8], want[1] = sum(comb(k, 3) for k in sizes), sum(comb(k, 2) * (n - k) for k in sizes)
    want[0] = comb(n, 3) - sum(want)
    assert n > 16384
    assert _census(n, d) == want
    lab = _lab(n, d)
    assert lab[21] == want[8] and sum(lab) == comb(n, 3)
    assert all(lab[s] == 0 for s in range(64) if s not in (0, 1, 4, 16, 21))


@pytest.mark.parametrize("shape", ["path", "grid", "tree"])
def test_low_degrees_against_the_merge(torch, shape):
    rng = np.random.default_rng(5)
    n = 60000
    i = np.arange(n)
    if shape == "path":
        s, t = i[:-1], i[1:]
    elif shape == "grid":
        s, t = np.concatenate([i[i % 300 > 0], i[300:]]), np.concatenate([i[i % 300 > 0] - 1, i[300:] - 300])
    else:
        s, t = i[1:], (rng.random(n - 1) * i[1:]).astype(np.int64)
    extra = rng.integers(0, n, 20000)  # some triangles
    s, t = np.concatenate([s, extra]), np.concatenate([t, np.minimum(extra + 2, n - 1)])
    p = rng.permutation(n)
    flip = rng.random(s.size) < 0.5
    g = graphs.build_csr(n, p[np.where(flip, t, s)].astype(np.int32), p[np.where(flip, s, t)].astype(np.int32),
                         recip_p=0.2, recip_seed=1)
    d = triad.to_device(g)
    assert _census(n, d) == _census(n, d, chunk=32768) == oracle.census_mt(g)
    assert _lab(n, d) == _lab(n, d, chunk=32768)


def test_batch_rows_taken_together(torch):
    """Members above and below the id-indexed tables one after another, so that the
    64 rows a wavefront looks at belong to several: rows of all list lengths."""
    rng = np.random.default_rng(12)
    members = []
    for n in (17000, 5, 30, 9, 20000, 1, 300, 16500, 40, 2):
        k = min(n, 150)
        core = rng.permutation(n)[:k]
        s = np.concatenate([rng.choice(core, 2 * k), rng.integers(0, n, 3 * n)])
        t = np.concatenate([rng.choice(core, 2 * k), rng.integers(0, n, n), rng.choice(core, 2 * n)])
        members.append(graphs.build_csr(n, s.astype(np.int32), t.astype(np.int32), recip_p=0.2, recip_seed=2))
    B = graphs.concat_csrs(members * 2)
    d = triad.batch_to_device(B)
    want = [oracle.census_mt(g) for g in members] * 2
    assert triad.triad_census_batch(B.G, int(B.vbase[-1]), B.nnz, *d) == want
    plan = triad.BatchPlan(B.G, int(B.vbase[-1]), B.nnz, *d, waves_per_group=1, grid_groups=5, kernel_variant=1)
    for _ in range(2):
        plan.launch()
        assert plan.result() == want
    plan.close()
