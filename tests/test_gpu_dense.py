"""Graphs with long lists towards higher degrees past the ranks that a small
workgroup's table covers (65,536): around 512 entries, the sorted length 4,096
and the windows of the large table (524,288 ranks, labelled 262,144). Against
closed forms of disjoint cliques and the merge kernel. Whole numbers: equality."""
from math import comb

import pytest

from paper_1209_6308_amd import triad

from test_gpu_sweep import _census, _cliques, _lab

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no HIP device")
    return t


@pytest.mark.parametrize("sizes", [
    [1100] * 62 + [513, 514] * 40 + [2] * 100,  # a window, lists of up to 1,099
    [4200] * 17,                                # lists past the sorted length
    [700] * 760,                                # 532,000 ranks: two hash passes or two windows
    [1100] * 480,                               # 528,000 ranks: two windows
], ids=lambda s: "%dx%d" % (len(s), s[0]))
def test_cliques(torch, sizes):
    for mutual in (True, False):
        n, d = _cliques(torch, sizes, mutual)
        c = [0] * 16
        c[15 if mutual else 8] = sum(comb(k, 3) for k in sizes)
        c[2 if mutual else 1] = sum(comb(k, 2) * (n - k) for k in sizes)
        c[0] = comb(n, 3) - sum(c)
        assert _census(n, d) == c
    del d
    torch.cuda.empty_cache()


def _random(torch, n, narcs):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    s, t = (torch.randint(0, n, (narcs,), dtype=torch.int32, device="cuda", generator=g) for _ in range(2))
    return triad.csr_from_arcs(n, s, t)


@pytest.mark.parametrize("n,degree", [(70001, 1600), (131073, 2300)])
def test_random_against_the_merge(torch, n, degree):
    d = _random(torch, n, n * degree // 2)
    want = _census(n, d, chunk=32768)
    assert _census(n, d) == want
    assert _lab(n, d) == _lab(n, d, chunk=32768)


def test_labelled_windows_against_the_merge(torch):
    n = 280001
    d = _random(torch, n, n * 650)
    assert _lab(n, d) == _lab(n, d, chunk=32768)


def _concatenated(torch, sizes, arcs):
    """A batch's arrays from each member's arcs (local ids, device tensors)."""
    base = [0]
    for n in sizes:
        base.append(base[-1] + n)
    s = torch.cat([a + b for (a, _), b in zip(arcs, base)])
    t = torch.cat([a + b for (_, a), b in zip(arcs, base)])
    off, nbr, flg = triad.csr_from_arcs(base[-1], s, t)
    vb = torch.tensor(base, dtype=torch.int64, device="cuda")
    row = torch.repeat_interleave(torch.arange(base[-1], device="cuda"), off[1:] - off[:-1])
    nbr = nbr - vb[torch.searchsorted(vb, row, right=True) - 1].to(torch.int32)
    return vb, off, nbr.contiguous(), flg


@pytest.mark.parametrize("sizes", [[20011, 500, 131072], [16385, 40, 131073], [524288], [524289, 3, 20011, 1050000]])
def test_batch_members_with_dense_cores(torch, sizes):
    """Members with complete cores on ids spread over the whole member (so over
    every window of the table), of sizes around 512, 1,024 and 1,536 entries,
    random arcs around them: against the merge."""
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(sizes))
    arcs = []
    for n in sizes:
        s, t = (torch.randint(0, n, (6 * n,), dtype=torch.int32, device="cuda", generator=g) for _ in range(2))
        for k in (400, 514, 1026, 1540, 2100) if n > 16384 else ():
            core = torch.randperm(n, device="cuda", generator=g)[:k].to(torch.int32)
            core[:2] = torch.tensor([0, n - 1], dtype=torch.int32, device="cuda")
            i, j = torch.triu_indices(k, k, 1, device="cuda")
            flip = torch.rand(i.numel(), device="cuda", generator=g) < 0.5
            s = torch.cat([s, torch.where(flip, core[i], core[j])])
            t = torch.cat([t, torch.where(flip, core[j], core[i])])
        arcs.append((s, t))
    d = _concatenated(torch, sizes, arcs)
    size = (len(sizes), sum(sizes), int(d[2].numel()))
    want = triad.triad_census_batch(*size, *d, short_tasks=-1)
    assert triad.triad_census_batch(*size, *d) == want
    plan = triad.BatchPlan(*size, *d, waves_per_group=2, grid_groups=300)
    for _ in range(3):
        plan.launch()
        assert plan.result() == want
    plan.close()
