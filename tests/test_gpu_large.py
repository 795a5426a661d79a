"""Sizes at which other instantiations run: vertices past 2^24 (16 rows a thread),
entries past 2^29 (hubs read 32-bit lists) and past 2^30 (64-bit positions), for
one graph, labelled and in batches. Against the merge kernel; whole numbers."""
import pytest

from paper_1209_6308_amd import triad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no HIP device")
    return t


@pytest.fixture(autouse=True)
def _free():
    yield
    import torch
    torch.cuda.empty_cache()
    triad.release_memory()


def _gen(torch, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _int(torch, n, k, g):
    return torch.randint(0, n, (k,), dtype=torch.int32, device="cuda", generator=g)


def _compare(n, d):
    nnz = int(d[1].numel())
    want = triad.triad_census_device(n, nnz, *d, chunk=32768)[0]
    assert triad.triad_census_device(n, nnz, *d)[0] == want
    lab = triad.labelled_census_device(n, nnz, *d, chunk=32768)[0]
    assert triad.labelled_census_device(n, nnz, *d)[0] == lab


def test_more_than_2_24_vertices(torch):
    n, g = (1 << 24) + 12345, _gen(torch, 1)
    core = _int(torch, n, 3000, g)
    s = torch.cat([_int(torch, n, 24_000_000, g), core[_int(torch, 3000, 2_000_000, g).long()]])
    t = torch.cat([_int(torch, n, 24_000_000, g), core[_int(torch, 3000, 2_000_000, g).long()]])
    _compare(n, triad.csr_from_arcs(n, s, t))


@pytest.mark.parametrize("narcs", [290_000_000, 560_000_000])
def test_more_than_2_29_and_2_30_entries(torch, narcs):
    """Random arcs, a core of 100,000 vertices with long lists among themselves (all
    three workgroup kernels) and a thousand of high degree."""
    n, g = 1 << 23, _gen(torch, narcs)
    s, t = _int(torch, n, narcs, g), _int(torch, n, narcs, g)
    k = narcs // 10
    s[:k] = _int(torch, 100_000, k, g) * 83
    t[:k] = _int(torch, 100_000, k, g) * 83
    s[k:k + 4_000_000] = _int(torch, 1000, 4_000_000, g) * 8191
    d = triad.csr_from_arcs(n, s, t)
    del s, t
    assert d[1].numel() > (1 << 29 if narcs < 400_000_000 else 1 << 30)
    _compare(n, d)


@pytest.mark.parametrize("first", [8192, 32768])
def test_batch_of_more_than_2_30_entries(torch, first):
    """Members of 8,192 vertices, the first one also past the id-indexed tables."""
    narcs, rows, g = 560_000_000, 1 << 23, _gen(torch, first)
    s, t = _int(torch, rows, narcs, g), _int(torch, rows, narcs, g)
    # 4 M of the first member's arcs, 2 M of them among 1,000 of its vertices
    s[:4_000_000] = _int(torch, first, 4_000_000, g)
    t[:2_000_000] = _int(torch, 1000, 2_000_000, g) * (first // 1000)
    s[:2_000_000] = _int(torch, 1000, 2_000_000, g) * (first // 1000)
    inside = s < first
    t = torch.where(inside, t & (first - 1), (s & ~8191) | (t & 8191))
    del inside
    off, nbr, flg = triad.csr_from_arcs(rows, s, t)
    del s, t
    nbr[int(off[first]):] &= 8191
    sizes = torch.full(((rows - first) // 8192 + 1,), 8192, dtype=torch.int64, device="cuda")
    sizes[0] = first
    vb = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(sizes, 0)])
    size = (int(sizes.numel()), rows, int(nbr.numel()))
    assert size[2] > 1 << 30
    want = triad.triad_census_batch(*size, vb, off, nbr, flg, short_tasks=-1)
    triad.release_memory()
    assert triad.triad_census_batch(*size, vb, off, nbr, flg) == want
