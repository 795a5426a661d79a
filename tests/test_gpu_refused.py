"""Graphs that break the symmetry the census rests on, at sizes where scratch is
laid out by it: refused at both levels of validation, by the device and the host
entry, with nothing written, and the next census is right."""
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


def _one_sided(n, hubs, back):
    """Every other row lists the same two hubs, whose rows list each other and `back`
    of the others: the lists towards higher degrees hold nearly all entries, in
    pairs, and one hub has a long in-list and a higher neighbour."""
    rows = np.full(n, 2, np.int64)
    rows[list(hubs)] = back + 1
    off = np.zeros(n + 1, np.int64)
    np.cumsum(rows, out=off[1:])
    nbr = np.empty(off[-1], np.int32)
    others = np.ones(n, bool)
    others[list(hubs)] = False
    at = off[:-1][others]
    nbr[at], nbr[at + 1] = hubs
    leaf = np.flatnonzero(others)
    leaf = np.concatenate([leaf[:back // 2], leaf[-(back // 2):]])
    for h, other in (hubs, hubs[::-1]):
        nbr[off[h]:off[h + 1]] = np.sort(np.append(leaf, other))
    return off, nbr, np.full((nbr.size + 3) // 4, 0x55, np.uint8)


@pytest.mark.parametrize("hubs", [(0, 1), (1600000, 1600001)])
def test_one_sided_lists_longer_than_the_packed_half(torch, hubs):
    """3.2 M rows of two entries: twice the packed units of a symmetric graph with
    as many entries. With the hubs in the middle as many entries lie above the
    diagonal as below it."""
    n = 3200002
    host = _one_sided(n, hubs, 400)
    nnz = int(host[0][-1])
    d = [torch.from_numpy(a).cuda() for a in host]
    for level in (0, 1):
        out = torch.full((17,), -5, dtype=torch.int64, device="cuda")
        with pytest.raises(triad.TriadError) as e:
            triad.triad_census_device(n, nnz, *d, d_out=out, validate=level)
        assert e.value.status == triad.EASYM
        assert bool((out == -5).all())
        with pytest.raises(triad.TriadError) as e:
            triad.triad_census(n, *host, validate=level)
        assert e.value.status == triad.EASYM
    g = graphs.rmat(14, 8, seed=2)
    assert triad.triad_census_device(g.n, g.nnz, *triad.to_device(g))[0] == oracle.census_mt(g)
