"""CSR construction by parts (csr_parts.hip) at the edges of its sizes: one
bucket, one and two digits, buckets at the capacities of the sorting kernels and
beyond them, long runs of equal arcs, ids beside the general sort's. The result
equals the host builder's byte for byte."""
import numpy as np
import pytest

from paper_1209_6308_amd import graphs, triad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no HIP device")
    return t


def _check(torch, n, src, dst, skip=0):
    # skip > 0: the arrays start at an address that is a multiple of 4 only
    pad = np.zeros(skip, np.int32)
    ds = torch.from_numpy(np.concatenate([pad, src.astype(np.int32)])).cuda()[skip:]
    dd = torch.from_numpy(np.concatenate([pad, dst.astype(np.int32)])).cuda()[skip:]
    off, nbr, flg = triad.csr_from_arcs(n, ds, dd)
    want = graphs.build_csr(n, src.astype(np.int32), dst.astype(np.int32))
    assert np.array_equal(off.cpu().numpy(), want.offsets)
    assert np.array_equal(nbr.cpu().numpy(), want.nbrs)
    assert np.array_equal(flg.cpu().numpy(), want.flags)


# arcs from one tile's last entry on; ids that fill their bit width and not;
# 2^11 entries a bucket: 1,024 arcs one bucket, 1,025 two, 2^20 + 1 two digits
@pytest.mark.parametrize("n,narcs", [(2, 1), (7, 700), (1000, 1024), (1024, 1025), (1025, 4096), (3000, 4097),
                                     (33000, 262144), (65536, 1 << 20), (65537, (1 << 20) + 1), (300001, 2500000)])
def test_sizes(torch, n, narcs):
    rng = np.random.default_rng(n + narcs)
    src, dst = rng.integers(0, n, narcs), rng.integers(0, n, narcs)
    _check(torch, n, src, dst, skip=narcs % 4)


# one row of `deg` neighbours among random arcs: at and past the capacity of the
# LDS sorts (4,096, 16,384 and 32,768 keys), past them, and nearly everything
@pytest.mark.parametrize("n,narcs,deg", [(50000, 200000, 4000), (50000, 200000, 4097), (50000, 200000, 20000),
                                         (50000, 200000, 40000), (1 << 17, 1 << 22, 16000), (1 << 17, 1 << 22, 32000),
                                         (1 << 17, 1 << 22, 40000), (1 << 17, 1 << 22, 110000), (90000, 9000, 89000)])
def test_heavy_row(torch, n, narcs, deg):
    rng = np.random.default_rng(deg)
    hub = int(rng.integers(0, n))
    others = rng.permutation(n)[:deg]
    out = rng.random(deg) < 0.5
    src = np.concatenate([rng.integers(0, n, narcs), np.where(out, hub, others)])
    dst = np.concatenate([rng.integers(0, n, narcs), np.where(out, others, hub)])
    p = rng.permutation(src.size)
    _check(torch, n, src[p], dst[p])


# runs of equal arcs, one direction and both, within and past one tile of the sort
@pytest.mark.parametrize("copies", [3, 70, 3000, 5000, 20000])
def test_repeated_arcs(torch, copies):
    rng = np.random.default_rng(copies)
    n, narcs = 1 << 16, 1 << 22
    src, dst = rng.integers(0, n, narcs), rng.integers(0, n, narcs)
    a = np.array([[5, 9], [700, 40000], [40000, 700], [65535, 0]])
    src = np.concatenate([src, np.repeat(a[:, 0], copies)])
    dst = np.concatenate([dst, np.repeat(a[:, 1], copies)])
    p = rng.permutation(src.size)
    _check(torch, n, src[p], dst[p])


# clustered ids (the heavy rows next to each other), few rows in use, the most ids
# for the entries (32-bit keys) and more than that (the general sort)
@pytest.mark.parametrize("n,lo,hi,narcs", [(1 << 20, 0, 3000, 600000), (1 << 20, 1 << 19, (1 << 19) + 999, 600000),
                                           (1 << 21, 0, 1 << 21, 1 << 20), ((1 << 21) + 1, 0, 1 << 21, 1 << 20),
                                           (1 << 23, 0, 1 << 23, 9 << 20), (1 << 22, 0, 1 << 22, 100000)])
def test_uneven_ids(torch, n, lo, hi, narcs):
    rng = np.random.default_rng(hi)
    src, dst = rng.integers(lo, hi, narcs), rng.integers(lo, hi, narcs)
    _check(torch, n, src, dst)
