"""T-CSR builds of edge lists in time order, which skip the sort by time,
against the oracle: times that are all different, in ties of a few, in ties
that span tiles of the merge (2048 edges) and all equal, with -0 beside +0 and
infinities; sizes around a tile; directed and undirected; both sort-key
layouts (with 2^22 nodes and signed times the fields need more than 64 bits).
A list with one edge out of order takes the full sort."""
import numpy as np
import pytest

import oracle
import paper_2203_14883_amd as P
from gpu_util import announce, require_gpu, tcsr_to_host, upload

pytestmark = pytest.mark.gpu


def _times(rng, kind, m):
    if kind == "distinct":
        t = np.sort(rng.standard_normal(m).astype(np.float32) * 1e6)
    elif kind == "few":
        t = np.sort(rng.integers(-m // 6, m // 6 + 1, m)).astype(np.float32)
    elif kind == "long":
        t = np.sort(rng.integers(-1, 2, m)).astype(np.float32)
        z = np.flatnonzero(t == 0)
        t[z[::3]] = -0.0
    elif kind == "equal":
        t = np.full(m, 3.0, np.float32)
    else:
        t = np.sort(rng.integers(0, 40, m)).astype(np.float32)
        t[: m // 3] = -np.inf
        t[m - m // 3:] = np.inf
    return t


@pytest.mark.parametrize("nodes", [37, 1 << 22])
@pytest.mark.parametrize("kind", ["distinct", "few", "long", "equal", "infinite"])
def test_chronological(kind, nodes):
    require_gpu()
    rng = np.random.default_rng(5)
    for m in (1, 2, 3, 65, 2047, 2048, 2049, 4097, 20_011) if nodes == 37 else (2, 20_011):
        src = rng.integers(0, nodes, m).astype(np.int32)
        dst = np.where(rng.random(m) < 0.1, src, rng.integers(0, nodes, m)).astype(np.int32)   # self-loops among them
        ts = _times(rng, kind, m)
        eid = rng.integers(-5, 1 << 40, m) if m % 2 else None
        for und in (True, False):
            for late in (False, True):
                t = ts.copy()
                if late:
                    if m < 2:
                        continue
                    t[m - 1] = t[0] - np.float32(1)
                    if not t[m - 1] < t[m - 2]:
                        continue
                announce("%s nodes %d edges %d undirected=%s late=%s" % (kind, nodes, m, und, late))
                g = P.tcsr_build(upload(src), upload(dst), upload(t), None if eid is None else upload(eid), nodes, und)
                got = tcsr_to_host(g)
                want = oracle.build_tcsr(src, dst, t, eid, nodes, und)
                assert np.array_equal(got.indptr, want.indptr)
                assert np.array_equal(got.nbr, want.nbr)
                assert np.array_equal(got.eid, want.eid)
                assert np.array_equal(got.ts.view(np.int32), want.ts.view(np.int32))


@pytest.mark.parametrize("m", [262_144, 262_145])
def test_histogram_sizes(m):
    """Digit histograms of 128 tiles of 4096 entries (16,384 counts, scanned by
    one block) and of one tile more (the general scan)."""
    require_gpu()
    rng = np.random.default_rng(m)
    src, dst = (rng.integers(0, 9000, m).astype(np.int32) for _ in range(2))
    ts = np.sort(rng.random(m).astype(np.float32) * 1e6)
    announce("edges %d" % m)
    got = tcsr_to_host(P.tcsr_build(upload(src), upload(dst), upload(ts), None, 9000, True))
    want = oracle.build_tcsr(src, dst, ts, None, 9000, True)
    assert np.array_equal(got.indptr, want.indptr) and np.array_equal(got.eid, want.eid)
    assert np.array_equal(got.nbr, want.nbr) and np.array_equal(got.ts, want.ts)


def test_unaligned_workspace():
    """A workspace at any multiple of 8 bytes, with the records of an edge per
    entry (a key without the neighbour, edge ids given)."""
    torch = require_gpu()
    rng = np.random.default_rng(8)
    m, nodes = 30_000, 1 << 22
    src, dst = (upload(rng.integers(0, nodes, m).astype(np.int32)) for _ in range(2))
    ts = upload(rng.standard_normal(m).astype(np.float32) * 1e6)
    eid = upload(rng.integers(-5, 1 << 40, m))
    need = P.binding.tcsr_build_workspace(m, nodes, True)
    want = P.tcsr_build(src, dst, ts, eid, nodes, True)
    for off in (8, 24, 40):
        announce("workspace offset %d" % off)
        ws = torch.empty(need + off, dtype=torch.uint8, device="cuda")[off:]
        got = P.tcsr_build(src, dst, ts, eid, nodes, True, workspace=ws)
        assert torch.equal(got.entries, want.entries) and torch.equal(got.indptr, want.indptr)


@pytest.mark.parametrize("m", [17_000_001, 34_000_003])
def test_blocks_of_several_tiles(m):
    """Lists in time order of so many edges that a block of the merge takes
    two or three tiles of 2048 in a row and carries the time that leaves one to
    the next: all times equal, a few long ties whose ends lie off the tiles'
    (most spanning whole tiles), ties of about a tile, and short ones.  Every
    field against two stable sorts on the device."""
    torch = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(m)
    nodes = 1_000_000
    src, dst = (torch.randint(0, nodes, (m,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    for ties in (1, 9, 3000, m // 2048, m // 3):
        announce("edges %d times %d" % (m, ties))
        ts = torch.randint(0, ties, (m,), generator=gen, device="cuda").sort().values.float()
        g = P.tcsr_build(src, dst, ts, None, nodes, True, hist=False)
        own = torch.cat([src, dst])
        order = torch.cat([ts, ts]).sort(stable=True).indices
        order = order[own[order].sort(stable=True).indices]
        assert torch.equal(g.nbr, torch.cat([dst, src])[order])
        assert torch.equal(g.eid, order % m)
        assert torch.equal(g.ts, torch.cat([ts, ts])[order])
        assert torch.equal(g.indptr[1:], torch.bincount(own, minlength=nodes).cumsum(0)) and int(g.indptr[0]) == 0
        del g, order, own
