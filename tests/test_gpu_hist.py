"""Neighbour histories against their definition (the lower bound of every
entry's time in its neighbour's run), where their kernel's branches meet: runs
of as many entries as a node record holds, a few more (with and without a
search-index slot of their own), one and several held stretches, long runs
whose times are even, all equal, or crowded into one directory cell; with a
directory, with the index only and with neither; and entry counts around a
wavefront's 64."""
import numpy as np
import pytest

import oracle
import paper_2203_14883_amd as P
from gpu_util import announce, first_hints, hist_of, require_gpu, upload

pytestmark = pytest.mark.gpu


def _times(rng, kind, m):
    if kind == "even":
        return rng.integers(0, 1 << 20, m).astype(np.float32)
    if kind == "ties":
        return rng.integers(0, 4, m).astype(np.float32)
    if kind == "equal":
        return np.full(m, 7.0, np.float32)
    t = rng.standard_exponential(m).astype(np.float32) ** 9        # nearly all in the first cells
    t[: m // 50] = np.inf                                          # and no finite span
    return t


@pytest.mark.parametrize("index,tdir", [(True, True), (False, True), (True, False), (False, False)])
@pytest.mark.parametrize("kind", ["even", "ties", "equal", "crowded"])
def test_run_lengths(kind, index, tdir):
    torch = require_gpu()
    rng = np.random.default_rng(31)
    lengths = [1, 27, 28, 29, 31, 32, 33, 60, 61, 62, 63, 64, 65, 549, 550, 5000]
    n = len(lengths) + 200
    # node i < len(lengths) owns lengths[i] edges, to random nodes; the other
    # nodes point back at them
    src = np.concatenate([np.full(c, i, np.int32) for i, c in enumerate(lengths)]
                         + [rng.integers(len(lengths), n, 4000).astype(np.int32)])
    dst = rng.integers(0, len(lengths), len(src)).astype(np.int32)
    dst[: len(src) // 3] = rng.integers(0, n, len(src) // 3)
    for und in (False, True):
        for m in (1, 63, 64, 65, len(src)):
            sel = rng.permutation(len(src))[:m] if m < len(src) else np.arange(m)
            ts = _times(rng, kind, m)
            announce("%s index=%s dir=%s undirected=%s edges %d" % (kind, index, tdir, und, m))
            g = P.tcsr_build(upload(src[sel]), upload(dst[sel]), upload(ts), None, n, und, index=index, dir=tdir)
            og = oracle.build_tcsr(src[sel], dst[sel], ts, None, n, und)
            lo, hi = hist_of(og.indptr, og.nbr, og.ts)
            got = g.hist.cpu().numpy().view(np.uint32).astype(np.int64)
            assert np.array_equal(got[:, 0], lo) and np.array_equal(got[:, 1], hi)
            assert np.array_equal(g.first_hint.cpu().numpy(), first_hints(og.indptr, og.nbr, og.ts))
    torch.cuda.synchronize()


@pytest.mark.parametrize("index,tdir", [(True, True), (True, False), (False, False)])
def test_unaligned_times(index, tdir):
    """tgl_tcsr_nodes takes timestamps at any multiple of 4 bytes: the same
    histories, directories and index from slices at 0, 4, 8 and 12 bytes."""
    torch = require_gpu()
    rng = np.random.default_rng(4)
    m, n = 60_000, 300
    src, dst = (rng.integers(0, n, m).astype(np.int32) for _ in range(2))
    g = P.tcsr_build(upload(src), upload(dst), upload(rng.random(m).astype(np.float32)), None, n, True)
    nbr, eid = P.tcsr_columns(g)
    buf = torch.empty(g.num_entries + 4, device="cuda")
    for off in range(4):
        announce("index=%s dir=%s offset %d" % (index, tdir, off))
        ts = buf[off:off + g.num_entries]
        ts.copy_(g.ts)
        c = P.tcsr_from_columns(g.indptr, nbr, ts, eid, index=index, dir=tdir)
        assert torch.equal(c.hist, g.hist) and torch.equal(c.entries, g.entries) and torch.equal(c.nodes, g.nodes)
        assert not tdir or torch.equal(c.dir, g.dir)
        assert not index or torch.equal(c.ts_index, g.ts_index)
