"""Sampling calls of every size class the launch rules tell apart, against
the oracle bit for bit: chunks of 8, 16, 32 and 64 candidates per wavefront
(one root, around a chunk, around the numbers of roots where the chunk
doubles), and the hops that take their root indices from raw counts (at most
8192 groups, with limits on their slots) or from a scan, on both sides of those
lines."""
import math

import numpy as np
import pytest

import oracle
import paper_2203_14883_amd as P
from paper_2203_14883_amd import workloads as W
from checks import assert_hops_equal
from gpu_util import announce, hops_to_numpy, require_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graphs():
    require_gpu()
    w = W.make_c2(n_users=2000, n_items=250, num_edges=40_000, seed=9)
    og = oracle.build_tcsr(w.src, w.dst, w.ts, None, w.num_nodes, True)
    args = [upload(a) for a in (w.src, w.dst, w.ts)]
    return w, og, {h: P.tcsr_build(*args, None, w.num_nodes, True, hist=h) for h in (True, False)}


def _roots(w, n):
    rng = np.random.default_rng(n)
    e = rng.integers(0, w.num_edges, n)
    x = np.where(rng.random(n) < 0.5, w.src[e], w.dst[e]).astype(np.int32)
    x[rng.random(n) < 0.02] = -1                              # out of range: only PAD
    return x, w.ts[e]


# the first hop's chunk doubles at 3072 x 16 and 3072 x 32 roots, a later
# hop's at 1024 (histories) or 3072 (search) x 32 and x 64 candidates
@pytest.mark.parametrize("n", [0, 1, 7, 8, 9, 31, 33, 63, 65, 2730, 2731, 4096, 8191, 8192, 8193, 24576, 49151,
                               49152, 98303, 98304])
@pytest.mark.parametrize("fan,mode,S,anchor,hist", [((4, 3), "uniform", 1, "own", True),
                                                    ((4, 3), "uniform", 3, "root", False),
                                                    ((3,), "recent", 3, "own", True),
                                                    ((2, 1, 2), "recent", 1, "own", True),
                                                    ((1, 2, 1), "uniform", 2, "root", True)])
def test_sizes(graphs, n, fan, mode, S, anchor, hist):
    w, og, gs = graphs
    delta = math.inf if S == 1 else 3.0e5
    x, t = _roots(w, n)
    announce("roots %d fan %s %s S=%d %s hist=%s" % (n, fan, mode, S, anchor, hist))
    got = hops_to_numpy(P.sample(gs[hist], upload(x, np.int32), upload(t, np.float32), fan, mode, S, delta, 5, 17,
                                 anchor=anchor))
    want = oracle.sample(og, x, t, fan, mode, S, delta, seed=5, root_base=17, anchor=anchor)
    assert [h["num_roots"] for h in got] == [h.num_roots for h in want]
    assert_hops_equal(got, want, "roots %d" % n)


# where the counts of few groups are scanned after all: past 512 groups and 2^18
# slots of a hop whose next one searches, past 2^34 of groups x slots with histories
@pytest.mark.parametrize("n,fan,hist", [(4096, (64, 2), False), (4096, (65, 2), False), (4097, (64, 2), False),
                                        (512, (520, 1), False), (513, (520, 1), False), (8192, (256, 1), True),
                                        (8192, (257, 1), True), (4096, (1024, 1), True), (64, (64, 64, 1), False),
                                        (64, (64, 65, 1), False)])
def test_wide_fanouts(graphs, n, fan, hist):
    w, og, gs = graphs
    x, t = _roots(w, n)
    for mode in ("uniform", "recent"):
        announce("roots %d fan %s %s hist=%s" % (n, fan, mode, hist))
        got = hops_to_numpy(P.sample(gs[hist], upload(x, np.int32), upload(t, np.float32), fan, mode, 1, math.inf, 5, 17))
        want = oracle.sample(og, x, t, fan, mode, 1, math.inf, seed=5, root_base=17)
        assert [h["num_roots"] for h in got] == [h.num_roots for h in want]
        assert_hops_equal(got, want, "roots %d fan %s" % (n, fan))
