"""tgl_mfg_export against the MFG block oracle, byte for byte, for hops given
as plain slot arrays: group counts around the count pass's tiles (256 groups,
and 1024 when the capacity exceeds 2^20 groups), fanouts from 1 to the most,
valid prefixes of every length, PAD slots with valid ones after them (not
exported), fewer counted groups than the capacity, hop 1 with windows and a
later hop."""
import ctypes
import types

import numpy as np
import pytest

import paper_2203_14883_amd as P
from oracle import mfg as M
from paper_2203_14883_amd import binding as B
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def _hop(rng, groups, k, roots):
    nbr = rng.integers(0, 1000, (groups, k)).astype(np.int32)
    c = rng.integers(0, k + 1, groups)
    c[rng.random(groups) < 0.4] = 0
    c[rng.random(groups) < 0.3] = k
    nbr[np.arange(k)[None, :] >= c[:, None]] = -1
    late = (rng.random(groups) < 0.1) & (c < k - 1)             # a valid slot after a PAD
    nbr[late, k - 1] = 5
    n = groups * k
    return types.SimpleNamespace(nbr=nbr.reshape(-1), eid=rng.integers(0, 1 << 40, n), num_roots=roots,
                                 ts=rng.random(n).astype(np.float32), dt=rng.random(n).astype(np.float32),
                                 parent=rng.integers(0, 50, groups))


@pytest.mark.parametrize("k", [1, 3, 10, 64, 65, 1024])
def test_tiles(k):
    torch = require_gpu()
    rng = np.random.default_rng(k)
    big = (1 << 20) + 1 if k <= 10 else 0
    for groups, cap in [(1, 1), (255, 256), (256, 256), (257, 300), (511, 1000), (1023, 1 << 20), (1025, big),
                        (2049, big), (4 * 1024 * 5 + 3, big), (big, big)]:
        if cap < groups or groups == 0 or cap * k > 12_000_000:
            continue
        for windows, prev in ((1, False), (1, True)) + (((3, False),) if groups % 3 == 0 else ()):
            announce("mfg k %d groups %d cap %d windows %d prev %s" % (k, groups, cap, windows, prev))
            roots = groups // windows
            h = _hop(rng, groups, k, roots)
            r = rng.integers(0, 99, roots).astype(np.int32)
            rt = rng.random(roots).astype(np.float32)
            p = _hop(rng, 50, 1, 50) if prev else None
            want = M.block(h, p, r, rt, windows, k)

            def dev(a, pad=0):
                t = torch.zeros(len(a) + pad, dtype=torch.from_numpy(a[:0]).dtype, device="cuda")
                t[:len(a)] = torch.from_numpy(a).cuda()
                return t

            pad = (cap - groups) * k
            hd = [dev(x, pad) for x in (h.nbr, h.eid, h.ts, h.dt)] + [dev(h.parent, cap - groups)]
            pd = [dev(x) for x in (p.nbr, p.eid, p.ts, p.dt, p.parent)] if prev else None
            rd, rtd = dev(r), dev(rt)
            count = torch.tensor([roots], device="cuda")
            out = dict(indptr=torch.empty(cap + 1, dtype=torch.int64, device="cuda"),
                       edge_dst=torch.empty(cap * k, dtype=torch.int64, device="cuda"),
                       edge_eid=torch.empty(cap * k, dtype=torch.int64, device="cuda"),
                       edge_dt=torch.empty(cap * k, device="cuda"),
                       src_nid=torch.empty(cap * (k + 1), dtype=torch.int32, device="cuda"),
                       src_ts=torch.empty(cap * (k + 1), device="cuda"),
                       sizes=torch.zeros(2, dtype=torch.int64, device="cuda"))
            ws = torch.empty(P.lib().tgl_mfg_workspace(cap), dtype=torch.uint8, device="cuda")
            ho = B.c_hop_out(*(t.data_ptr() for t in hd))
            po = B.c_hop_out(*(t.data_ptr() for t in pd)) if prev else None
            mo = B.c_mfg(*(out[f].data_ptr() for f in ("indptr", "edge_dst", "edge_eid", "edge_dt", "src_nid",
                                                       "src_ts", "sizes")))
            rc = P.lib().tgl_mfg_export(ctypes.byref(ho), ctypes.byref(po) if prev else None, rd.data_ptr(),
                                        rtd.data_ptr(), count.data_ptr(), windows, k, cap, ctypes.byref(mo),
                                        ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
            assert rc == B.OK
            G, E = out["sizes"].cpu().tolist()
            assert (G, E) == (want["G"], want["E"])
            for f, n in (("indptr", G + 1), ("edge_dst", E), ("edge_eid", E), ("edge_dt", E), ("src_nid", G + E),
                         ("src_ts", G + E)):
                assert out[f][:n].cpu().numpy().tobytes() == want[f].tobytes(), f
