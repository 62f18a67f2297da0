"""tgl_gather by words, byte for byte against torch indexing: row widths from
one 16-byte word to the largest, and slot counts whose words end before, at
and after a wavefront's span (256 words) and a block's (1024), alone and as
several tables of different widths in one call, whole and cut by a count."""
import pytest

import paper_2203_14883_amd as P
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("words", [1, 2, 3, 25, 63, 64, 65, 255, 256, 257, 4096])
def test_spans(words):
    torch = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(words)

    def table(rows, w):
        return torch.randint(-2**31, 2**31 - 1, (rows, 4 * w), generator=gen, device="cuda", dtype=torch.int32)

    for total in (1, 255, 256, 257, 1023, 1024, 1025, 5000, 70_001):
        n = max(1, total // words) if total > words else 1
        if n * words > 400_000:
            continue
        rows = 37
        nbr = torch.randint(-3, rows + 3, (n,), generator=gen, device="cuda", dtype=torch.int32)
        eid = torch.randint(-3, rows + 3, (n,), generator=gen, device="cuda")
        tabs = [(table(rows, words), "node"), (table(rows - 5, 7), "edge"), (table(rows, words), "edge")]
        for cnt in (None, 0, n // 2, n + 5):
            announce("words %d slots %d count %s" % (words, n, cnt))
            outs = [torch.full((n, t.shape[1]), 77, dtype=torch.int32, device="cuda") for t, _ in tabs]
            count = None if cnt is None else torch.tensor([cnt], device="cuda")
            P.gather(nbr, eid, tabs, count=count, outs=outs)
            m = n if cnt is None else min(n, cnt)
            for (t, key), o in zip(tabs, outs):
                k = (nbr if key == "node" else eid).long()[:m]
                ok = (k >= 0) & (k < t.shape[0])
                want = torch.where(ok[:, None], t[k.clamp(0, t.shape[0] - 1)], 0)
                assert torch.equal(o[:m], want) and bool((o[m:] == 77).all())


def test_counted_blocks():
    """A call with a count runs on a bounded number of blocks (6144 for eight
    tables, of 1024 words a round): one word more than they cover in a round, and
    counts from none to all."""
    torch = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(1)
    words, rows, n = 64, 1000, 6144 * 1024 // 64 + 1

    def table(w):
        return torch.randint(-2**31, 2**31 - 1, (rows, 4 * w), generator=gen, device="cuda", dtype=torch.int32)

    nbr = torch.randint(-3, rows + 3, (n,), generator=gen, device="cuda", dtype=torch.int32)
    eid = torch.randint(-3, rows + 3, (n,), generator=gen, device="cuda")
    tabs = [(table(words), "node"), (table(words), "edge")] + [(table(1 + i), "node") for i in range(6)]
    for cnt in (0, 1, 17, n // 2, n - 1, n, n + 5):
        announce("count %d of %d" % (cnt, n))
        outs = [torch.full((n, t.shape[1]), 77, dtype=torch.int32, device="cuda") for t, _ in tabs]
        P.gather(nbr, eid, tabs, count=torch.tensor([cnt], device="cuda"), outs=outs)
        m = min(n, cnt)
        for (t, key), o in zip(tabs, outs):
            k = (nbr if key == "node" else eid).long()[:m]
            want = torch.where(((k >= 0) & (k < rows))[:, None], t[k.clamp(0, rows - 1)], 0)
            assert torch.equal(o[:m], want) and bool((o[m:] == 77).all())
