"""Time encoding against the 64-bit cosine where its kernels' rules meet: rows
of fewer elements than a 16-byte word, of whole words and of parts of one;
widths whose lanes' columns repeat after few or many blocks; one word, one
block and several words per lane; arguments on both sides of 2^19 turns (the
phase in a double's low word) and 2^24; PAD slots, and a count that cuts the
last rows; an output that is not 16-byte aligned.

Tolerance: 1e-6 by the entry point's contract, plus half a bfloat16 step for
bfloat16: a value in [2^e, 2^(e+1)) has steps of 2^(e-7), half of one being at
most 2^-8 of the value."""
import pytest

import paper_2203_14883_amd as P
from gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [1, 3, 4, 5, 7, 8, 9, 12, 33, 100, 101, 256, 1021, 1024, 1025, 4095, 4096])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_words(dim, dtype):
    torch = require_gpu()
    dt_ = getattr(torch, dtype)
    gen = torch.Generator(device="cuda").manual_seed(dim)
    omega = 10.0 ** (-9.0 * torch.rand(dim, generator=gen, device="cuda"))
    phi = torch.randn(dim, generator=gen, device="cuda")
    omega[0] = 1.0
    edge = 6.283185307179586 * 2.0 ** 19
    special = torch.tensor([0.0, -0.0, 1.0, edge * 0.999999, edge, edge * 1.000001, edge * 33, edge * 400, 3e38, -1.0],
                           device="cuda")
    for n in (1, 2, 3, 257, 5000, 70_001):
        if n * dim > 6_000_000:
            continue
        d = torch.empty(n, device="cuda").exponential_(1 / 3e5, generator=gen)
        d = torch.where(torch.rand(n, generator=gen, device="cuda") < 0.3, -1.0, d)
        k = min(n, len(special))
        d[:k] = special[:k]
        want = (torch.outer(d.double(), omega.double()) + phi.double()).cos()
        want = torch.where((d < 0)[:, None], 0.0, want)
        for cnt, shift in ((None, 0), (n - n // 3, 0), (None, 1)):
            announce("dim %d %s slots %d count %s shift %d" % (dim, dtype, n, cnt, shift))
            m = n if cnt is None else cnt
            off = shift * (1 if dtype == "float32" else 2)
            buf = torch.full((n * dim + off,), 77.0, dtype=dt_, device="cuda")
            out = buf[off:].view(n, dim)
            count = None if cnt is None else torch.tensor([cnt], device="cuda")
            P.time_encode(d, omega, phi, dt_, count=count, out=out)
            err = (out[:m].double() - want[:m]).abs()
            bound = 1e-6 + (want[:m].abs() * 2.0 ** -8 if dtype == "bfloat16" else 0.0)
            assert bool((err <= bound).all()), float(err.max())
            assert bool((out[m:] == 77).all())


def _ladder(torch, dim):
    return (10.0 ** (-9.0 * torch.arange(dim, dtype=torch.float64) / (dim - 1))).float().cuda()


@pytest.mark.parametrize("dim", [100, 101, 128])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_near_one(dim, dtype):
    """No value exceeds 1, and where the argument is below 0.1 rad (the slow
    columns) a float32 value is its cosine rounded once: half a step below 1
    is 2^-25 = 3.0e-8, and 1 - cos < 0.005 is summed with steps of 2^-31, so
    that 3.2e-8 bounds the error."""
    torch = require_gpu()
    gen = torch.Generator(device="cuda").manual_seed(dim)
    omega, phi = _ladder(torch, dim), torch.zeros(dim, device="cuda")
    d = torch.empty(200_000, device="cuda").exponential_(1 / 2e5, generator=gen)
    announce("dim %d %s" % (dim, dtype))
    out = P.time_encode(d, omega, phi, getattr(torch, dtype)).double()
    assert float(out.abs().max()) <= 1.0
    if dtype == "float32":
        x = torch.outer(d.double(), omega.double())
        err = (out - x.cos()).abs()
        assert float(err[x < 0.1].max()) <= 3.2e-8
        # over all arguments: a step of the float argument's rest (below 1/2
        # quarter: 2^-26 of pi / 2) and two of the result's (2^-25), at most
        assert float(err.max()) <= 2.0 ** -26 * 1.5708 + 2 * 2.0 ** -25 + 5e-9


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_value_alone(dtype):
    """An element depends on its own slot, omega and phi: the same slots in
    another order, and alone, give the same bits, small arguments beside ones
    past 2^24 turns and past 2^50 rad."""
    torch = require_gpu()
    for dim in (100, 101, 128):
        gen = torch.Generator(device="cuda").manual_seed(dim)
        omega = _ladder(torch, dim)
        phi = torch.randn(dim, generator=gen, device="cuda")
        n = 3000
        d = torch.empty(n, device="cuda").exponential_(1 / 3e5, generator=gen)
        big = torch.rand(n, generator=gen, device="cuda") < 0.05
        d = torch.where(big, d * 10.0 ** torch.randint(1, 13, (n,), generator=gen, device="cuda"), d)
        announce("dim %d %s" % (dim, dtype))
        out = P.time_encode(d, omega, phi, getattr(torch, dtype))
        perm = torch.randperm(n, generator=gen, device="cuda")
        assert torch.equal(P.time_encode(d[perm].contiguous(), omega, phi, getattr(torch, dtype)), out[perm])
        for i in (0, 1, n - 1, int(d.argmax())):
            assert torch.equal(P.time_encode(d[i:i + 1].clone(), omega, phi, getattr(torch, dtype))[0], out[i])


@pytest.mark.parametrize("dim", [33, 100, 128, 172])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_few_counted(dim, dtype):
    """Calls for many slots of which the device counts few: as many blocks as
    the counted slots need take part, from one to the most there are, and
    the counted rows hold the bits of a call for those slots alone."""
    torch = require_gpu()
    dt_ = getattr(torch, dtype)
    gen = torch.Generator(device="cuda").manual_seed(dim)
    omega, phi = _ladder(torch, dim), torch.randn(dim, generator=gen, device="cuda")
    n = 1_500_000
    d = torch.empty(n, device="cuda").exponential_(1 / 3e5, generator=gen)
    out = torch.empty(n, dim, dtype=dt_, device="cuda")
    for cnt in (0, 1, 2, 31, 4096, 4097, 50_003, 333_333, 1_499_999, n):
        announce("dim %d %s count %d" % (dim, dtype, cnt))
        out.fill_(77)
        P.time_encode(d, omega, phi, dt_, count=torch.tensor([cnt], device="cuda"), out=out)
        if cnt:
            assert torch.equal(out[:cnt], P.time_encode(d[:cnt].clone(), omega, phi, dt_))
        assert bool((out[cnt:] == 77).all())
