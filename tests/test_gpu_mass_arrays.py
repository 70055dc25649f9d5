"""The load vector on arrays that overlap at different offsets, below and above
each other, by one point up to almost the whole length (several blocks of the
ordered kernel, the last one partly filled), and on arrays at an odd multiple of
eight bytes, which the 16-byte words of the fused form then straddle.  Only the
place of the arrays differs from the plain call, so results agree bit for bit
(no tolerance)."""
import pytest

from paper_2608_24348_amd import sem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _ctx(nel, order):
    return sem.Context(sem.mesh_desc(nel, order), sem.flow_desc(mode=sem.MODE_OPERATOR), sem.tier("fp64"), device="cuda:0")


def _rand(n):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(4)
    return torch.randn(n, dtype=torch.float64, device="cuda:0", generator=g)


@pytest.mark.parametrize("assemble", [False, True])
@pytest.mark.parametrize("nel,order", [((2, 1, 2), 2), ((9, 4, 3), 5), ((7, 3, 2), 8)])
def test_overlapping_arrays(nel, order, assemble):
    c = _ctx(nel, order)
    f = _rand(c.np)
    want = c.mass(f, assemble=assemble)
    for d in (1, 2, 63, c.np // 3, c.np - 1):
        for lo, hi in ((0, d), (d, 0)):     # out above f, out below f
            buf = torch.zeros(c.np + d, dtype=torch.float64, device="cuda:0")
            buf[lo:lo + c.np] = f
            got = c.mass(buf[lo:lo + c.np], out=buf[hi:hi + c.np], assemble=assemble)
            assert torch.equal(got, want), (d, lo, hi)
    c.close()


@pytest.mark.parametrize("nel,order", [((5, 3, 2), 3), ((4, 3, 2), 7), ((3, 2, 2), 9), ((3, 2, 2), 11)])
def test_arrays_at_odd_offsets(nel, order):
    c = _ctx(nel, order)
    f = _rand(c.np)
    want = c.mass(f)
    for a, b in ((1, 0), (0, 1), (1, 1)):
        src = torch.zeros(c.np + 1, dtype=torch.float64, device="cuda:0")
        dst = torch.zeros(c.np + 1, dtype=torch.float64, device="cuda:0")
        src[a:a + c.np] = f
        assert torch.equal(c.mass(src[a:a + c.np], out=dst[b:b + c.np]), want), (a, b)
    c.close()
