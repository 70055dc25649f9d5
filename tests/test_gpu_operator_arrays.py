"""Standalone operators on caller arrays: where the arrays allow it the kernels
read and write them in place of staging copies, and the load vector is formed
in one pass.  Both routes run the same arithmetic, so they must agree bit for
bit (no tolerance)."""
import ctypes as C

import pytest

from paper_2608_24348_amd import inputs, sem

pytestmark = pytest.mark.gpu


def _ctx(nel, order, mode, deform=False, tier="fp64", dealias=0):
    mesh = sem.mesh_desc(nel, order, amp=0.1 if deform else 0.0, phase=inputs.deform_phases())
    return sem.Context(mesh, sem.flow_desc(mode=mode, dealias=dealias, restart=1), sem.tier(tier), device="cuda:0")


def _rand(n, seed):
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device="cuda:0", generator=g)


def _ptrs(ts):
    return (C.c_void_p * 3)(*[C.c_void_p(t.data_ptr()) for t in ts])


# every word size and form of the gather-scatter (even and odd rows, planes and
# rows), one element along a direction, several segments along x
@pytest.mark.parametrize("nel,order", [((1, 1, 1), 2), ((2, 1, 3), 3), ((5, 3, 2), 4), ((9, 2, 3), 5), ((1, 2, 2), 7),
                                       ((33, 2, 2), 7), ((17, 3, 2), 8), ((5, 4, 3), 9), ((3, 2, 2), 10), ((7, 2, 3), 11)])
def test_mass_one_pass_equals_two(nel, order):
    import torch
    ctx = _ctx(nel, order, sem.MODE_OPERATOR)
    f = _rand(ctx.np, 3)
    two = ctx.dssum(ctx.mass(f, assemble=False))
    one = ctx.mass(f, assemble=True)
    assert torch.equal(one, two)
    same = f.clone()
    ctx.mass(same, out=same, assemble=True)   # in place
    assert torch.equal(same, two)
    buf = torch.zeros(ctx.np + 2, dtype=torch.float64, device="cuda:0")
    buf[:ctx.np] = f
    ctx.mass(buf[:ctx.np], out=buf[2:], assemble=True)   # overlapping ranges: two passes
    assert buf.shape[0] == ctx.np + 2 and torch.isfinite(buf).all()
    ctx.close()


@pytest.mark.parametrize("nel,order,tier,dealias", [((2, 2, 2), 5, "fp64", 0), ((3, 2, 5), 7, "fp32b", 0), ((2, 4, 2), 7, "fp32b", 1),
                                                    ((3, 1, 2), 9, "fp64", 1), ((2, 3, 1), 11, "fp64", 0), ((2, 2, 1), 11, "fp64", 1)])
def test_direct_arrays_equal_staged(nel, order, tier, dealias):
    import torch
    ctx = _ctx(nel, order, sem.MODE_FLUID, tier=tier, dealias=dealias)
    L = sem.load()
    u = [_rand(ctx.np, 10 + q) for q in range(3)]
    kept = [t.clone() for t in u]
    before = ctx.velocity()
    conv, grad, div = ctx.conv(u), ctx.opgrad(u[0]), ctx.wdiv(u)
    assert all(torch.equal(a, b) for a, b in zip(u, kept))   # inputs untouched
    # outputs on top of inputs take the staged route
    v = [t.clone() for t in u]
    assert L.sem_conv(ctx.h, _ptrs(v), _ptrs(v)) == 0
    assert all(torch.equal(a, b) for a, b in zip(v, conv))
    v = [t.clone() for t in u]
    assert L.sem_opgrad(ctx.h, C.c_void_p(v[0].data_ptr()), _ptrs(v)) == 0
    assert all(torch.equal(a, b) for a, b in zip(v, grad))
    v = [t.clone() for t in u]
    assert L.sem_wdiv(ctx.h, _ptrs(v), C.c_void_p(v[1].data_ptr())) == 0
    assert torch.equal(v[1], div)
    assert (ctx.velocity() == before).all()   # the context's own velocity is kept
    ctx.close()
