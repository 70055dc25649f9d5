"""The passes over the GMRES basis come in instances for 8, 16 and 31 vectors.
A solve picks the smallest that holds the steps run so far; one advanced piece by
piece takes the largest throughout.  Both run the same sums: iterations and
solutions agree bit for bit (no tolerance), with restarts on both sides of each
size and requests of one batch that restart at different steps."""
import pytest

from paper_2608_24348_amd import sem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier,hsmg", [("fp64", 0), ("fp32b", 0), ("fp64", 1), ("fp32b", 1)])
@pytest.mark.parametrize("restart", [1, 7, 8, 9, 16, 17, 30])
def test_instances_agree(restart, tier, hsmg):
    ctxs = [sem.Context(sem.mesh_desc(nel, 5), sem.flow_desc(mode=sem.MODE_POISSON, pres_tol=tol, pres_maxit=70, restart=restart, hsmg=hsmg),
                        sem.tier(tier), device="cuda:0") for nel, tol in (((2, 2, 2), 1e-3), ((4, 3, 5), 1e-9), ((5, 2, 4), 1e-6))]
    g = torch.Generator(device="cuda:0")
    g.manual_seed(7)
    rhs = [c.mass(torch.randn(c.np, dtype=torch.float64, device="cuda:0", generator=g)) for c in ctxs]
    one = [torch.empty_like(r) for r in rhs]
    st = sem.poisson_solve(ctxs, rhs, one)
    sem.poisson_begin(ctxs, rhs)
    for _ in range(200):
        if not any(sem.poisson_advance(ctxs, 1)):
            break
    two = [torch.empty_like(r) for r in rhs]
    piecewise = [sem.poisson_finish(c, x) for c, x in zip(ctxs, two)]
    assert [s["iters"] for s in st] == [s["iters"] for s in piecewise]
    assert [s["status"] for s in st] == [s["status"] for s in piecewise]
    for a, b in zip(one, two):
        assert torch.equal(a, b)
    for c in ctxs:
        c.close()
