"""Both sides of each rule that chooses the Helmholtz operator's kernel at N =
9..11 (element counts beside each case: workgroups of the column kernel a CU,
waves of the matrix-core kernel a SIMD).  Where both kernels or both forms of the
fused dot exist, a request computes the same bits alone (one side) and batched
with a second one (the other side).  N = 9 in fp64 arithmetic has no column form
and is held to the oracle, as is 16-bit arithmetic, whose large launches differ
from the small ones only in the kernel."""
import numpy as np
import pytest

from oracle import OracleMesh
from paper_2608_24348_amd import inputs, sem
import opbounds

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# fused dot of the velocity solves, three components.  N = 9: blocks of five waves
# (fp64, fp32) up to 768 blocks, then single waves with the dots in scratch: 720
# and 780; 16-bit arithmetic stays with the column kernel.  N = 10, fp32: 3 (768
# blocks) and 4 workgroups a CU (777); fp64: 2 (507) and 3 (516)
@pytest.mark.parametrize("N,nel,other,tiers", [(9, (12, 10, 10), (4, 5, 5), ("fp64", "fp32b", "fp32b+fp16", "fp32b+fp16c", "fp32b+bf16c")),
                                               (10, (8, 8, 8), (2, 3, 1), ("fp32b", "fp32b+bf16")),
                                               (10, (13, 13, 2), (2, 3, 1), ("fp64",))])
def test_velocity_steps_alone_and_batched(N, nel, other, tiers):
    for tier in tiers:
        def ctx(n, nu):
            return sem.Context(sem.mesh_desc(n, N), sem.flow_desc(nu=nu, dt=1e-3, hsmg=0, vel_tol=1e-6, pres_tol=1e-2, pres_maxit=30),
                               sem.tier(tier), device="cuda:0")
        alone, pair = ctx(nel, 1.0 / 200), [ctx(nel, 1.0 / 200), ctx(other, 1.0 / 90)]
        a = sem.fluid_step([alone], 2)[0]
        b = sem.fluid_step(pair, 2)[0]
        assert [s["vit"] for s in a] == [s["vit"] for s in b] and max(a[-1]["vit"]) > 1, tier
        assert (alone.velocity() == pair[0].velocity()).all(), tier
        assert (alone.pressure() == pair[0].pressure()).all(), tier
        for c in [alone] + pair:
            c.close()


# the one-component pressure operator: N = 9, fp32 arithmetic: 1 and 2 workgroups
# (240 and 260); N = 10: 2 and 3 (480, 528, fp64), 3 and 4 (768, 800, fp32); N = 11:
# 1 and 2 (256, 260).  With Jacobi the diagonal is applied as the vector is loaded
@pytest.mark.parametrize("hsmg", [0, 1])
@pytest.mark.parametrize("N,nel,other,tiers", [(9, (10, 10, 12), (4, 5, 5), ("fp32b-p32", "fp32b+fp16pc")),
                                               (10, (8, 12, 10), (4, 4, 6), ("fp64", "fp32b", "fp32b+fp16p")),
                                               (10, (12, 16, 8), (4, 4, 4), ("fp32b-p32",)),
                                               (11, (8, 8, 8), (2, 2, 2), ("fp64", "fp32b", "fp32b-p32", "fp32b+fp16p", "fp32b+fp16pc"))])
def test_poisson_alone_and_batched(N, nel, other, tiers, hsmg):
    for tier in tiers:
        cs = [sem.Context(sem.mesh_desc(n, N), sem.flow_desc(mode=sem.MODE_POISSON, pres_tol=1e-12, pres_maxit=12, hsmg=hsmg), sem.tier(tier),
                          device="cuda:0") for n in (nel, other)]
        g = torch.Generator(device="cuda:0")
        g.manual_seed(3)
        rhs = [c.mass(torch.randn(c.np, dtype=torch.float64, device="cuda:0", generator=g)) for c in cs]
        alone, both = torch.empty_like(rhs[0]), [torch.empty_like(r) for r in rhs]
        sem.poisson_solve(cs[:1], rhs[:1], [alone])
        sem.poisson_solve(cs, rhs, both)
        assert torch.isfinite(alone).all() and torch.equal(alone, both[0]), tier
        for c in cs:
            c.close()


# one workgroup past a round of the column kernel (270 and 260) and three waves a
# SIMD against two full rounds (2560 elements: back to the column kernel)
@pytest.mark.parametrize("N,nel", [(9, (2, 26, 26)), (9, (16, 16, 10)), (11, (2, 26, 10))])
@pytest.mark.parametrize("buf,geom", [("float32", "FP16"), ("float16", "FP16"), ("float32", "BF16"), ("bfloat16", "BF16")])
def test_16bit_arithmetic_matches_oracle(N, nel, buf, geom):
    ph = inputs.deform_phases()
    c = sem.Context(sem.mesh_desc(nel, N, amp=0.1, phase=ph), sem.flow_desc(mode=sem.MODE_OPERATOR),
                    sem.tier("fp32b+%sall" % geom.lower()), device="cuda:0")
    m = OracleMesh(nel, N, amp=0.1, phase=ph)
    ut = torch.from_numpy(inputs.local_normal(nel, N, seed=5)).to("cuda:0").to(getattr(torch, buf))
    u = ut.double().cpu().numpy()
    eps16, tiny16 = {"FP16": (2.0 ** -11, 2.0 ** -25), "BF16": (2.0 ** -8, 2.0 ** -134)}[geom]
    for h1, h2 in ((1.0, 0.0), (1 / 1600, 11 / 6 / 5e-4)):
        w = torch.empty_like(ut)
        c.ax(ut, w, h1, h2, geom=getattr(sem, geom), half_compute=True)
        err = np.abs(w.double().cpu().numpy() - m.ax(u, h1, h2))
        bound = opbounds.ax16_bound(m, u, h1, h2, eps16, tiny16, eps16, 2.0 ** -24 if buf == "float32" else eps16, opbounds.TINY[buf])
        assert np.all(err <= bound), (err / bound).max()
    c.close()


# fp64 arithmetic at N = 9 is on matrix cores at every size: one element, a last
# workgroup that is not full, and more than a wave a SIMD
@pytest.mark.parametrize("nel", [(1, 1, 1), (2, 2, 2), (2, 26, 26)])
def test_fp64_at_order_9_matches_oracle(nel):
    amp = 0.1 if min(nel) > 1 else 0.0
    ph = inputs.deform_phases()
    c = sem.Context(sem.mesh_desc(nel, 9, amp=amp, phase=ph), sem.flow_desc(mode=sem.MODE_OPERATOR), sem.tier("fp64"), device="cuda:0")
    m = OracleMesh(nel, 9, amp=amp, phase=ph)
    u = inputs.local_normal(nel, 9, seed=5)
    ut = torch.from_numpy(u).to("cuda:0")
    for h1, h2 in ((1.0, 0.0), (1 / 1600, 11 / 6 / 5e-4)):
        ref = m.ax(u, h1, h2)
        w = torch.empty_like(ut)
        c.ax(ut, w, h1, h2)
        assert np.abs(w.cpu().numpy() - ref).max() < 1e-12 * np.abs(ref).max()
    c.close()
