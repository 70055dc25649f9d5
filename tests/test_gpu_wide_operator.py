"""The matrix-core Helmholtz operator of N = 9..11 runs where a launch fills
the chip, the column kernel below that.  Both give the same bits, so a request
computes the same alone (column kernel) and in a batch that fills the chip;
against the oracle the large launches meet the bounds of the small ones (with
stored fp32 or 16-bit geometry, whose rounding the bounds are made of; fp64
geometry is covered by the bitwise comparison)."""
# At N = 9 fp64 arithmetic has no column form: there both sides of the comparison
# run on matrix cores.  The one-component pressure operators of these batches stay
# with the column kernel.  test_gpu_wide_rule.py takes both, and the Jacobi forms.
import numpy as np
import pytest

from oracle import OracleMesh
from paper_2608_24348_amd import inputs, sem
import opbounds

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (N, requests of 4^3 elements whose three components pass one round of the CUs)
@pytest.mark.parametrize("N,n", [(9, 8), (10, 7), (11, 4)])
@pytest.mark.parametrize("tier", ["fp64", "fp32b"])
def test_steps_bitwise_alone_and_in_a_large_batch(N, n, tier):
    def ctx(i):
        return sem.Context(sem.mesh_desc((4, 4, 4), N), sem.flow_desc(nu=1.0 / (100 + 50 * i), dt=1e-3, hsmg=1, vel_tol=1e-6,
                                                                        pres_tol=1e-4), sem.tier(tier), device="cuda:0")
    batch = [ctx(i) for i in range(n)]
    sem.fluid_step(batch, 3)
    for i in (0, n - 1):
        alone = ctx(i)
        sem.fluid_step([alone], 3)
        assert (alone.velocity() == batch[i].velocity()).all()
        assert (alone.pressure() == batch[i].pressure()).all()
        alone.close()
    for c in batch:
        c.close()


# one element block past a round of the CUs, and a last block that is not full
@pytest.mark.parametrize("N,nel", [(9, (2, 26, 26)), (10, (10, 2, 54)), (11, (2, 26, 10))])
@pytest.mark.parametrize("tier,buf,geom,half", [("fp32b", "float64", "FP32", False),
                                                ("fp32b", "float32", "FP32", False), ("fp32b+fp16all", "float32", "FP16", False),
                                                ("fp32b+bf16all", "bfloat16", "BF16", False),
                                                ("fp32b+fp16all", "float32", "FP16", True)])
def test_large_launch_matches_oracle(N, nel, tier, buf, geom, half):
    c = sem.Context(sem.mesh_desc(nel, N, amp=0.1, phase=inputs.deform_phases()), sem.flow_desc(mode=sem.MODE_OPERATOR),
                    sem.tier(tier), device="cuda:0")
    m = OracleMesh(nel, N, amp=0.1, phase=inputs.deform_phases())
    dt = getattr(torch, buf)
    ut = torch.from_numpy(inputs.local_normal(nel, N, seed=5)).to("cuda:0").to(dt)
    u = ut.double().cpu().numpy()
    eps = {"FP32": 2.0 ** -24, "FP16": 2.0 ** -11, "BF16": 2.0 ** -8}[geom]
    out = {"float64": 2.0 ** -53, "float32": 2.0 ** -24, "bfloat16": 2.0 ** -8}[buf]
    arith = 2.0 ** -53 if buf == "float64" else 2.0 ** -24
    for h1, h2 in ((1.0, 0.0), (1 / 1600, 11 / 6 / 5e-4)):
        w = torch.empty_like(ut)
        c.ax(ut, w, h1, h2, geom=getattr(sem, geom), half_compute=half)
        err = np.abs(w.double().cpu().numpy() - m.ax(u, h1, h2))
        if half:
            bound = opbounds.ax16_bound(m, u, h1, h2, 2.0 ** -11, 2.0 ** -25, 2.0 ** -11, out, opbounds.TINY[buf])
        else:
            bound = opbounds.ax_bound(m, u, h1, h2, arith, eps, out, opbounds.TINY[buf])
        assert np.all(err <= bound), (err / bound).max()
    c.close()
