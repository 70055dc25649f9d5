"""Dealiased convection at every order: lines of lx and ceil(3 lx / 2) points in
their padded groups (rows in threes or sixes, waves of 64 lines), one element
and several, each metric storage (lane-ordered 16-bit terms up to lx = 10,
point-ordered above).  fp64 within 1e-12 of the oracle (the bar of the operator
tests); fp32 and 16-bit storage within gamma_K |terms| (+ eps16 |terms|), the
point-wise rounding bound of the operator tests."""
import numpy as np
import pytest

from oracle import OracleMesh, lxd
from paper_2608_24348_amd import inputs, sem
from test_gpu_parity import _dealias_abs_bound

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,amp", [((1, 1, 1), 0.0), ((2, 2, 2), 0.1)])
@pytest.mark.parametrize("N", range(2, 12))
def test_dealiased_convection_at_every_order(N, nel, amp):
    ph = inputs.deform_phases()
    m = OracleMesh(nel, N, amp=amp, phase=ph)
    u = np.stack([inputs.local_normal(nel, N, seed=s) for s in (12, 13, 14)])
    ref = m.conv_dealias(u)
    terms, coarse = _dealias_abs_bound(m, u), _dealias_abs_bound(m, u, floor=2.0 ** -13)
    K = 6 * (N + 1) + 3 * lxd(N + 1) + 6 + 12
    gam = K * 2.0 ** -24 / (1 - K * 2.0 ** -24)
    ud = [torch.from_numpy(u[q]).to("cuda:0") for q in range(3)]
    for tier, eps16 in (("fp64", None), ("fp32b", 0.0), ("fp32b+fp16a", 2.0 ** -11), ("fp32b+bf16a", 2.0 ** -8)):
        ctx = sem.Context(sem.mesh_desc(nel, N, amp=amp, phase=ph), sem.flow_desc(mode=sem.MODE_FLUID, dealias=1), sem.tier(tier))
        got = np.stack([g.cpu().numpy() for g in ctx.conv(ud)])
        ctx.close()
        err = np.abs(got - ref)
        if eps16 is None:
            assert err.max() < 1e-12 * np.abs(ref).max(), tier
        else:
            assert np.all(err <= gam * terms + eps16 * coarse), (tier, float((err / terms).max()))
