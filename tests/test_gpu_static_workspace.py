"""A step on the library's static scratch leaves the plan's own workspace in
place, all of its fields: an ordinary step after it writes the plan's
workspace again, the parabolic face slots (the last field) among them."""
import pytest
import torch

from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV, tdtype

pytestmark = pytest.mark.gpu
NG = 4
FAMILIES = {
    "parabolic": dict(recon="ppm", riemann="hlld", parabolic_mask=7, nu=2e-3, eta=1e-3, kappa_par=3e-3,
                      kappa_perp=5e-4, tc_phi=0.3),
    "mt_corner": dict(recon="lin_mc", riemann="hllc", corner="mt"),
    "shock_hybrid": dict(recon="ppm", riemann="hlld", shock_eps=0.05),
}


@pytest.mark.parametrize("family", sorted(FAMILIES))
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_step_after_a_static_step_uses_the_plans_workspace(precision, family):
    n = (20, 12, 9)
    g = torch.Generator().manual_seed(7)
    V = torch.rand((9,) + tuple(m + 2 * NG for m in reversed(n)), generator=g, dtype=torch.float64) * 0.2
    V[0] += 1.0
    V[4] += 0.8
    plan = ctu.Plan(ctu.make_opts(dim=3, precision=precision, dx=(1 / 32,) * 3, **FAMILIES[family]),
                    [((0, 0, 0), n, 0, 0)], NG, workspace="caller")
    Vd = V.reshape(-1).to(tdtype(precision)).to(DEV)
    U, out = torch.empty_like(Vd), torch.zeros_like(Vd)
    plan.prim_to_cons(Vd, U)
    params = torch.tensor([1e-4, 0.5], dtype=torch.float64, device=DEV)
    rate = torch.zeros(1, dtype=torch.float64, device=DEV)
    FILL = 0xAB

    def written():
        """256-byte pieces of the workspace that a step writes, and its state"""
        plan._ws.fill_(FILL)
        out.zero_()
        plan.step(U, out, params, rate)
        torch.cuda.synchronize()
        w = plan._ws[:plan._ws.numel() // 256 * 256].reshape(-1, 256)
        return (w != FILL).any(1), out.clone()

    before, ref = written()
    assert before[int(0.68 * before.numel()):].any()  # parabolic: the face slots, from 46 of 70 planes on
    out.zero_()
    plan.step_static(U, out, params, rate)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    after, got = written()
    assert torch.equal(got, ref)
    assert torch.equal(after, before)
