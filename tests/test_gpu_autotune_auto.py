"""The autotuner reaches the automatic split from any shape: a plan that was
given t^n blocks far too long for its box goes back to the automatic chunk,
which no explicit candidate equals there."""
import pytest
import torch

from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV, tdtype

pytestmark = pytest.mark.gpu
NG = 4


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_tuning_returns_to_the_automatic_chunk(precision):
    n = (64, 64, 64)
    ctu.tune_cache_clear()
    plan = ctu.Plan(ctu.make_opts(dim=3, precision=precision, recon="ppm", dx=(1 / 64,) * 3), [((0, 0, 0), n, 0, 0)], NG)
    V = torch.zeros((9,) + tuple(m + 2 * NG for m in n), dtype=tdtype(precision), device=DEV)
    V[0] = 1.0 + 0.1 * torch.rand(V[0].shape, dtype=V.dtype, device=DEV)
    V[4] = 0.6
    V[5:8] = 0.3
    U = torch.empty_like(V)
    plan.prim_to_cons(V, U)
    out = torch.zeros_like(U)
    params = torch.tensor([1e-4, 0.5], dtype=torch.float64, device=DEV)
    plan.set_shape(tc_chunk=4096)
    best, _ = plan.autotune(U, out, params, reps=20)
    ctu.tune_cache_clear()
    assert best["tc_chunk"] == 0, best
