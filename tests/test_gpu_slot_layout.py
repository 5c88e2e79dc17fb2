"""The parabolic face slots' own layout: rows padded to whole lines, the last x
faces in a plane of their own, unpadded rows where padding would not fit the
workspace (large boxes of a width just above a line), next to V^{n+1/2} in the
corner-coupling increments' layout; one batch whose boxes start at every
alignment, each box against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV, assert_parity, tdtype
from tests.test_gpu_parity import TOL32, TOL64

pytestmark = pytest.mark.gpu
NG = 4
BOXES3 = [(32, 12, 10), (31, 9, 8), (33, 17, 5), (64, 3, 2), (62, 64, 3), (33, 64, 40), (17, 64, 64), (1, 1, 1), (95, 7, 3)]
BOXES2 = [(32, 9, 1), (256, 5, 1), (255, 3, 1), (33, 33, 1), (1, 3, 1), (288, 2, 1)]


def state(n, dim, seed):
    rng = np.random.default_rng(seed)
    V = np.zeros((9,) + tuple(m + 2 * NG if d < dim else m for d, m in reversed(list(enumerate(n)))))
    V[0] = 1.0 + 0.3 * rng.random(V[0].shape)
    V[4] = 0.8 + 0.2 * rng.random(V[0].shape)
    for q in (1, 2, 3, 5, 6, 7):
        V[q] = 0.2 * rng.standard_normal(V[0].shape)
    return V


@pytest.mark.parametrize("layout", ["tiles", "flat"])
@pytest.mark.parametrize("precision,tol", [("fp64", TOL64), ("fp32", TOL32)])
@pytest.mark.parametrize("dim", [3, 2])
def test_every_box_matches_the_oracle(dim, precision, tol, layout):
    boxes = BOXES3 if dim == 3 else BOXES2
    h = 1.0 / 64
    kw = dict(dim=dim, recon="ppm", riemann="hlld", gamma=5.0 / 3.0, dx=(h, h, h), parabolic_mask=7, nu=2e-2, eta=1.5e-2,
              kappa_par=3e-2, kappa_perp=4e-3, tc_phi=0.3)
    oo = O.make_opts(**kw)
    ins = [O.prim2cons(oo, state(n, dim, 60 + q)) for q, n in enumerate(boxes)]
    offs = np.concatenate([[0], np.cumsum([u.size for u in ins])])
    plan = ctu.Plan(ctu.make_opts(precision=precision, **kw),
                    [((512 * q, 0, 0), n, 0, int(o)) for q, (n, o) in enumerate(zip(boxes, offs))], NG)
    plan.set_shape(tc_layout=layout)
    U = torch.from_numpy(np.concatenate([u.reshape(-1) for u in ins])).to(tdtype(precision)).to(DEV)
    out = U.clone()
    dt, ch = 2e-4, 0.5
    params = torch.tensor([dt, ch], dtype=torch.float64, device=DEV)
    rate = torch.zeros(1, dtype=torch.float64, device=DEV)
    plan.step(U, out, params, rate)
    got = out.cpu().numpy().astype(np.float64)
    for n, u, o in zip(boxes, ins, offs):
        print(n, layout, precision, flush=True)
        ref = O.step(oo, u, NG, dt, ch)[0]
        assert_parity(got[o:o + u.size].reshape(u.shape), ref, NG, dim, ch, tol, what=(n, layout))
