"""The corner-coupling increments' own layout: rows padded to whole lines,
transposed strip columns, flat position order, and the unpadded rows of boxes
whose padded layout would not fit the workspace (3 ghosts, widths just above a
line), in one batch whose boxes start at every alignment; each box against the
FP64 oracle, t^n and MT corner coupling."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV, assert_parity, tdtype

pytestmark = pytest.mark.gpu
NG = 3
BOXES3 = [(40, 12, 10), (62, 9, 8), (63, 66, 5), (41, 3, 2), (64, 64, 3), (30, 5, 5), (33, 62, 4), (1, 1, 1), (31, 7, 3)]
BOXES2 = [(40, 9, 1), (254, 5, 1), (62, 3, 1), (257, 4, 1), (1, 3, 1)]


def state(n, dim, seed):
    rng = np.random.default_rng(seed)
    shape = (9,) + tuple(m + 2 * NG if d < dim else m for d, m in reversed(list(enumerate(n))))
    V = np.zeros(shape)
    V[0] = 1.0 + 0.3 * rng.random(shape[1:])
    V[4] = 0.8 + 0.2 * rng.random(shape[1:])
    for q in (1, 2, 3, 5, 6, 7):
        V[q] = 0.2 * rng.standard_normal(shape[1:])
    return V


@pytest.mark.parametrize("layout", ["auto", "tiles", "flat"])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-6)])
@pytest.mark.parametrize("dim,corner", [(3, "tn"), (3, "mt"), (2, "tn")])
def test_every_box_matches_the_oracle(dim, corner, precision, tol, layout):
    boxes = BOXES3 if dim == 3 else BOXES2
    h = 1.0 / 64
    kw = dict(dim=dim, recon="ppm", riemann="hlld", gamma=5.0 / 3.0, dx=(h, h, h), corner=corner)
    oo = O.make_opts(**kw)
    ins = [O.prim2cons(oo, state(n, dim, 40 + q)) for q, n in enumerate(boxes)]
    offs = np.concatenate([[0], np.cumsum([u.size for u in ins])])
    plan = ctu.Plan(ctu.make_opts(precision=precision, **kw),
                    [((64 * q, 0, 0), n, 0, int(o)) for q, (n, o) in enumerate(zip(boxes, offs))], NG)
    plan.set_shape(tc_layout=layout)
    U = torch.from_numpy(np.concatenate([u.reshape(-1) for u in ins])).to(tdtype(precision)).to(DEV)
    out = U.clone()
    dt, ch = 1e-3, 0.5
    params = torch.tensor([dt, ch], dtype=torch.float64, device=DEV)
    rate = torch.zeros(1, dtype=torch.float64, device=DEV)
    plan.step(U, out, params, rate)
    got = out.cpu().numpy().astype(np.float64)
    for n, u, o in zip(boxes, ins, offs):
        ref = O.step(oo, u, NG, dt, ch)[0]
        assert_parity(got[o:o + u.size].reshape(u.shape), ref, NG, dim, ch, tol, what=(n, layout))
