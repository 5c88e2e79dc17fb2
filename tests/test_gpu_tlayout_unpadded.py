"""3D boxes whose rows, padded to whole lines, would not fit the box's ghosted
extent: the corner-coupling increments keep the region's own row width there.
With 3 ghosts that takes widths just above a line and long y and z, or boxes of
a few cells; each box against the FP64 oracle, t^n and MT corner coupling, in
one batch with boxes that are padded."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV, assert_parity, tdtype
from tests.test_gpu_tlayout import NG, state

pytestmark = pytest.mark.gpu
UNPADDED = [(33, 62, 62), (1, 5, 8), (17, 64, 64)]
PADDED = [(40, 6, 5), (30, 7, 3)]


def padded_fits(n, esize):
    """rows of W = n0 + 2 elements padded to 128 bytes, H W-rows per plane, D planes"""
    line = 128 // esize
    W, H, D = (m + 2 for m in n)
    assert W % 32 not in (1, 2)  # no strip columns
    return -(-W // line) * line * H * D <= np.prod([m + 2 * NG for m in n])


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-6)])
@pytest.mark.parametrize("corner", ["tn", "mt"])
def test_unpadded_boxes_match_the_oracle(corner, precision, tol):
    esize = 4 if precision == "fp32" else 8
    assert not any(padded_fits(n, esize) for n in UNPADDED) and all(padded_fits(n, esize) for n in PADDED)
    boxes = [UNPADDED[0], PADDED[0], UNPADDED[1], PADDED[1], UNPADDED[2]]
    h = 1.0 / 64
    kw = dict(dim=3, recon="ppm", riemann="hlld", gamma=5.0 / 3.0, dx=(h, h, h), corner=corner)
    oo = O.make_opts(**kw)
    ins = [O.prim2cons(oo, state(n, 3, 80 + q)) for q, n in enumerate(boxes)]
    offs = np.concatenate([[0], np.cumsum([u.size for u in ins])])
    plan = ctu.Plan(ctu.make_opts(precision=precision, **kw),
                    [((128 * q, 0, 0), n, 0, int(o)) for q, (n, o) in enumerate(zip(boxes, offs))], NG)
    plan.set_shape(tc_layout="tiles")
    U = torch.from_numpy(np.concatenate([u.reshape(-1) for u in ins])).to(tdtype(precision)).to(DEV)
    out = U.clone()
    dt, ch = 1e-3, 0.5
    params = torch.tensor([dt, ch], dtype=torch.float64, device=DEV)
    rate = torch.zeros(1, dtype=torch.float64, device=DEV)
    plan.step(U, out, params, rate)
    got = out.cpu().numpy().astype(np.float64)
    for n, u, o in zip(boxes, ins, offs):
        ref = O.step(oo, u, NG, dt, ch)[0]
        assert_parity(got[o:o + u.size].reshape(u.shape), ref, NG, 3, ch, tol, what=(n, precision))
