"""The automatic work split (x lines in runs of one pencil, y / z lines in runs
of rows, t^n chunks of 1, 2 or 4 planes) repeats the two rows below each run
with the arithmetic of the run that owns them, so the default shape is bitwise
the step with whole lines: state, CFL rate, flux registers and failure counts,
on lines that end just below, at and above the run lengths."""
import numpy as np
import pytest
import torch

from paper_1110_0740_amd import ctu, inputs as I
from tests.gpu_common import DEV, tdtype

pytestmark = pytest.mark.gpu
NG = 4
SIZES = [(1, 1), (3, 2), (253, 5), (254, 5), (255, 4), (511, 3), (1030, 6), (5, 700), (64, 63), (130, 129), (67, 3, 66),
         (256, 2, 3), (9, 257, 2)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_default_split_is_bitwise_the_whole_lines(n, precision):
    dim = len(n)
    n3 = n + (1,) * (3 - dim)
    h = 1.0 / 64
    go = ctu.make_opts(dim=dim, recon="lin_mc" if dim == 2 else "ppm", gamma=5.0 / 3.0, dx=(h, h, h),
                       precision=precision)
    # every x face plane and every y face plane of the box
    regs, slot = [], 0
    for d in range(dim):
        t = [e for e in range(3) if e != d]
        tn = (n3[t[0]], n3[t[1]])
        for f in range(n3[d] + 1):
            regs.append((0, d, f, (0, 0), tn, slot))
            slot += tn[0] * tn[1]
    shape = (9,) + tuple(m + 2 * NG if d < dim else m for d, m in reversed(list(enumerate(n3))))
    rng = np.random.default_rng(n3[0] + 7 * n3[1])
    V = np.zeros(shape)
    V[0] = 1.0 + 0.3 * rng.random(shape[1:])
    V[4] = 0.6 + 0.2 * rng.random(shape[1:])
    for q in (1, 2, 3, 5, 6, 7):
        V[q] = 0.3 * rng.standard_normal(shape[1:])
    V[4].flat[V[4].size // 2] = -0.05  # one unphysical cell: the counts of re-run rows must not add up
    plan = ctu.Plan(go, [((0, 0, 0), n3, 0, 0)], NG, regfaces=regs)
    Vd = torch.from_numpy(V.reshape(-1)).to(tdtype(precision)).to(DEV)
    U = torch.empty_like(Vd)
    plan.prim_to_cons(Vd, U)
    params = torch.tensor([1e-3, 0.5], dtype=torch.float64, device=DEV)

    def step():
        out, reg = torch.zeros_like(U), torch.zeros(9 * slot, dtype=torch.float64, device=DEV)
        rate = torch.zeros(1, dtype=torch.float64, device=DEV)
        fails = torch.zeros(5, dtype=torch.int32, device=DEV)
        plan.step(U, out, params, rate, reg=reg, fails=fails)
        torch.cuda.synchronize()
        return [x.cpu().numpy().tobytes() for x in (out, reg, rate)], fails.cpu().tolist()

    got, fails = step()
    assert sum(fails) > 0
    plan.set_shape(x_pencils=1, yz_segments=1, tc_chunk=4096)
    ref, fref = step()
    assert fails == fref
    assert got == ref
