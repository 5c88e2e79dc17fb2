"""Failure counts of a step: those of its own input alone, whatever happened
to the plan's earlier steps, and summed over the level steps of an AMR cycle."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1110_0740_amd import ctu
from tests.gpu_common import DEV

pytestmark = pytest.mark.gpu
NG = 4


def hip_runtime():
    """the HIP runtime that this process has loaded"""
    with open("/proc/self/maps") as f:
        paths = sorted({ln.split()[-1] for ln in f if "libamdhip64.so" in ln})
    assert paths
    return C.CDLL(paths[0])


def failing_input(plan, n, nbad):
    """a state with `nbad` ghosted cells of negative pressure"""
    V = torch.zeros((9,) + tuple(m + 2 * NG for m in reversed(n)), dtype=torch.float64)
    V[0] = 1.0
    V[4] = 0.6
    V[5] = 0.3
    V[4].view(-1)[:nbad] = -0.1
    Vd = V.reshape(-1).to(DEV)
    U = torch.empty_like(Vd)
    plan.prim_to_cons(Vd, U)
    return U


def make_plan(n, **kw):
    return ctu.Plan(ctu.make_opts(dim=3, precision="fp64", recon="lin_mc", dx=(1 / 32,) * 3, **kw),
                    [((0, 0, 0), n, 0, 0)], NG)


@pytest.mark.parametrize("kw", [{}, {"corner": "mt", "riemann": "hllc"}, {"parabolic_mask": 1, "nu": 1e-3}],
                         ids=["tn", "mt", "viscous"])
def test_counts_after_a_step_that_returned_an_error(kw):
    """An error that another call left in the thread makes a step return
    early, with some of its kernels queued; the next step counts only its own
    failures."""
    n = (12, 10, 8)
    plan = make_plan(n, **kw)
    U = failing_input(plan, n, 5)
    out = torch.zeros_like(U)
    params = torch.tensor([1e-4, 0.5], dtype=torch.float64, device=DEV)
    rate = torch.zeros(1, dtype=torch.float64, device=DEV)
    fails = torch.zeros(5, dtype=torch.int32, device=DEV)
    plan.step(U, out, params, rate, fails=fails)
    ref = fails.cpu().tolist()
    assert ref[1] >= 5
    assert hip_runtime().hipSetDevice(4096) != 0
    try:
        plan.step(U, out, params, rate, fails=fails)
    except ctu.CtuError:
        pass
    torch.cuda.synchronize()
    plan.step(U, out, params, rate, fails=fails)
    assert fails.cpu().tolist() == ref


def test_own_and_static_workspace_keep_separate_counts():
    """Steps on the plan's workspace and on the static scratch, queued on two
    streams, touch no common memory."""
    n = (16, 12, 10)
    plan = make_plan(n)
    Ua, Ub = failing_input(plan, n, 3), failing_input(plan, n, 700)
    params = torch.tensor([1e-4, 0.5], dtype=torch.float64, device=DEV)

    def buffers():
        return (torch.zeros_like(Ua), torch.zeros(1, dtype=torch.float64, device=DEV),
                torch.zeros(5, dtype=torch.int32, device=DEV))

    oa, ra, fa = buffers()
    ob, rb, fb = buffers()
    plan.step(Ua, oa, params, ra, fails=fa)
    plan.step_static(Ub, ob, params, rb, fails=fb)
    refa, refb = fa.cpu().tolist(), fb.cpu().tolist()
    assert refa[1] >= 3 and refb[1] >= 700
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(50):
        plan.step(Ua, oa, params, ra, fails=fa, stream=sa)
        plan.step_static(Ub, ob, params, rb, fails=fb, stream=sb)
        sa.synchronize()
        sb.synchronize()
        assert fa.cpu().tolist() == refa and fb.cpu().tolist() == refb


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_cycle_sums_the_counts_of_its_level_steps(precision):
    """One cell of negative pressure per level: the cycle's counts are the sum
    of those of its level steps, counted one by one on the same inputs, and
    what was in the buffer before."""
    from tests import test_gpu_amr_cycle as T
    h = T.hierarchy()
    U, offs = T.level_states(h)
    dt0 = 0.2 / h.base
    ch = 0.4 * h.dx(0)[0] / dt0 * 0.5
    clean, fails, missing, _ = T.run_gpu_cycle(h, U, offs, precision, dt0, ch)
    assert fails == [0] * 5 and missing == 0
    # a cell in the middle of the first box of the finest level, whose own
    # steps see it: 2^(nlev-1) level steps at least
    lev = len(h.levels) - 1
    u = U[lev][0]
    k, j, i = (s // 2 for s in u.shape[1:])
    u[4, k, j, i] = 0.1 * u[4, k, j, i]
    one_levels = [T.run_gpu_cycle(h, U, offs, precision, dt0, ch, ncycles=c)[1] for c in (1, 2)]
    c1, c2 = np.array(one_levels[0]), np.array(one_levels[1])
    assert c1[1] >= 1
    # the state after the first cycle is the second one's start: counted alone
    state, _, _, _ = T.run_gpu_cycle(h, U, offs, precision, dt0, ch)
    second = np.array(T.run_gpu_cycle(h, state, offs, precision, dt0, ch)[1])
    assert (c2 == c1 + second).all(), (c1, second, c2)
