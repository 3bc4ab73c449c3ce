"""The adjoint's hand-over from step t to step t - 1 across a sort: rollouts whose tape has fewer slots than
keep the order before their sort, as many, and more, over one and several segments, against the step
adjoints one by one.  The hand-over repeats the prologue's arithmetic, so the two differ at most in how a
product and sum are contracted: one rounding (6e-8, 1.1e-16) per step, and 16 steps scale that by less than
100 here."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state
from paper_2507_21684_amd.lib import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,side,dtype,steps,depth", [(2, 33, "f32", 3, 3), (2, 33, "f32", 6, 6), (2, 33, "f32", 9, 9),
                                                        (3, 14, "f32", 14, 7), (2, 24, "f64", 12, 12),
                                                        (3, 13, "f64", 16, 8)])
def test_handover(dim, side, dtype, steps, depth):
    spec = SimSpec(dim, side, jitter=0.2)
    npdt, tdt, eps = (np.float32, torch.float32, 6e-8) if dtype == "f32" else (np.float64, torch.float64, 1.1e-16)
    rng = np.random.default_rng(61)
    x, v, rho = make_state(spec, 60)
    x = x + 0.45 * spec.dx * rng.uniform(-1, 1, size=x.shape)      # particles change cells within a few steps
    st = [a.astype(npdt) for a in (x, 3 * v, rho)]
    cot = [rng.normal(size=a.shape).astype(npdt) for a in st]
    gpu = lambda arrs: [torch.tensor(a, dtype=tdt, device="cuda").contiguous() for a in arrs]
    plan = Plan([spec.params()], [spec.n], dtype, tape_depth=depth)
    g = gpu(st)
    states = []
    for _ in range(steps):
        states.append([t.clone() for t in g])
        plan.step(*g, 1)
    want = gpu(cot)
    for s in reversed(states):
        plan.step_adjoint(*s, *want)
    g = gpu(st)
    nseg = (steps + depth - 1) // depth
    ck = [plan.empty_state() for _ in range(nseg)]
    plan.step(*g, steps, ck, depth)
    for _ in range(2):   # on the forward's tape where it holds every step, then recomputed or again
        got = gpu(cot)
        plan.rollout_backward(ck, steps, depth, *got)
        for a, b in zip(got, want):
            assert float((a - b).abs().max()) <= 100 * steps * eps * float(b.abs().max())
        plan.rhs(*g)     # overwrites a slot
    assert np.all(plan.poll() == 0)
