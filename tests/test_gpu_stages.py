"""Multistage steps whose later stages are formed and packed in one pass (list reuse), at a workgroup's
edges and for one and several simulations: schemes of one to four stages, the taped backward that steps
from one tape state into the next, and the same without a skin, where every stage is sorted.  Tolerances:
the path's accuracy targets against the FP64 oracle (gradients 1e-3 of the largest in FP32, 1e-9 in FP64)."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state
from paper_2507_21684_amd.lib import Plan

pytestmark = pytest.mark.gpu

EULER = ([[0.0]], [1.0])
RK3 = ([[0, 0, 0], [0.5, 0, 0], [-1.0, 2.0, 0]], [1 / 6, 2 / 3, 1 / 6])


@pytest.mark.parametrize("scheme,dtype,dim,sides,skin", [(EULER, "f32", 2, (16,), 0.1), (RK3, "f64", 2, (16, 17), 0.1),
                                                         ("rk4", "f32", 3, (14,), 0.1), ("heun", "f64", 3, (14, 15), 0.1),
                                                         (RK3, "f32", 2, (17,), 0.0)])
def test_taped_stage_gradient(orc, scheme, dtype, dim, sides, skin):
    specs = [SimSpec(dim, s, jitter=0.2) for s in sides]
    npdt, tdt = (np.float32, torch.float32) if dtype == "f32" else (np.float64, torch.float64)
    states = [[a.astype(npdt) for a in make_state(s, 50 + k)] for k, s in enumerate(specs)]
    rng = np.random.default_rng(51)
    cots = [[rng.normal(size=a.shape).astype(npdt) for a in st] for st in states]
    cat = lambda parts: [torch.tensor(np.concatenate([p[k] for p in parts], axis=-1), dtype=tdt, device="cuda")
                         for k in range(3)]
    plan = Plan([s.params() for s in specs], [s.n for s in specs], dtype, integrator=scheme, skin=skin, tape_depth=3)
    g, c = cat(states), cat(cots)
    tape = [plan.empty_state()]
    plan.step(*g, 3, tape, 3)
    plan.rollout_backward(tape, 3, 3, *c)
    assert np.all(plan.poll() == 0)
    tol = 1e-9 if dtype == "f64" else 1e-3
    off = 0
    for s, st, ct in zip(specs, states, cots):
        p = orc.Params(**s.params())
        steps = [st]
        for _ in range(2):
            steps.append(orc.step_rk(p, *steps[-1], 1, scheme))
        want = ct
        for n in (2, 1, 0):
            want = orc.step_rk_adjoint(p, *steps[n], *want, scheme)
        for got, ref in zip(c, want):
            got = got[..., off:off + s.n].cpu().numpy().astype(np.float64)
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
        off += s.n
