"""Replayed step graphs and the table of list slots: which slot's neighbour lists a tape slot uses is decided
on the host, and a replay has to leave it as the captured call did.  After a replay whose tape slots other
calls have used with other lists in between, the backward and the retained adjoint give bitwise what a
plan without graphs gives."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state
from paper_2507_21684_amd.lib import Plan

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
SPEC = SimSpec(2, 36, amplitude=1.2)
T = 8


def _state(seed):
    return [torch.tensor(a.astype(np.float32), device=DEV) for a in make_state(SPEC, seed)]


def _plan(R, graphs, depth=T):
    p = Plan([SPEC.params()], [SPEC.n], "f32", tape_depth=depth, device=DEV, skin=0.3, rebuild_every=R)
    p.set_graphs(graphs)
    return p


class _Rollout:
    """Buffers of a rollout at fixed addresses, so that a repeated forward is a replay."""

    def __init__(self, plan, st):
        self.plan, self.st = plan, st
        self.u = [t.clone() for t in st]
        self.ck = [plan.empty_state()]
        self.cot = [torch.empty_like(t) for t in st]

    def forward(self):
        for b, a in zip(self.u, self.st):
            b.copy_(a)
        self.plan.step(*self.u, T, self.ck, T)

    def backward(self, cot=None):
        c = [torch.empty_like(t) for t in self.st] if cot is None else cot
        c[0].zero_()
        c[1].copy_(2.0 * self.u[1])
        c[2].zero_()
        self.plan.rollout_backward(self.ck, T, T, *c)
        torch.cuda.synchronize()
        return [t.clone() for t in c]


def _direct(R, st):
    r = _Rollout(_plan(R, False), st)
    r.forward()
    return r.backward()


def _equal(got, want):
    for k, (a, b) in enumerate(zip(got, want)):
        assert torch.equal(a, b), k


@pytest.mark.parametrize("R", [4, 8])
def test_backward_after_a_call_that_rebuilt_a_tape_slot(R):
    st = _state(6)
    job = _Rollout(_plan(R, True), st)
    job.forward()
    # sorts and builds in the last tape slot, whose lists the taped step shares with an earlier one
    job.plan.rhs(*[t.flip(-1).contiguous() for t in _state(7)])
    for _ in range(2):
        job.forward()
        _equal(job.backward(), _direct(R, st))   # into new cotangents: captured after the replay
    assert np.all(job.plan.poll() == 0)


def test_backward_after_another_interval():
    st = _state(8)
    job = _Rollout(_plan(2, True), st)
    job.forward()
    job.plan.set_reuse(4)
    job.forward()
    job.plan.set_reuse(2)
    job.forward()
    _equal(job.backward(), _direct(2, st))
    assert np.all(job.plan.poll() == 0)


def test_interval_changed_between_forward_and_backward():
    st = _state(9)
    job = _Rollout(_plan(4, True), st)
    job.forward()
    job.plan.set_reuse(2)
    _equal(job.backward(job.cot), _direct(4, st))   # on the tape of the other interval
    job.forward()
    _equal(job.backward(job.cot), _direct(2, st))
    job.plan.set_reuse(4)
    job.forward()
    job.plan.set_reuse(2)
    _equal(job.backward(job.cot), _direct(4, st))
    assert np.all(job.plan.poll() == 0)


def test_retained_adjoint_after_steps_that_alternate_slots():
    st = _state(10)
    plan = _plan(3, True, depth=1)
    u = [t.clone() for t in st]
    cot = lambda: [torch.full_like(t, 0.5) for t in st]
    ref = cot()
    plan.step_adjoint(*st, *ref)
    for rep in range(3):
        for b, a in zip(u, st):
            b.copy_(a)
        plan.step(*u, 1)
        c = cot()
        plan.step_adjoint(*st, *c, retained=plan.retained_lists())
        torch.cuda.synchronize()
        _equal(c, ref)
        plan.step(*_state(11), 6)   # without a tape: step 4 is in slot 0 with the lists of slot 1
    assert np.all(plan.poll() == 0)
