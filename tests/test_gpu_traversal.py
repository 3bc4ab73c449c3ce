"""The sweeps' walk over the list rows, where it changes: rows shorter than a turn and one entry either
side of 8, 16 and 32 positions, list widths that end in half a group of 16 with rows reaching into it,
2, 4 and 8 lanes per particle, wavefronts inside the box and at its faces, exact lists and lists with a
skin, and plans large enough to run four lanes for eight.  The adjoint of two steps within one reuse
interval hands its cotangents on in sorted order.  Tolerances: the accuracy targets of the path against
the FP64 oracle (rates 1e-4 and gradients 1e-3 of the largest in FP32, 1e-9 in FP64; densities 1e-5 and
1e-10); lanes and widths change nothing, bitwise."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state

pytestmark = pytest.mark.gpu

# (dim, side, support factor, dtype): mean entries of a row about 6, 12, 16, 32, 50, 100 (2D), 8, 17,
# 34, 65, 270 (3D)
CASES = [(2, 24, 1.4, "f32"), (2, 24, 1.9, "f64"), (2, 26, 2.25, "f32"), (2, 24, 3.2, "f32"), (2, 20, 4.0, "f64"),
         (2, 30, 5.6, "f32"), (3, 12, 1.25, "f32"), (3, 12, 1.6, "f64"), (3, 14, 2.0, "f32"), (3, 13, 2.5, "f32"),
         (3, 13, 4.0, "f64"), (2, 182, 2.6, "f32")]


def _err(a, ref):
    a, ref = np.atleast_2d(a).astype(np.float64), np.atleast_2d(ref)
    return np.sqrt(((a - ref) ** 2).sum(axis=0)).max() / np.sqrt((ref ** 2).sum(axis=0)).max()


@pytest.mark.parametrize("dim,side,sf,dtype", CASES)
def test_traversal(orc, dim, side, sf, dtype):
    from paper_2507_21684_amd.lib import Plan
    spec = SimSpec(dim, side, support_factor=sf, jitter=0.2)
    npdt, tdt = (np.float32, torch.float32) if dtype == "f32" else (np.float64, torch.float64)
    rng = np.random.default_rng(11)
    x, v, rho = make_state(spec, 6)
    rho = rho * (1 + 0.01 * rng.uniform(-1, 1, size=rho.shape))
    st = [a.astype(npdt) for a in (x, v + 0.2 * rng.normal(size=v.shape), rho)]
    cot = [rng.normal(size=a.shape).astype(npdt) for a in st]
    gpu = lambda arrs: [torch.tensor(a, dtype=tdt, device="cuda").contiguous() for a in arrs]
    p = orc.Params(**spec.params())
    off, _ = orc.neighbors(st[0].astype(np.float64), spec.box, spec.H, dtype)
    pairs = int(off[-1])
    need = int(np.diff(off).max()) + 1   # the widest row, the particle itself included if it is not in off
    first = None
    # (list width, lanes, skin): the smallest width that holds every row, and half a group more
    for width, lanes, skin in ((need, 2, 0.0), (need + 8, 4, 0.0), (need, 8, 0.0), (need + 8, 8, 0.0), (need, 4, 0.0),
                               (0, 2, 0.2), (0, 4, 0.2), (0, 8, 0.2)):
        plan = Plan([spec.params()], [spec.n], dtype, max_neighbors=width, skin=skin, rebuild_every=2 if skin else 1)
        plan.set_tuning(lanes, lanes)
        g = gpu(st)
        out = list(plan.rhs(*g))
        if skin:
            plan.pair_count()
            plan.rhs(*g)
            counted = plan.pair_count()
            assert counted in (pairs, pairs - spec.n)   # the particle itself is not a pair
        c = gpu(cot)
        plan.step_adjoint(*g, *c)
        a = [t.clone() for t in g]
        tape = [plan.empty_state()]
        plan.step(*a, 2, tape, 2)
        c2 = gpu(cot)
        plan.rollout_backward(tape, 2, 2, *c2)
        out = [t.cpu().numpy() for t in out + c + a + c2]
        assert np.all(plan.poll() == 0)
        # list order is the candidate order, which the skin changes with the cell side
        if first is None or (skin and not first[0]):
            first = (skin, out)
            d_r, a_r, s_r = orc.rhs(p, *st)
            tol = (1e-5, 1e-4, 1e-3) if dtype == "f32" else (1e-10, 1e-9, 1e-9)
            assert np.abs(out[2] / s_r - 1).max() <= tol[0]
            assert _err(out[0], d_r) <= tol[1] and _err(out[1], a_r) <= tol[1]
            for got, ref in zip(out[3:6], orc.step_adjoint(p, *st, *cot)):
                assert _err(got, ref) <= tol[2]
            s1 = orc.step(p, *st, 1)
            g1 = orc.step_adjoint(p, *s1, *cot)
            for got, ref in zip(out[9:12], orc.step_adjoint(p, *st, *g1)):
                assert _err(got, ref) <= tol[2]
        else:
            for got, ref in zip(out, first[1]):
                np.testing.assert_array_equal(got, ref)
