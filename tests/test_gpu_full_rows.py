"""Rows that fill their list to the last place: a whole last group of 16 positions, and a whole half group behind
them.  Bitwise what a wider list gives, for every lane count; and the pair count of lists with a skin,
which leaves the particle itself and the filled-up places out."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state

pytestmark = pytest.mark.gpu

# (dim, side, support factor, seed, widest row with the particle itself)
CASES = [(2, 24, 3.0, 0, 32), (2, 24, 3.3, 11, 40), (2, 24, 2.5, 22, 24), (3, 12, 1.8, 8, 32), (3, 12, 1.6, 1, 24),
         (3, 13, 2.5, 21, 80), (3, 13, 2.45, 0, 72)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("dim,side,sf,seed,widest", CASES)
def test_full_rows_and_pair_count(orc, dim, side, sf, seed, widest, dtype):
    from paper_2507_21684_amd.lib import Plan
    spec = SimSpec(dim, side, support_factor=sf, jitter=0.3)
    npdt, tdt = (np.float32, torch.float32) if dtype == "f32" else (np.float64, torch.float64)
    rng = np.random.default_rng(seed)
    st = [a.astype(npdt) for a in make_state(spec, seed)]
    cot = [rng.normal(size=a.shape).astype(npdt) for a in st]
    off, _ = orc.neighbors(st[0].astype(np.float64), spec.box, spec.H, dtype)
    assert int(np.diff(off).max()) == widest
    gpu = lambda arrs: [torch.tensor(a, dtype=tdt, device="cuda").contiguous() for a in arrs]
    outs = []
    for width, lanes in ((widest + 16, 4), (widest, 2), (widest, 4), (widest, 8)):
        plan = Plan([spec.params()], [spec.n], dtype, max_neighbors=width)
        assert plan.max_neighbors == width
        plan.set_tuning(lanes, lanes)
        g, c = gpu(st), gpu(cot)
        out = list(plan.rhs(*g))
        plan.step_adjoint(*g, *c)
        out += [plan.density_adjoint(*g, c[2])] + c
        assert np.all(plan.poll() == 0)   # no row overflowed
        outs.append(out)
    for out in outs[1:]:
        for a, b in zip(outs[0], out):
            assert torch.equal(a, b)
    for lanes in (2, 4, 8):
        plan = Plan([spec.params()], [spec.n], dtype, skin=0.2, rebuild_every=2)
        plan.set_tuning(lanes, lanes)
        plan.rhs(*gpu(st))
        assert plan.pair_count() == int(off[-1]) - spec.n
