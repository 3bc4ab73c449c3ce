"""The counting sort where its path changes: plans whose cells are scanned inside the gather, by the scan
launches, and with the members scattered after them; cells with more particles than places for them (the
rest are chained) and plans with fewer places than cells.  Integer output: the lists equal the oracle's.
Two steps in one call, which count the second sort's cells in the first step's sweep, equal two calls,
bitwise."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec

pytestmark = pytest.mark.gpu

# (dim, box cells set by side, particles, edge of the region they fill, dtype, list width: the default or all)
CASES = [(2, 20, 400, 1.0, "f32", 0),         # one wavefront's share of the cells
         (2, 64, 900, 0.15, "f32", 900),     # dense cells: chains
         (3, 20, 3000, 0.3, "f64", 3000),     # the same in 3D
         (2, 250, 300, 0.03, "f64", 300),     # one place per cell, cells scanned in the gather
         (2, 256, 20000, 0.6, "f32", 0),      # 16 384 cells, the most of that path
         (2, 260, 20000, 0.6, "f32", 0),      # one row of blocks more
         (2, 300, 3000, 0.05, "f32", 3000),   # scan launches, chains
         (3, 60, 6000, 0.4, "f32", 0),
         (2, 732, 5000, 0.04, "f32", 5000),    # members scattered after the scan
         (3, 104, 5000, 0.15, "f64", 5000)]


@pytest.mark.parametrize("dim,side,n,edge,dtype,width", CASES)
def test_sort(orc, dim, side, n, edge, dtype, width):
    from paper_2507_21684_amd.lib import Plan
    spec = SimSpec(dim, side)
    npdt, tdt = (np.float32, torch.float32) if dtype == "f32" else (np.float64, torch.float64)
    rng = np.random.default_rng(31)
    x = (0.3 + edge * rng.uniform(size=(dim, n))).astype(npdt)
    st = [x, (0.1 * rng.normal(size=(dim, n))).astype(npdt), np.ones(n, dtype=npdt)]
    gpu = lambda: [torch.tensor(a, dtype=tdt, device="cuda").contiguous() for a in st]
    plan = Plan([spec.params()], [n], dtype, max_neighbors=width, tape_depth=0)
    off_r, nbr_r = orc.neighbors(x.astype(np.float64), spec.box, spec.H, dtype)
    for _ in range(2):   # the counts are cleared for the next sort
        off, nbr = plan.neighbors(*gpu())
        np.testing.assert_array_equal(off.cpu().numpy(), off_r)
        np.testing.assert_array_equal(nbr.cpu().numpy(), nbr_r)
    a, b = gpu(), gpu()
    plan.step(*a, 3)
    for _ in range(3):
        plan.step(*b, 1)
    assert np.all(plan.poll() == 0)
    for p, q in zip(a, b):
        assert torch.equal(p, q)
