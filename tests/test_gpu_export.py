"""CSR export of rows on each path of the row sort: up to 64 entries (registers), up to 1024 (bucket
sort in LDS), longer ones (ranked against the full row), with the particles in lattice order, in random
order, and shifted so that rows cross the periodic boundary in both index directions.  Integer output:
equal to the oracle's."""
import numpy as np
import pytest
import torch

from paper_2507_21684_amd.inputs import SimSpec, make_state

pytestmark = pytest.mark.gpu

# (dim, side, support factor): rows of about 49; 50 to 75 (both sides of 64); 113; 900 to 1150 (both sides
# of 1024); 1200
CASES = [(2, 24, 4.0), (2, 30, 4.55), (3, 16, 3.0), (3, 20, 6.25), (3, 20, 6.6)]


@pytest.mark.parametrize("dim,side,sf", CASES)
@pytest.mark.parametrize("shuffled", [False, True])
def test_export_rows(orc, dim, side, sf, shuffled):
    from paper_2507_21684_amd.lib import Plan
    spec = SimSpec(dim, side, support_factor=sf, jitter=0.4)
    x, v, rho = make_state(spec, 11)
    if shuffled:
        p = np.random.default_rng(5).permutation(spec.n)
        x, v, rho = x[:, p], v[:, p], rho[p]
    x = x.astype(np.float32)
    plan = Plan([spec.params()], [spec.n], "f32", tape_depth=0)
    t = [torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda") for a in (x, v, rho)]
    off, nbr = plan.neighbors(*t)
    off_r, nbr_r = orc.neighbors(x.astype(np.float64), spec.box, spec.H, "f32")
    np.testing.assert_array_equal(off.cpu().numpy(), off_r)
    np.testing.assert_array_equal(nbr.cpu().numpy(), nbr_r)
