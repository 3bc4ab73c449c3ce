"""The workspace follows the particles and the tape; many empty cells add only their own tables."""
import pytest

from paper_2507_21684_amd import lib as L
from paper_2507_21684_amd.inputs import SimSpec


@pytest.mark.parametrize("n,tape", [(1000, 158), (2000, 79)])
def test_a_mostly_empty_box_fits_the_static_workspace(n, tape):
    spec = SimSpec(2, 700)
    assert L.workspace_bytes([spec.params()], [n], "f32", tape_depth=tape) <= L.SCRATCH_BYTES


@pytest.mark.parametrize("dim,side", [(2, 700), (3, 100)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_empty_cells_cost_their_tables_alone(dim, side, dtype):
    """Counts, starts, the simulation index and the blocks' two tables: 12 bytes per cell, 8 per block (of at
    least 8 cells) and 4 per scan tile; the rest is the particles'."""
    few, many = SimSpec(dim, 48), SimSpec(dim, side)
    grow = [L.workspace_bytes([dict(s.params(), H=s.H)], [1000], dtype, max_neighbors=64, tape_depth=4)
            for s in (few, many)]
    side_cells = int(2.0 / (many.H * (1 + 1 / 1024)))
    side_blocks = -(-side_cells // (4 if dim == 2 else 2))
    blocks = side_blocks ** dim
    cells = blocks * (16 if dim == 2 else 8)
    assert grow[1] - grow[0] <= 12 * cells + 8 * blocks + 4 * (cells // 2048 + 1) + 6 * 256
