"""The lane settings the tuner times: eight lanes only where the library runs them."""
from types import SimpleNamespace

import pytest

from paper_2507_21684_amd import autotune


@pytest.mark.parametrize("dim,dtype,n,want", [(2, "f32", 32767, (2, 4, 8)), (2, "f32", 32768, (2, 4)),
                                              (2, "f64", 16383, (2, 4, 8)), (2, "f64", 16384, (2, 4)),
                                              (3, "f32", 1000000, (2, 4, 8)), (3, "f64", 1000000, (2, 4, 8))])
def test_lane_choices(dim, dtype, n, want):
    assert autotune.lane_choices(SimpleNamespace(dim=dim, dtype=dtype, N=n)) == want
