"""Pixel-wise HOG with every cell size at the edges of its 64 x 32 tiles, against
the oracle under the bounds of test_gpu_fhog.py."""
import pytest

from tests.test_gpu_fhog import cf, test_fhog_volume_and_sat_match_oracle as check  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell", range(1, 9))
@pytest.mark.parametrize("H,W", [(1, 1), (32, 64), (33, 65), (70, 131)])
def test_tile_edges(cf, cell, H, W):  # noqa: F811
    check(cf, H, W, cell, 110 + cell)
