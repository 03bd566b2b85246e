"""Extraction of few tiles (three channels between barriers, the summed-area
table's carries formed by each tile) against that of many tiles in one launch,
bit by bit: every channel count of a group's remainder, every radius, both
schemes, and the tile counts at which the carries change hands.  The many are
what the oracle tests cover."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1808_06194_amd import cfog
    cfog.load()
    return cfog


@pytest.fixture(scope="module")
def big():
    return torch.rand((1100, 1300), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")


def _alone_and_among(cf, big, H, W, **kw):
    print("[case] spread", H, W, kw, flush=True)
    img = torch.rand((H, W), generator=torch.Generator(device="cuda").manual_seed(H * 7 + W), device="cuda")
    one = cf.cfog_extract_batch([img], **kw)
    many = cf.cfog_extract_batch([img, big], **kw)
    torch.cuda.synchronize()
    assert torch.equal(one[0][0], many[0][0])
    assert torch.equal(one[1][0], many[1][0])


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 9, 16])
@pytest.mark.parametrize("scheme", [1, 2])
@pytest.mark.parametrize("R", range(9))
def test_channels_and_radii(cf, big, m, scheme, R):
    _alone_and_among(cf, big, 37, 150, m=m, sigma=0.8, radius=R, scheme=scheme)


@pytest.mark.parametrize("H,W", [(1, 1), (16, 128), (17, 129), (256, 257), (257, 130), (512, 100), (513, 100),
                                 (20, 8192), (20, 8193), (120, 8192), (512, 2048), (500, 2100)])
def test_tile_counts(cf, big, H, W):
    """16 and 17 tile rows (one and two to a sum), 32 and 33, 64 and 65 tile
    columns, 256 and 512 tiles and one more."""
    _alone_and_among(cf, big, H, W)
