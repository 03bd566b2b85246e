"""Extraction launches of exactly as many tiles as each rule takes, and one more
(three channels between barriers: a tile per compute unit; the table's carries
formed by each tile: 512), against the same images in a launch of many tiles, bit
by bit.  Both stay within 64 tile columns and 32 tile rows, so the count decides."""
import pytest
import torch

from tests.test_gpu_extract_spread import big, cf  # noqa: F401

pytestmark = pytest.mark.gpu

TX, TY = 128, 16


def _shapes(tiles):
    """Images of `tiles` tiles in all: one of 16 or 32 tile rows, and single tiles for the rest."""
    rows = 32 if tiles > 16 * 64 or tiles >= 512 else 16
    cols = tiles // rows
    assert cols <= 64
    return [(rows * TY, cols * TX)] + [(TY, TX)] * (tiles - rows * cols)


@pytest.mark.parametrize("limit", ["cus", 512])
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("m,R", [(9, 3), (5, 2)])
def test_exact_tile_counts(cf, big, limit, more, m, R):  # noqa: F811
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = _shapes((cus // 16 * 16 if limit == "cus" else limit) + more)
    print("[case] tiles", shapes, m, R, flush=True)
    assert len(shapes) <= 7  # with the big one, one launch
    g = torch.Generator(device="cuda").manual_seed(more + m)
    imgs = [torch.rand(s, generator=g, device="cuda") for s in shapes]
    few = cf.cfog_extract_batch(imgs, m=m, sigma=0.8, radius=R)
    many = cf.cfog_extract_batch(imgs + [big], m=m, sigma=0.8, radius=R)
    torch.cuda.synchronize()
    for k in range(len(imgs)):
        assert torch.equal(few[0][k], many[0][k])
        assert torch.equal(few[1][k], many[1][k])
