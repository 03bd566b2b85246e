"""The Harris kernel at its edges: every Gaussian radius, chips whose width is
no multiple of a thread's four columns or below them, chips of a wave's rows
and one more, ties over all waves, and chips with too few finite responses;
against the oracle under the rules of test_gpu_harris.py."""
import numpy as np
import pytest

from paper_1808_06194_amd import synth
from tests.test_gpu_harris import _check, _run, _say, cf  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", range(9))
@pytest.mark.parametrize("H,W,n,k,chip", [(190, 150, 3, 5, 64), (130, 141, 2, 7, 61), (97, 66, 2, 2, 17),
                                          (60, 59, 4, 3, 5), (40, 40, 6, 1, 2), (33, 3, 1, 4, 64)])
def test_radii_and_widths(cf, R, H, W, n, k, chip):  # noqa: F811
    _say("harris edges", R, H, W, n, k, chip)
    A, _, _ = synth.make_pair(synth.PairSpec(max(H, 64), max(W, 64), 12, (3.0, 15.0), 4, 4), (71, R))
    A = np.asarray(A)[:H, :W]
    sigma = max(R / 4.0, 0.1)
    cps, resp = _run(cf, A, n, k, chip, sigma)
    _check(A, n, k, chip, cps, resp, sigma)


def test_ties_take_the_smallest_index(cf):  # noqa: F811
    _say("harris ties 64x64 k=64")
    cps, resp = _run(cf, np.full((64, 64), 2.0), 1, 64, 64)
    assert [(x, y) for x, y, _, _ in cps.tolist()] == [(x, 0) for x in range(64)] and (resp == 0).all()


def test_too_few_finite_responses(cf):  # noqa: F811
    """NaN from column 7 on: with radius 4 and the gradient's 1, columns 0 and 1 are finite."""
    _say("harris finite 16 of 20")
    img = np.random.default_rng(3).random((8, 8)).astype(np.float32)
    img[:, 7] = np.nan
    cps, resp = _run(cf, img, 1, 20, 8)
    assert {(x, y) for x, y, _, _ in cps[:16].tolist()} == {(x, y) for x in (0, 1) for y in range(8)}
    assert (np.diff(resp[:16]) <= 0).all()
    assert (cps[16:] == -1).all() and np.isnan(resp[16:]).all()
