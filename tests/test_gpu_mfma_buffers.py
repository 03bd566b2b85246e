"""The BF16 matcher's launches of more points than the GPU has compute units,
where templates of about 118 to 128 rows take one template buffer instead of two
(and odd ones a kernel of their own): each point's surface is, bit by bit, that of
a launch of few points, which test_gpu_mfma_sizes.py holds to FP64."""
import numpy as np
import pytest
import torch

from tests.test_gpu_mfma_sizes import cf  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [97, 112, 117, 118, 119, 121, 127, 128, 129, 139])
@pytest.mark.parametrize("r", [0, 5, 7, 8, 15, 16])
def test_many_points_as_few(cf, N, r):  # noqa: F811
    print("[case] mfma buffers", N, r, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda").manual_seed(1000 * N + r)
    Ws, K, h, m = N + 2 * r, 2 * r + 1, N // 2, 3
    H, W = Ws + 3, Ws + 6  # the last point's windows end at the volumes' last row and column
    A, B = (torch.rand((m, H, W), generator=g, device="cuda") for _ in range(2))

    def table(v):
        s = torch.zeros((H + 1, W + 1), dtype=torch.float64, device="cuda")
        s[1:, 1:] = (v.double() ** 2).sum(0).cumsum(0).cumsum(1)
        return s

    few = torch.tensor([[h + r + x, h + r + y, h + r + x, h + r + y] for x, y in ((0, 0), (3, 1), (6, 3))],
                       dtype=torch.int32, device="cuda")
    many = few.repeat((cus // 3 + 2, 1))
    got = []
    for cps in (few, many):
        surf = torch.full((len(cps), K, K), float("nan"), device="cuda")
        cf.match_batch([cf.Job(A, table(A), B, table(B), cps, N, r, surfaces=surf)], m=m, flags=cf.PATH_MFMA_BF16)
        torch.cuda.synchronize()
        got.append(surf)
    assert len(many) > cus and torch.isfinite(got[0]).all()
    assert torch.equal(got[1], got[0].repeat((cus // 3 + 2, 1, 1)))
