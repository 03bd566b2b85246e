"""Outlier rejection of sets held in registers (up to 4096 points): the edges
of waves, of the workgroup, of its two halves and of the kernel, ties over
waves and threads, and non-finite points; against the FP64 oracle under the
rules of test_gpu_outlier.py."""
import numpy as np
import pytest

from tests.test_gpu_outlier import _compare, _points, _say, cf, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [11, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1025, 4095, 4096, 4097])
def test_sizes(cf, n):  # noqa: F811
    _say("reject edges", n)
    P, Q, _ = _points(100 + n, n, max(1, n // 100))
    _compare(cf, P, Q, 1.0)


def test_ten_points_are_kept(cf):  # noqa: F811
    _say("reject n=10")
    P, Q, _ = _points(90, 10, 1)
    keep, res = cf.reject_outliers(torch.from_numpy(P).cuda(), torch.from_numpy(Q).cuda(), 0.0)
    assert res["status"] == 0 and res["removed"] == 0 and keep.cpu().numpy().all()


@pytest.mark.parametrize("copies", [(40, 41), (40, 40 + 64), (40, 40 + 256), (40, 300, 296, 552, 1000)])
def test_equal_residuals_leave_by_index(cf, copies):  # noqa: F811
    """Points that are the same in every bit: the first of them leaves first."""
    _say("reject ties", copies)
    P, Q, _ = _points(91, 1100, 1, noise=0.1)
    for i in copies:
        P[i], Q[i] = P[copies[0]], Q[copies[0]] + (30 if i == copies[0] else 0)
    for thr in np.linspace(0.3, 6.0, 12):
        _compare(cf, P, Q, float(thr))


@pytest.mark.parametrize("where", [3, 700])
def test_non_finite_target(cf, where):  # noqa: F811
    _say("reject NaN", where)
    P, Q, _ = _points(92, 800, 4)
    Q[where, 1] = np.nan
    keep, res = cf.reject_outliers(torch.from_numpy(P).cuda(), torch.from_numpy(Q).cuda(), 1.0)
    assert res["status"] == 1 and res["removed"] == 0 and keep.cpu().numpy().all() and np.isnan(res["rmse"])
