"""The BF16 matcher's kernels (blocks of 16 offsets x chunks of 32 template
columns): each at the largest and an odd template, with one and two template
buffers, and the limit of what is taken.  The reference is the correlation of the
BF16-rounded windows in FP64, so what is left is the FP32 accumulation: a chain of
L = m ceil(Ws / 8) 32 ceil(N / 32) + 8 additions, of which the SSD has twice the
error, gamma_L (E1 + E2) at most, and its own rounding, 2^-22 (E1 + E2)."""
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


def _taken(N, r):
    K, NP, Ws = 2 * r + 1, (N + 31) // 32 * 32, N + 2 * r
    nblk = (K + 15) // 16
    t, s = (N + 30) * (NP // 2 + 4) * 4, Ws * (NP + 16 * nblk + 2) // 2 * 4
    return nblk <= 5 and max(t + s, 20 * K * K + 128) <= 160 * 1024


def _run(cf, N, r, m, n=3):
    print("[case] mfma", N, r, m, flush=True)
    g = torch.Generator(device="cuda").manual_seed(1000 * N + r)
    Ws, K, h = N + 2 * r, 2 * r + 1, N // 2
    H, W = Ws + 3, Ws + 6
    vols = [torch.rand((m, H, W), generator=g, device="cuda") for _ in range(2)]
    sats = []
    for v in vols:
        s = torch.zeros((H + 1, W + 1), dtype=torch.float64, device="cuda")
        s[1:, 1:] = (v.double() ** 2).sum(0).cumsum(0).cumsum(1)
        sats.append(s)
    cps = np.array([[h + r + k, h + r + k % 4, h + r + k, h + r + (k + 1) % 4] for k in range(n)], np.int32)
    surf = torch.empty((n, K, K), device="cuda")
    cf.match_batch([cf.Job(vols[0], sats[0], vols[1], sats[1], torch.from_numpy(cps).cuda(), N, r, surfaces=surf)], m=m,
                   flags=cf.PATH_MFMA_BF16)
    torch.cuda.synchronize()
    A, B = (v.double().cpu().numpy() for v in vols)
    Ab, Bb = (v.to(torch.bfloat16).double().cpu().numpy() for v in vols)
    for k, (x, y, bx, by) in enumerate(cps):
        T, S = np.s_[:, y - h:y - h + N, x - h:x - h + N], np.s_[:, by - h - r:by - h - r + Ws, bx - h - r:bx - h - r + Ws]
        C = np.fft.irfft2((np.conj(np.fft.rfft2(Ab[T], (Ws, Ws))) * np.fft.rfft2(Bb[S])).sum(0), (Ws, Ws))[:K, :K]
        q = np.zeros((Ws + 1, Ws + 1))
        q[1:, 1:] = (B[S] ** 2).sum(0).cumsum(0).cumsum(1)
        E = (A[T] ** 2).sum() + q[N:, N:] - q[:K, N:] - q[N:, :K] + q[:K, :K]
        L = m * ((Ws + 7) // 8) * 32 * ((N + 31) // 32) + 8
        tol = (L * 2.0 ** -24 / (1 - L * 2.0 ** -24) + 2.0 ** -22) * E
        assert (np.abs(surf[k].cpu().numpy() - (E - 2 * C)) <= tol).all(), (N, r, k)


@pytest.mark.parametrize("nb", range(1, 6))
@pytest.mark.parametrize("kc", range(1, 7))
def test_kernels(cf, nb, kc):
    rs = (8 * nb - 8, 8 * nb - 1)  # fewest and most offsets of nb blocks: 16 (nb - 1) + 1 and 16 nb - 1
    sizes = [(N, r) for r in rs for N in (32 * kc, 32 * kc - 31, 32 * kc - 5) if _taken(N, r)]
    for N, r in sizes:
        _run(cf, N, r, 2)


@pytest.mark.parametrize("N,r", [(1, 0), (3, 1), (5, 0), (128, 32)])
def test_small_windows_and_channels(cf, N, r):
    """Windows of fewer rows than waves; one channel and the usual nine."""
    _run(cf, N, r, 1)
    _run(cf, N, r, 9)


@pytest.mark.parametrize("r", [0, 7, 8, 20, 32, 39])
def test_what_is_taken(cf, r):
    N = max(N for N in range(1, 400) if _taken(N, r))
    _run(cf, N, r, 2, n=1)
    with pytest.raises(cf.CfogError):
        _run(cf, N + 1, r, 1, n=1)
