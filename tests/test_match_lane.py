"""The matcher's lane layout (FFT sides from 60): its real-input codelets on
the host, the sizes it takes, and every side at the edges of its range against
the oracle under the parity rules."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle as O
from paper_1808_06194_amd import cfog, synth
from tests import parity

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIDES = (60, 64, 72, 80, 90, 96, 100, 108, 120, 144, 160, 192)


def test_rdft_codelets_host_build(tmp_path):
    exe = tmp_path / "rdft_codelets"
    r = subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O2", "-x", "hip", "--offload-arch=gfx950", "-I",
                        os.path.join(ROOT, "paper_1808_06194_amd", "csrc"),
                        os.path.join(ROOT, "tests", "cpp", "rdft_codelets.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def _takes(P, N, r):
    """A side holds the window, a template of at most 134 rows at 144, and the
    K x K correlation behind the rows of the group layout's inverse."""
    K = 2 * r + 1
    return P >= N + 2 * r and N <= (134 if P == 144 else P) and K * K <= 2 * (P - 2 * ((K + 1) // 2)) * (P // 2 + 1)


def test_sizes_taken():
    for N in range(1, 200):
        for r in range(0, 100):
            fit = [P for P in (16, 24, 32, 40, 48) + SIDES if _takes(P, N, r)]
            assert cfog.fft_size(N, r) == (fit[0] if fit else 0), (N, r)


def _edges():
    prev = 48
    for P in SIDES:
        r = 3 + P // 16
        yield P, P - 2 * r, r, 9                       # the window fills the side
        yield P, prev + 1 - 2 * (r // 2), r // 2, 2     # the smallest window of the side
        r = max(r for r in range(P // 2) if _takes(P, 1, r))
        yield P, min(P - 2 * r, 134), r, 3              # the most offsets
        prev = P
    yield 60, 60, 0, 1                                  # one offset, one channel
    yield 144, 1, 40, 1                                 # a template of one pixel
    yield 144, 134, 5, 2                                # the most template rows
    yield 192, 191, 0, 5


@pytest.mark.gpu
@pytest.mark.parametrize("P,N,r,m", list(_edges()))
def test_every_side_at_its_edges(P, N, r, m):
    print("lane", P, N, r, m, flush=True)
    rng = np.random.default_rng(1000 * P + N)
    H, W = N + 2 * r + 9, N + 2 * r + 14
    A, B, _ = synth.make_pair(synth.PairSpec(H, W, 12, (2.0, 9.0), 6, 2), (P, N))
    vA, sA = cfog.cfog_extract(torch.from_numpy(A).cuda(), m=m)
    vB, sB = cfog.cfog_extract(torch.from_numpy(B).cuda(), m=m)
    h = N // 2
    x, y = rng.integers(h + r, W - (N - h) - r + 1, 5), rng.integers(h + r, H - (N - h) - r + 1, 5)
    cps = np.stack([x, y, x, y], 1).astype(np.int32)
    cps[4] = (0, 0, W, H)  # its windows leave the images
    K = 2 * r + 1
    try:
        cfog.set_plan(N, r, P)
        for flags in (cfog.PATH_PLAIN_FFT, cfog.PATH_PLAIN_FFT | cfog.NO_SPLIT):
            surf = torch.full((len(cps), K, K), -1.0, device="cuda")
            job = cfog.Job(vA, sA, vB, sB, torch.from_numpy(cps).cuda(), N, r, surfaces=surf)
            cfog.match_batch([job], m=m, flags=flags)
            torch.cuda.synchronize()
            res = {k: v.cpu().numpy() for k, v in cfog.results(job.out).items()}
            s = surf.cpu().numpy()
            DA, DB = vA.cpu().numpy().astype(np.float64), vB.cpu().numpy().astype(np.float64)
            for k in range(4):
                cp = tuple(int(v) for v in cps[k])
                E1, E2 = O.energies(DA, DB, cp, N, r)
                parity.check_point(k, res, O.ssd_surface_direct(DA, DB, cp, N, r), E1, E2, r, s[k])
            assert res["status"][4] == cfog.CP_OUT_OF_BOUNDS and np.isnan(s[4]).all()
        # more points than are resident at once: the smaller workgroups, the same roundings
        many = torch.from_numpy(np.tile(cps, (700, 1))).cuda()
        surf = torch.full((len(many), K, K), -1.0, device="cuda")
        cfog.match_batch([cfog.Job(vA, sA, vB, sB, many, N, r, surfaces=surf)], m=m,
                         flags=cfog.PATH_PLAIN_FFT | cfog.NO_SPLIT)
        torch.cuda.synchronize()
        assert np.array_equal(surf.cpu().numpy(), np.tile(s, (700, 1, 1)), equal_nan=True)
    finally:
        cfog.set_plan(N, r, 0)


@pytest.mark.gpu
def test_images_wider_than_the_byte_offsets():
    """Images of more than 2^21 columns take the group layout: the same points
    cut out of them, which take the lane layout, agree under the parity rules'
    surface tolerance (1e-4 of E1 + E2)."""
    N, r, H, W, m = 40, 8, 64, (1 << 21) + 77, 1
    print("lane wide", W, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    vol = torch.rand((m, H, W), generator=g, device="cuda")
    sat = torch.zeros((H + 1, W + 1), dtype=torch.float64, device="cuda")
    sat[1:, 1:] = (vol.double() ** 2).sum(0).cumsum(0).cumsum(1)
    x0, K = W - 128, 2 * r + 1
    cut = vol[:, :, x0:].contiguous()
    csat = torch.zeros((H + 1, 129), dtype=torch.float64, device="cuda")
    csat[1:, 1:] = (cut.double() ** 2).sum(0).cumsum(0).cumsum(1)
    cps = np.array([[x, 30, x + 1, 31] for x in (40, 70, 99)], np.int32)
    out = []
    for v, s, dx in ((vol, sat, x0), (cut, csat, 0)):
        surf = torch.empty((len(cps), K, K), device="cuda")
        c = torch.from_numpy(cps + np.array([dx, 0, dx, 0], np.int32)).cuda()
        job = cfog.Job(v, s, v, s, c, N, r, surfaces=surf)
        cfog.match_batch([job], m=m)
        torch.cuda.synchronize()
        assert (cfog.results(job.out)["status"] == 0).all()
        out.append(surf.cpu().numpy().astype(np.float64))
    energy = float(2 * (cut.double() ** 2).mean()) * N * N * m
    assert np.abs(out[0] - out[1]).max() <= 1e-4 * energy
