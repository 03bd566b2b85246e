"""Full or spread workgroups of the lane layout: the rule on the host, and the
autotuner, whose trials run in the workgroups that the call will take."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle as O
from paper_1808_06194_amd import cfog, synth
from tests import parity

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_spread_rule_host_build(tmp_path):
    exe = tmp_path / "spread_rule_test"
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_1808_06194_amd", "csrc"),
                        os.path.join(ROOT, "tests", "cpp", "spread_rule_test.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.fixture(scope="module")
def scene():
    A, B, _ = synth.make_pair(synth.PairSpec(160, 170, 12, (2.0, 9.0), 6, 2), (7, 8))
    return [cfog.cfog_extract(torch.from_numpy(i).cuda()) for i in (A, B)]


def _job(scene, N, r, n):
    (va, sa), (vb, sb) = scene
    rng, h = np.random.default_rng([N, r, n]), N // 2
    x, y = rng.integers(h + r, 170 - (N - h) - r + 1, n), rng.integers(h + r, 160 - (N - h) - r + 1, n)
    cps = torch.from_numpy(np.stack([x, y, x, y], 1).astype(np.int32)).cuda()
    return cfog.Job(va, sa, vb, sb, cps, N, r, surfaces=torch.empty((n, 2 * r + 1, 2 * r + 1), device="cuda"))


def _check(scene, job):
    torch.cuda.synchronize()
    DA, DB = (v.cpu().numpy().astype(np.float64) for v, _ in scene)
    res = {k: v.cpu().numpy() for k, v in cfog.results(job.out).items()}
    surf = job.surfaces.cpu().numpy()
    for k in sorted({0, len(surf) // 2, len(surf) - 1}):
        cp = tuple(int(v) for v in job.cps[k].tolist())
        E1, E2 = O.energies(DA, DB, cp, job.N, job.r)
        parity.check_point(k, res, O.ssd_surface_direct(DA, DB, cp, job.N, job.r), E1, E2, job.r, surf[k])


@pytest.mark.gpu
@pytest.mark.parametrize("N,r", [(40, 4), (44, 8), (50, 6), (60, 10), (91, 4), (100, 22)])
@pytest.mark.parametrize("n", [1, 40, 300, 3000])
def test_autotuned_calls(scene, N, r, n, tmp_path, monkeypatch):
    """Fewer points than the trials run on, as many and more; the pick is one of the three smallest sides and is kept."""
    print("[case] autotune", N, r, n, flush=True)
    monkeypatch.setenv("CFOG_PLAN_CACHE", str(tmp_path / "plans"))
    ctx = cfog.Context(0)
    try:
        sides = [P for P in (16, 24, 32, 40, 48, 60, 64, 72, 80, 90, 96, 100, 108, 120, 144, 160, 192)
                 if P >= cfog.fft_size(N, r)][:3]
        for flags in (cfog.PATH_PLAIN_FFT, cfog.PATH_BATCHED_FFT):
            jobs = [_job(scene, N, r, n), _job(scene, N, r, 7)]
            cfog.match_batch(jobs, flags=flags | cfog.AUTOTUNE, ctx=ctx)
            for job in jobs:
                _check(scene, job)
        lines = [tuple(map(int, line.split())) for line in open(tmp_path / "plans")]
        assert len(lines) == 1 and lines[0][:3] == (N, r, 9) and lines[0][3] in sides
    finally:
        ctx.close()


@pytest.mark.gpu
def test_batched_sizes_of_one_launch(scene):
    """Several sizes, whose launches are of all the points of a side."""
    print("[case] autotune batched", flush=True)
    ctx = cfog.Context(0)
    try:
        jobs = [_job(scene, N, r, n) for N, r, n in ((60, 10, 90), (62, 8, 200), (58, 9, 5), (72, 10, 30), (50, 4, 1))]
        for _ in range(2):
            cfog.match_batch(jobs, flags=cfog.PATH_BATCHED_FFT | cfog.AUTOTUNE, ctx=ctx)
            for job in jobs:
                _check(scene, job)
    finally:
        ctx.close()
