#!/usr/bin/env python3
"""Benchmark of the CFOG + 3-D-FFT SSD matching hot path on one MI355X.

One step = the whole hot path on one batch of synthetic input: CFOG extraction
of every image (volume + FP64 summed-area table; all images in one batched
extraction call, up to 8 per launch; pixel-wise HOG volumes alternate between
two streams) and SSD matching of every control point (correlation, FP64
energies, argmin).  Inputs are resident in HBM before the timed region starts.

Workloads (--workload):
  plain_2048 (default): one 2048^2 fp32 pair (800 blobs sigma 3-40, 300
      rectangles, |sin(3A)| x Gamma(4) speckle, |shift| <= 20), 400 control
      points on a 20x20 grid, template 100, radius 20.
  plain_256: one 256^2 pair, 25 control points, template 48, radius 10.
  precision_4096: one 4096^2 pair (3200 blobs sigma 3-40, 1200 rectangles),
      10,000 random control points, template 128, radius 32; --path fft
      (FP32 FFT) or mfma (BF16 MFMA direct correlation).
  batch_64: 64 pairs with sides from {512, 1024, 2048, 4096}, templates in
      [40, 120], radii in [5, 30], 50-600 control points per pair; --path
      batched (fused persistent launches, autotuned FFT sizes, hipGraph
      replay) or plain (one launch per pair).
  harris_8192: block-based Harris feature points (Section IV) of one 8192^2
      image: 128 x 128 cells, 60 x 60 chips, 4 points per chip; reports
      feature points/s (the control-point producer, not a CP-match rate).
  reject_3000: iterative cubic outlier rejection (Section IV) of one set of
      3000 matched points (5% gross outliers, threshold 1 px); reports point
      sets/s.
--descriptor (matching workloads): cfog (Eq. 2, default), scheme1 (CFOG
  with binned orientations) or fhog (36-channel pixel-wise HOG, cell 4); the
  matcher then takes that volume (m = 9, 9, 36).
  serve: the matching server with 32 resident pairs (8 each of 1024^2,
      2048^2, 4096^2, 8192^2) under open-loop Poisson arrivals of requests
      (1-500 control points, template 40-128, radius 5-32): latency
      percentiles at 200 requests/s, then a rate sweep; `value` is the highest
      CP matches/s sustained in the sweep.  Also checks that a seeded sample
      of requests gives bit-identical results alone and in the mix.

Prints ONE JSON line.  `--gpus N` with N > 1 is refused: the benchmark runs on
one GPU.
"""
from __future__ import annotations

import argparse
import dataclasses
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# Vector FP32 without packed instructions (the library is compiled with packed
# FP32 disabled): 256 CUs x 4 SIMDs x 16 lanes x 2 flops (FMA) x 2.4 GHz.
FP32_PEAK_TFS = 78.6
BF16_PEAK_TFS = 2500.0     # dense BF16 MFMA


def algorithmic_bytes_per_cp(N: int, r: int, m: int = 9, surfaces: bool = False) -> int:
    """HBM bytes one control point must move at minimum: the template and
    search-window volumes (fp32, m channels), the four SAT corner blocks of the
    (2r+1)^2 window energies (fp64), the CP and the 24-byte result."""
    Ws, K = N + 2 * r, 2 * r + 1
    b = 4 * m * (N * N + Ws * Ws) + 4 * 8 * K * K + 16 + 24
    if surfaces:
        b += 4 * K * K
    return b


def fft_flops_per_cp(N: int, r: int, P: int, m: int = 9) -> float:
    """Flops of the FFT matcher per control point with the 5 n log2 n model per
    complex FFT of length n: per channel, ceil(N/2) + ceil(Ws/2) packed row
    FFTs and 2 (P/2+1) column FFTs, a complex multiply-add per half-spectrum
    point; then (P/2+1) + ceil(K/2) inverse FFTs."""
    Ws, K, PH = N + 2 * r, 2 * r + 1, P // 2 + 1
    f = 5.0 * P * np.log2(P)
    per_ch = ((N + 1) // 2 + (Ws + 1) // 2 + 2 * PH) * f + 8.0 * P * PH
    return m * per_ch + (PH + (K + 1) // 2) * f


def direct_flops_per_cp(N: int, r: int, m: int = 9) -> float:
    """Useful multiply-adds of the spatial correlation: 2 m N^2 (2r+1)^2."""
    return 2.0 * m * N * N * (2 * r + 1) ** 2


def extract_bytes_per_px(m: int = 9) -> int:
    """Image read (4) + volume write (4m) + FP64 SAT write (8)."""
    return 4 + 4 * m + 8


# ------------------------------------------------------------ CPU leg
#
# The oracle (FP64, test infrastructure) is timed on the host cores on a
# bounded sample of the workload's control points, in forked worker processes
# started before anything touches the GPU.  The same oracle outputs are then
# the reference for the GPU's results on those points (the parity block of the
# JSON line).

CFOG_R = 3  # Gaussian radius at sigma = 0.8: int(4 sigma + 0.5)
PAPER_CFOG_MPX_S = 512 * 512 / 0.210 / 1e6  # Table III: 0.210 s per 512^2 image on an i7-4710MQ


def cpu_workers() -> int:
    """Host cores this process may use: its CPU affinity, at most 16 (one
    GPU's share of the host)."""
    try:
        n = len(os.sched_getaffinity(0))
    except AttributeError:
        n = os.cpu_count() or 1
    return max(1, min(16, n))


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def _crop(img: np.ndarray, y0: int, x0: int, h: int, w: int, margin: int):
    """Rows [y0 - margin, y0 + h + margin) x cols [x0 - margin, ...) of img,
    clipped to the image, and the offset of (y0, x0) inside the crop.  CFOG at
    a pixel reads only its (2R + 3)^2 neighbourhood, so with margin R + 1 the
    oracle's CFOG of the crop equals that of the whole image on the box."""
    H, W = img.shape
    ya, xa = max(0, y0 - margin), max(0, x0 - margin)
    yb, xb = min(H, y0 + h + margin), min(W, x0 + w + margin)
    return np.ascontiguousarray(img[ya:yb, xa:xb]), y0 - ya, x0 - xa


def _oracle_point_task(args):
    """One sampled control point through the oracle: CFOG of the crops that
    hold its template and search box, the direct SSD surface (Eq. 3) and the
    FP64 FFT form (Eqs. 5, 8-9) with its own SATs; times of each part."""
    import oracle as O
    A, B, cp, N, r, m, desc = args
    x, y, bx, by = (int(v) for v in cp)
    h = N // 2
    Ws = N + 2 * r
    M = CFOG_R + 1
    ca, ay, ax = _crop(A, y - h, x - h, N, N, M)
    cb, by0, bx0 = _crop(B, by - h - r, bx - h - r, Ws, Ws, M)
    fn = {"cfog": lambda I: O.cfog(I, m=m), "scheme1": lambda I: O.cfog(I, m=m, scheme=1), "fhog": O.fhog}[desc]
    t0 = time.perf_counter()
    D1 = fn(ca.astype(np.float64))
    D2 = fn(cb.astype(np.float64))
    t1 = time.perf_counter()
    T = np.ascontiguousarray(D1[:, ay:ay + N, ax:ax + N])
    Sw = np.ascontiguousarray(D2[:, by0:by0 + Ws, bx0:bx0 + Ws])
    loc = (h, h, h + r, h + r)
    S = O.ssd_surface_direct(T, Sw, loc, N, r)
    t2 = time.perf_counter()
    sat1 = O.sat(np.sum(T * T, axis=0))
    sat2 = O.sat(np.sum(Sw * Sw, axis=0))
    t3 = time.perf_counter()
    Sf = O.ssd_surface_fft(T, Sw, loc, N, r, None, sat1, sat2)
    t4 = time.perf_counter()
    E1, E2 = O.energies(T, Sw, loc, N, r)
    return dict(S=S, Sf=Sf, E1=E1, E2=E2, px=ca.size + cb.size, t_cfog=t1 - t0, t_direct=t2 - t1,
                t_fft=t4 - t3, t_sat=t3 - t2)


def _oracle_tile_task(args):
    """The oracle's CFOG of one image tile; returns (pixels, seconds)."""
    import oracle as O
    tile, m, desc = args
    fn = {"cfog": lambda I: O.cfog(I, m=m), "scheme1": lambda I: O.cfog(I, m=m, scheme=1), "fhog": O.fhog}[desc]
    t0 = time.perf_counter()
    fn(tile.astype(np.float64))
    return tile.size, time.perf_counter() - t0


def sample_points(name: str, pairs, n_sample: int):
    """Seeded sample of (pair, cp) indices: every control point of small
    workloads; for several pairs, n_sample / (pairs) distinct points of every
    pair (at least one, so every FFT-size bucket is in it); else n_sample
    points of the single pair."""
    rng = np.random.default_rng(np.random.SeedSequence([8, 1808]))
    if len(pairs) > 1:
        per = max(1, n_sample // len(pairs))
        out = []
        for j, p in enumerate(pairs):
            n = len(p["cps"])
            out += [(j, int(k)) for k in np.sort(rng.choice(n, min(per, n), replace=False))]
        return out
    n = len(pairs[0]["cps"])
    if n <= n_sample:
        return [(0, k) for k in range(n)]
    return [(0, int(k)) for k in np.sort(rng.choice(n, n_sample, replace=False))]


def cpu_leg(name: str, pairs, m: int, desc: str, pool, n_workers: int, n_sample: int):
    """The oracle on the sampled points (timed) and on image tiles (the CPU
    CFOG rate), extrapolated to the whole workload over n_workers cores:
      * cpu_baseline: FP64 CFOG of every image + direct SSD (Eq. 3) of every
        point, the oracle as it stands;
      * cpu_fft_baseline: FP64 CFOG + SATs + the FFT form (Eqs. 5, 8-9) per
        point, the CPU version of the same method.
    Returns (cpu_baseline, cpu_fft_baseline, cpu_cfog, sample, oracle
    outputs per sampled point)."""
    t_all = time.perf_counter()
    sample = sample_points(name, pairs, n_sample)
    tasks = [(pairs[j]["A"], pairs[j]["B"], pairs[j]["cps"][k], pairs[j]["N"], pairs[j]["r"], m, desc)
             for j, k in sample]
    outs = list(pool.map(_oracle_point_task, tasks, chunksize=1))
    # CPU CFOG rate on 512^2 tiles (Table III's image size), one per worker
    rng = np.random.default_rng(512)
    tiles = []
    for i in range(n_workers):
        p = pairs[i % len(pairs)]
        img = p["A"] if i % 2 == 0 else p["B"]
        H, W = img.shape
        th, tw = min(512, H), min(512, W)
        y0, x0 = int(rng.integers(0, H - th + 1)), int(rng.integers(0, W - tw + 1))
        tiles.append((np.ascontiguousarray(img[y0:y0 + th, x0:x0 + tw]), m, desc))
    tile_res = list(pool.map(_oracle_tile_task, tiles, chunksize=1))
    wall = time.perf_counter() - t_all
    px_s_core = sum(px for px, _ in tile_res) / sum(t for _, t in tile_res)
    # per-point cost models fitted on the sample: direct SSD ~ m N^2 (2r+1)^2,
    # FFT form ~ m Ws^2 log2(Ws^2) (numpy's FFT of the Ws x Ws window)
    def wd(N, r):
        return float(N * N * (2 * r + 1) ** 2)

    def wf(N, r):
        Ws = N + 2 * r
        return float(Ws * Ws * np.log2(Ws * Ws))
    cd = sum(o["t_direct"] for o in outs) / sum(wd(pairs[j]["N"], pairs[j]["r"]) for j, _ in sample)
    cf_ = sum(o["t_fft"] for o in outs) / sum(wf(pairs[j]["N"], pairs[j]["r"]) for j, _ in sample)
    n_cps = sum(len(p["cps"]) for p in pairs)
    px_total = sum(p["A"].size + p["B"].size for p in pairs)
    t_ext = px_total / px_s_core                      # core-seconds
    t_direct = cd * sum(len(p["cps"]) * wd(p["N"], p["r"]) for p in pairs)
    t_fft = cf_ * sum(len(p["cps"]) * wf(p["N"], p["r"]) for p in pairs)
    t_sat = px_total * 8.0 / 1e9                       # two cumulative sums: negligible, counted at 8 ns/px
    busy = sum(o["t_cfog"] + o["t_direct"] + o["t_fft"] + o["t_sat"] for o in outs) + sum(t for _, t in tile_res)
    smp = (f"{len(sample)} sampled control points (seeded; {'spread evenly over the pairs' if len(pairs) > 1 else 'of the pair'}) "
           f"through the oracle on {n_workers} worker processes: CFOG of their crops, direct SSD and FFT form, "
           f"plus CFOG of {len(tiles)} image tiles of up to 512^2; per-point costs fitted as m N^2 (2r+1)^2 "
           f"(direct) and m Ws^2 log2 Ws^2 (FFT form) and extrapolated to all {n_cps} points and "
           f"{px_total / 1e6:.1f} Mpx of CFOG; {busy:.1f} core-s of oracle work in {wall:.1f} s wall")
    host = f"{cpu_model()}, {n_workers} of {os.cpu_count()} cores used"
    base = dict(value=round(n_cps / ((t_ext + t_direct) / n_workers), 3), unit="CP matches/s", cores=n_workers,
                kind="oracle", sample=smp, host=host,
                est_core_seconds=dict(cfog=round(t_ext, 1), direct_ssd=round(t_direct, 1)))
    fft = dict(value=round(n_cps / ((t_ext + t_sat + t_fft) / n_workers), 3), unit="CP matches/s",
               cores=n_workers, kind="oracle FFT form (FP64 numpy FFT + SAT energies)", sample=smp, host=host,
               est_core_seconds=dict(cfog=round(t_ext, 1), sat=round(t_sat, 1), fft_form=round(t_fft, 1)))
    cfog_rate = dict(mpx_per_s_per_core=round(px_s_core / 1e6, 3),
                     mpx_per_s=round(px_s_core * n_workers / 1e6, 3), cores=n_workers,
                     paper_mpx_per_s=round(PAPER_CFOG_MPX_S, 3),
                     paper_hardware="Intel Core i7-4710MQ @ 2.5 GHz, one 512^2 image in 0.210 s (Table III)",
                     sample=f"{len(tiles)} tiles of up to 512^2 from the workload's images", host=host)
    return base, fft, cfog_rate, sample, outs


# ------------------------------------------------------------ parity block
#
# The GPU result of each sampled point against the oracle's direct surface,
# with the rules of the parity tests: the surface within tol (E1 + E2(d)) per
# element; the offset equal to the oracle's, or an excused near-tie where the
# oracle's own values differ by at most tol (2 E1 + E2(d_gpu) + E2(d_ora)).

def parity_block(sample, outs, results, surfaces, pairs, tol: float, plan_of=None):
    exact = excused = mismatched = bad_status = 0
    worst = 0.0
    rel_max = 0.0
    fft_vs_direct = 0.0
    buckets = {}
    for (j, k), o in zip(sample, outs):
        r = pairs[j]["r"]
        S, E1, E2 = o["S"], o["E1"], o["E2"]
        fft_vs_direct = max(fft_vs_direct, float(np.max(np.abs(o["Sf"] - S) / (E1 + E2))))
        res = results[j]
        if int(res[k, 4]) != 0:
            bad_status += 1
            continue
        sg = surfaces[j][k].astype(np.float64)
        err = np.abs(sg - S) / (E1 + E2)
        worst = max(worst, float(err.max()))
        rel_max = max(rel_max, float(np.max(np.abs(sg - S)) / max(1e-300, float(np.max(np.abs(S))))))
        dxg, dyg = int(res[k, 0]), int(res[k, 1])
        io = int(np.argmin(S))
        dyo, dxo = divmod(io, 2 * r + 1)
        dxo, dyo = dxo - r, dyo - r
        if (dxg, dyg) == (dxo, dyo):
            exact += 1
        else:
            gap = S[dyg + r, dxg + r] - S.reshape(-1)[io]
            allow = tol * (2 * E1 + E2[dyg + r, dxg + r] + E2[dyo + r, dxo + r])
            if gap <= allow:
                excused += 1
            else:
                mismatched += 1
        if plan_of is not None:
            P = plan_of(j)
            buckets[P] = buckets.get(P, 0) + 1
    n = len(sample)
    out = dict(points=n, exact_offsets=exact, excused_near_ties=excused, mismatches=mismatched,
               status_not_ok=bad_status, excused_fraction=round(excused / max(1, n), 4),
               mismatch_rate=round(mismatched / max(1, n), 4),
               max_norm_ssd_err=float(f"{worst:.3e}"), max_rel_ssd_err=float(f"{rel_max:.3e}"),
               tol_norm=float(f"{tol:.4e}"), oracle_fft_vs_direct=float(f"{fft_vs_direct:.2e}"),
               reference="oracle direct SSD (Eq. 3) in FP64 on the sampled points; normalised error "
                     "|S_gpu - S_ora| / (E1 + E2(d))")
    if buckets:
        out["points_per_fft_size"] = {str(k): v for k, v in sorted(buckets.items())}
    return out


def self_consistency(results, surfaces, pairs):
    """Every point: its offset is the argmin of its own surface and its best
    value that surface's minimum; returns the number of points that fail."""
    bad = 0
    for res, surf, p in zip(results, surfaces, pairs):
        K = 2 * p["r"] + 1
        ok = res[:, 4] == 0
        flat = surf.reshape(len(res), -1)
        i = np.argmin(np.where(np.isnan(flat), np.inf, flat), axis=1)
        bad += int(np.sum(ok & ((i % K - p["r"] != res[:, 0]) | (i // K - p["r"] != res[:, 1]))))
        best = res[:, 2].view(np.float32)
        bad += int(np.sum(ok & (flat[np.arange(len(res)), i] != best)))
    return bad


def make_workload(name: str, speckle_shape: float = 4.0, gen_workers: int = -1):
    from paper_1808_06194_amd import synth
    if name in ("plain_2048", "plain_256"):
        w = dict(synth.PLAIN_2048 if name == "plain_2048" else synth.PLAIN_256)
        if speckle_shape != 4.0:
            w["spec"] = dataclasses.replace(w["spec"], speckle_shape=speckle_shape)
        A, B, s, cps, N, r = synth.plain_workload(w)
        return [dict(A=A, B=B, shift=s, cps=cps, N=N, r=r)]
    if name == "precision_4096":
        spec = synth.PairSpec(4096, 4096, 3200, (3.0, 40.0), 1200, 20, speckle_shape=speckle_shape)
        A, B, s = synth.make_pair(spec, (3, 0))
        cps = synth.random_cps(np.random.default_rng(np.random.SeedSequence([3, 1])), 4096, 4096, 128, 32, 10000)
        return [dict(A=A, B=B, shift=s, cps=cps, N=128, r=32)]
    if name == "batch_64":
        if gen_workers == 0:  # in this process (e.g. under a profiler that has set up the GPU already)
            return synth.batch_workload(n_pairs=64, speckle_shape=speckle_shape)
        from concurrent.futures import ProcessPoolExecutor
        import multiprocessing as mp
        nw = cpu_workers() if gen_workers < 0 else gen_workers
        with ProcessPoolExecutor(max_workers=nw, mp_context=mp.get_context("fork")) as ex:
            return synth.batch_workload(n_pairs=64, pool_map=ex.map, speckle_shape=speckle_shape)
    raise ValueError(name)


def describe(name: str, pairs) -> str:
    ncp = sum(len(p["cps"]) for p in pairs)
    if name == "plain_2048":
        return "plain_2048: 2048^2 pair, 400 CPs (20x20 grid), template 100, radius 20, m=9, sigma=0.8"
    if name == "plain_256":
        return "plain_256: 256^2 pair, 25 CPs (5x5 grid), template 48, radius 10, m=9, sigma=0.8"
    if name == "precision_4096":
        return "precision_4096: 4096^2 pair, 10000 random CPs, template 128, radius 32, m=9, sigma=0.8"
    return (f"batch_64: 64 pairs (sides 512-4096), {ncp} CPs, templates 40-120, radii 5-30, m=9, sigma=0.8; "
            "all pairs extracted and matched in one step")


MATCHER_SOURCES = ("match_fft.hip", "match_lane.hpp", "dft.hpp", "epilogue.hpp", "kernels.hpp", "window.hpp", "split_plan.hpp",
                   "abi.hip")


def matcher_digest() -> str:
    """sha256 over the sources the FFT matcher launches are built from."""
    h = hashlib.sha256()
    for f in MATCHER_SOURCES:
        with open(os.path.join(ROOT, "paper_1808_06194_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


EXTRACT_SOURCES = ("cfog_extract.hip", "kernels.hpp", "abi.hip")


def extract_digest() -> str:
    """sha256 over the sources the extraction launches are built from."""
    h = hashlib.sha256()
    for f in EXTRACT_SOURCES:
        with open(os.path.join(ROOT, "paper_1808_06194_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def traffic_record(kernel_key: str, digest=None):
    """HBM bytes per call measured by counters (profiles/traffic.json), if
    recorded for the current sources (matcher sources unless `digest` names
    others); None otherwise."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    try:
        with open(path) as f:
            rec = json.load(f)
        e = rec.get(kernel_key)
        if e and e.get("sources_sha256") == (digest or matcher_digest()):
            return e["bytes_per_launch"]
    except (OSError, ValueError):
        pass
    return None


def bf16_tol(N: int, r: int, m: int = 9) -> float:
    """Bound on |S_bf16(d) - S(d)| / (E1 + E2(d)) of the BF16 MFMA path:
    bf16 rounding of both operands (unit roundoff 2^-8) plus FP32 accumulation
    over the kernel's longest chain of additions, with sum |T S| <= (E1 + E2)/2
    and the final FP32 rounding of S (the derivation is in match_direct.hip)."""
    u, u32 = 2.0 ** -8, 2.0 ** -24
    L = m * (-(-(N + 2 * r) // 8)) * (-(-N // 32)) * 32 + 8
    gamma = L * u32 / (1.0 - L * u32)
    return (2 * u + u * u) + gamma * (1 + u) ** 2 + 2 * u32


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="batch_64",
                    choices=["batch_64", "plain_2048", "plain_256", "precision_4096", "serve", "harris_8192",
                             "reject_3000"])
    ap.add_argument("--path", choices=["plain", "batched", "fft", "mfma"], default=None)
    ap.add_argument("--descriptor", choices=["cfog", "scheme1", "fhog"], default="cfog")
    ap.add_argument("--speckle-shape", type=float, default=4.0,
                    help="shape of B's Gamma speckle (4: the workload recipe; larger is milder)")
    ap.add_argument("--no-cpu-baseline", action="store_true",
                    help="skip the oracle leg (then no cpu_baseline and no parity block)")
    ap.add_argument("--cpu-sample", type=int, default=256,
                    help="control points the oracle leg runs (and the parity block compares)")
    ap.add_argument("--gen-workers", type=int, default=-1,
                    help="processes generating batch_64 (-1: the host cores, 0: this process only)")
    ap.add_argument("--calib-copy-mib", type=int, default=0,
                    help="after the timed steps, run one plain device-to-device copy of this many MiB "
                         "(a counter calibration point for HBM traffic)")
    ap.add_argument("--serve-rates", default="200:15,1000:5,2000:4,4000:3,6000:3",
                    help="serve: rate:seconds phases (the first one gives the latency figures; the value is "
                         "the highest CP rate any phase served, which the last rate is meant to saturate)")
    ap.add_argument("--serve-pairs", type=int, default=32)
    ap.add_argument("--serve-budget-gib", type=float, default=0.0,
                    help="serve: device memory budget (0: 80%% of free memory)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: the benchmark runs on exactly one GPU (asked for --gpus {args.gpus}); "
              "the matching path shards by control point and needs no collectives", file=sys.stderr)
        sys.exit(2)
    if args.workload == "serve":
        run_serve(args)
        return
    if args.workload == "harris_8192":
        run_harris(args)
        return
    if args.workload == "reject_3000":
        run_reject(args)
        return

    t_gen = time.perf_counter()
    pairs = make_workload(args.workload, args.speckle_shape, args.gen_workers)  # before anything touches the GPU
    print(f"[bench] {args.workload}: {len(pairs)} pairs, {sum(len(p['cps']) for p in pairs)} CPs generated in "
          f"{time.perf_counter() - t_gen:.1f} s", file=sys.stderr, flush=True)
    desc = args.descriptor
    m = 36 if desc == "fhog" else 9
    cpu = None
    if not args.no_cpu_baseline:
        # the oracle leg, in forked workers before the GPU is initialised
        from concurrent.futures import ProcessPoolExecutor
        import multiprocessing as mp
        nw = cpu_workers()
        t_cpu = time.perf_counter()
        with ProcessPoolExecutor(max_workers=nw, mp_context=mp.get_context("fork")) as ex:
            cpu = cpu_leg(args.workload, pairs, m, desc, ex, nw, args.cpu_sample)
        print(f"[bench] oracle leg: {len(cpu[3])} points on {nw} cores in {time.perf_counter() - t_cpu:.1f} s",
              file=sys.stderr, flush=True)

    import torch
    from paper_1808_06194_amd import cfog

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    path = args.path or {"batch_64": "batched", "precision_4096": "fft"}.get(args.workload, "plain")
    path_flags = {"plain": cfog.PATH_PLAIN_FFT, "fft": cfog.PATH_PLAIN_FFT, "mfma": cfog.PATH_MFMA_BF16,
                  "batched": cfog.PATH_BATCHED_FFT | cfog.AUTOTUNE | cfog.USE_GRAPH}
    flags = path_flags[path]
    imgs, jobs = [], []
    for p in pairs:
        H, W = p["A"].shape
        dA, dB = torch.from_numpy(p["A"]).to(dev), torch.from_numpy(p["B"]).to(dev)
        vA = torch.empty((m, H, W), dtype=torch.float32, device=dev)
        vB = torch.empty_like(vA)
        sA = torch.empty((H + 1, W + 1), dtype=torch.float64, device=dev)
        sB = torch.empty_like(sA)
        imgs.append((dA, vA, sA))
        imgs.append((dB, vB, sB))
        jobs.append(cfog.Job(vA, sA, vB, sB, torch.from_numpy(p["cps"]).to(dev), p["N"], p["r"]))
    # CFOG volumes: all images in one batched extraction call (up to 8 images
    # per launch); pixel-wise HOG: the images on two streams (every second
    # image on the other one, each stream with its own workspace), joined
    # before matching
    ws_bytes = max(cfog.extract_workspace_size(*img[0].shape) for img in imgs)
    ws_ext = [torch.empty(ws_bytes, dtype=torch.uint8, device=dev) for _ in range(2)]
    ws_batch = torch.empty(max(1, cfog.extract_batch_workspace_size([img[0].shape for img in imgs])),
                           dtype=torch.uint8, device=dev)
    batch_imgs, batch_vols, batch_sats = ([img[k] for img in imgs] for k in range(3))
    n_cps = sum(len(p["cps"]) for p in pairs)
    stream = torch.cuda.current_stream()
    side = torch.cuda.Stream(device=dev)  # default priority
    fork, join = torch.cuda.Event(), torch.cuda.Event()
    ev = lambda: torch.cuda.Event(enable_timing=True)  # noqa: E731

    def extract(st=None):
        st = stream if st is None else st
        if desc == "fhog":
            fork.record(st)
            side.wait_event(fork)
            for i, (img, vol, sat) in enumerate(imgs):
                s2 = st if i % 2 == 0 else side
                cfog.fhog_extract(img, vol=vol, sat=sat, stream=s2, workspace=ws_ext[i % 2])
            join.record(side)
            st.wait_event(join)
        else:
            cfog.cfog_extract_batch(batch_imgs, m=m, vols=batch_vols, sats=batch_sats, stream=st,
                                    workspace=ws_batch, scheme=1 if desc == "scheme1" else 2)

    def step(evs=None):
        if evs:
            evs[0].record(stream)
        extract()
        if evs:
            evs[1].record(stream)
        cfog.match_batch(jobs, m=m, flags=flags, stream=stream)
        if evs:
            evs[2].record(stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    evs = [[ev(), ev(), ev()] for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        step(evs[i])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms = (t1 - t0) * 1e3 / args.steps
    step_ms = np.array([e[0].elapsed_time(e[2]) for e in evs])
    ext_ms = np.array([e[0].elapsed_time(e[1]) for e in evs])
    match_ms = np.array([e[1].elapsed_time(e[2]) for e in evs])
    t_match = float(np.mean(match_ms)) * 1e-3
    t_ext = float(np.mean(ext_ms)) * 1e-3
    timed_out = [j.out.cpu().numpy() for j in jobs]

    ok = recovered = 0
    for p, res in zip(pairs, timed_out):
        ok += int(np.sum(res[:, 4] == 0))
        recovered += int(np.sum(np.hypot(res[:, 0] - p["shift"][0], res[:, 1] - p["shift"][1]) <= 1.5))

    out = {
        "metric": "CP matches/sec (CFOG+3DFFT SSD) on 1 MI355X; p50/p99 match latency",
        "value": round(n_cps / (ms * 1e-3), 1),
        "unit": "CP matches/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16 x bf16 -> f32 (FP64 energies)" if path == "mfma" else "f32 (FP64 energies)",
        "data": "synthetic",
        "config": {"workload": describe(args.workload, pairs), "path": path, "n_cps": n_cps, "pairs": len(pairs),
                   "descriptor": {"cfog": "CFOG (Eq. 2)", "scheme1": "CFOG scheme 1 (binned orientations)",
                                  "fhog": "pixel-wise HOG, 36 channels, cell 4"}[desc], "m": m,
                   "speckle_shape": args.speckle_shape},
        "latency_ms": {"step_p50": round(float(np.percentile(step_ms, 50)), 4),
                       "step_p99": round(float(np.percentile(step_ms, 99)), 4),
                       "match_p50": round(float(np.percentile(match_ms, 50)), 4),
                       "match_p99": round(float(np.percentile(match_ms, 99)), 4),
                       "extract_p50": round(float(np.percentile(ext_ms, 50)), 4)},
        "match_only_cp_per_s": round(n_cps / t_match, 1),
        "recovered_1p5px": round(recovered / max(1, n_cps), 4),
        "cp_status_ok": ok,
    }

    # roofline of the matching call (all matcher launches of the step: one
    # per FFT-size bucket on forked streams, plus the split reduce), timed by
    # HIP events on the stream the call is issued on; the forked streams join
    # back before the closing event
    bytes_launch = sum(len(p["cps"]) * algorithmic_bytes_per_cp(p["N"], p["r"], m) for p in pairs)
    gbs = bytes_launch / t_match / 1e9
    hbm = dict(achieved=round(gbs, 1), peak=HBM_PEAK_GBS, unit="GB/s", frac=round(gbs / HBM_PEAK_GBS, 4))
    plans = {}
    if path == "mfma":
        flops = sum(len(p["cps"]) * direct_flops_per_cp(p["N"], p["r"], m) for p in pairs)
        tfs = flops / t_match / 1e12
        roof = dict(bound="mfma", achieved=round(tfs, 2), peak=BF16_PEAK_TFS, unit="TFLOP/s",
                    frac=round(tfs / BF16_PEAK_TFS, 4))
        kernel = "match_direct_kernel"
    else:
        flops = 0.0
        for p in pairs:
            P = cfog.plan_for(p["N"], p["r"], m)
            plans[(p["N"], p["r"])] = P
            flops += len(p["cps"]) * fft_flops_per_cp(p["N"], p["r"], P, m)
        tfs = flops / t_match / 1e12
        roof = dict(hbm)
        roof["bound"] = "hbm"
        Ps = sorted(set(plans.values()))
        kernel = ("match kernels of FFT side " + ",".join(str(P) for P in Ps) + " + split_reduce_kernel, one "
                  "match_batch call")
    key = f"{args.workload}:{path}" + ("" if desc == "cfog" else f":{desc}")
    traffic = traffic_record(key) if path != "mfma" else None
    roof.update(kernel=kernel, traffic=traffic, bytes_per_launch=bytes_launch, flops_per_launch=flops,
                launch_ms=round(t_match * 1e3, 4), hbm=hbm,
                alu=dict(achieved=round(tfs, 3), unit="TFLOP/s",
                         peak=BF16_PEAK_TFS if path == "mfma" else FP32_PEAK_TFS,
                         frac=round(tfs / (BF16_PEAK_TFS if path == "mfma" else FP32_PEAK_TFS), 4)))
    out["roofline"] = roof
    # the extraction call (every image of the step) against the HBM roofline
    ext_bytes = sum(i[0].numel() for i in imgs) * extract_bytes_per_px(m)
    egbs = ext_bytes / t_ext / 1e9
    ext_traffic = traffic_record(f"{args.workload}:extract", extract_digest()) if desc == "cfog" else None
    out["roofline_extract"] = dict(bound="hbm", achieved=round(egbs, 1), peak=HBM_PEAK_GBS, unit="GB/s",
                                   frac=round(egbs / HBM_PEAK_GBS, 4), bytes_per_launch=ext_bytes,
                                   traffic=ext_traffic, launch_ms=round(t_ext * 1e3, 4),
                                   kernel="cfog_extract_kernel + sat_carry_kernel + sat_fix_kernel, one "
                                          "cfog_extract_batch call" if desc != "fhog" else "fhog_kernel + SAT")

    # one more step with every surface written: the results must be the timed
    # ones bit for bit; the surfaces feed the self-consistency check and the
    # parity block
    surfs = []
    for j in jobs:
        K = 2 * j.r + 1
        j.surfaces = torch.empty((len(j.cps), K, K), dtype=torch.float32, device=dev)
        surfs.append(j.surfaces)
    cfog.match_batch(jobs, m=m, flags=flags, stream=stream)
    torch.cuda.synchronize()
    res_s = [j.out.cpu().numpy() for j in jobs]
    surf_np = [s.cpu().numpy() for s in surfs]
    same = all(np.array_equal(a, b) for a, b in zip(res_s, timed_out))
    out["check"] = {"surfaces_run_equals_timed": bool(same),
                    "self_consistency_failures": self_consistency(res_s, surf_np, pairs)}
    if cpu is not None:
        base, fft_base, cfog_rate, sample, outs = cpu
        out["cpu_baseline"] = base
        out["cpu_fft_baseline"] = fft_base
        out["cpu_cfog"] = cfog_rate
        tol = bf16_tol(pairs[0]["N"], pairs[0]["r"], m) if path == "mfma" else 1e-4
        plan_of = (lambda j: plans[(pairs[j]["N"], pairs[j]["r"])]) if plans else None
        blocks = {path: parity_block(sample, outs, res_s, surf_np, pairs, tol, plan_of)}
        if args.workload == "precision_4096":
            # the other precision path on the same points (untimed): FP32 FFT
            # against BF16 MFMA, each at its own bound
            other = "mfma" if path == "fft" else "fft"
            for j in jobs:
                j.out = None
            cfog.match_batch(jobs, m=m, flags=path_flags[other], stream=stream)
            torch.cuda.synchronize()
            res_o = [j.out.cpu().numpy() for j in jobs]
            surf_o = [s.cpu().numpy() for s in surfs]
            tol_o = bf16_tol(pairs[0]["N"], pairs[0]["r"], m) if other == "mfma" else 1e-4
            blocks[other] = parity_block(sample, outs, res_o, surf_o, pairs, tol_o)
            blocks[other]["self_consistency_failures"] = self_consistency(res_o, surf_o, pairs)
            blocks["offsets_fft_vs_mfma_differ"] = int(sum(np.sum(np.any(a[:, :2] != b[:, :2], axis=1))
                                                          for a, b in zip(res_s, res_o)))
        out["parity"] = blocks

    if not args.calib_copy_mib:  # (a counter run keeps its one calibration copy)
        # the counter-measured traffic of each call against the peak and
        # against what a plain copy reaches on this GPU
        probe = hbm_probe(dev)
        out["hbm_probe"] = probe
        for key, t_call in (("roofline", t_match), ("roofline_extract", t_ext)):
            tr = out[key].get("traffic")
            if tr:
                g = tr / t_call / 1e9
                out[key].update(traffic_gbs=round(g, 1), traffic_frac_peak=round(g / HBM_PEAK_GBS, 4),
                                traffic_frac_copy_probe=round(g / probe["copy_gbs"], 4))

    if args.calib_copy_mib:
        # source written first, then 1 GiB of other writes so that the copy's
        # reads come from HBM rather than the last-level cache
        nb = args.calib_copy_mib << 20
        src = torch.ones(nb // 4, dtype=torch.float32, device=dev)
        junk = torch.empty(1 << 28, dtype=torch.float32, device=dev)
        junk.fill_(2.0)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        out["calib_copy_bytes"] = nb
        del junk
    print(json.dumps(out), flush=True)


def hbm_probe(dev, mib: int = 1024, reps: int = 10) -> dict:
    """Achievable HBM bandwidth on this GPU, as context for the counter-measured
    traffic: a plain device-to-device copy (bytes read + written) and a fill
    (bytes written) of a `mib` MiB buffer, four times the last-level cache,
    timed with HIP events after the timed steps.  Measurement only: nothing
    on the path uses it."""
    import torch
    n = (mib << 20) // 4
    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(reps):
        dst.copy_(src)
    ev[1].record()
    for _ in range(reps):
        dst.fill_(1.0)
    ev[2].record()
    torch.cuda.synchronize()
    t_copy = ev[0].elapsed_time(ev[1]) / reps * 1e-3
    t_fill = ev[1].elapsed_time(ev[2]) / reps * 1e-3
    nb = n * 4
    del src, dst
    return dict(copy_gbs=round(2 * nb / t_copy / 1e9, 1), fill_gbs=round(nb / t_fill / 1e9, 1), bytes=nb,
                kernel=f"torch copy_ and fill_ of a {mib} MiB fp32 buffer (the copy counts bytes read + written)")


def harris_flops_per_px(R: int = 4) -> int:
    """Flops per chip pixel: gradients (2), the three products (3), two
    Gaussian passes of 2R+1 taps on three channels (2 x 3 x 2 (2R+1)) and the
    response (6)."""
    return 2 + 3 + 12 * (2 * R + 1) + 6


def run_harris(args):
    from paper_1808_06194_amd import synth
    A, _, _ = synth.make_pair(synth.area_scaled_spec(8192, 8), (5, 0))
    import torch
    from paper_1808_06194_amd import cfog
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    img = torch.from_numpy(A).to(dev)
    n, k, chip = 128, 4, 60
    stream = torch.cuda.current_stream()
    for _ in range(args.warmup):
        cfog.harris_grid(img, n, k, chip, stream=stream)
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    t0 = time.perf_counter()
    for e0, e1 in evs:
        e0.record(stream)
        cfog.harris_grid(img, n, k, chip, stream=stream)
        e1.record(stream)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    kms = np.array([e0.elapsed_time(e1) for e0, e1 in evs])
    t = float(np.mean(kms)) * 1e-3
    chips = n * n
    pts = chips * k
    bytes_launch = chips * chip * chip * 4 + pts * 20
    flops = chips * chip * chip * harris_flops_per_px()
    gbs, tfs = bytes_launch / t / 1e9, flops / t / 1e12
    hbm = dict(achieved=round(gbs, 1), peak=HBM_PEAK_GBS, unit="GB/s", frac=round(gbs / HBM_PEAK_GBS, 4))
    alu = dict(achieved=round(tfs, 3), peak=FP32_PEAK_TFS, unit="TFLOP/s", frac=round(tfs / FP32_PEAK_TFS, 4))
    roof = dict(alu, bound="alu") if flops / (FP32_PEAK_TFS * 1e12) > bytes_launch / (HBM_PEAK_GBS * 1e9) \
        else dict(hbm, bound="hbm")
    roof.update(kernel="harris_grid_kernel", traffic=None, bytes_per_launch=bytes_launch, flops_per_launch=flops,
                hbm=hbm, alu=alu)
    out = {
        "metric": "Harris feature points/s (block-based, Section IV) on 1 MI355X",
        "value": round(pts / t, 1), "unit": "feature points/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "harris_8192: one 8192^2 image, 128 x 128 cells, 60 x 60 chips, 4 points per chip, "
                               "sigma 1, kappa 0.04", "chips": chips, "points": pts},
        "latency_ms": {"p50": round(float(np.percentile(kms, 50)), 4), "p99": round(float(np.percentile(kms, 99)), 4)},
        "roofline": roof,
    }
    print(json.dumps(out), flush=True)


def run_reject(args):
    from paper_1808_06194_amd import synth
    P, Q = synth.reject_points(np.random.default_rng(np.random.SeedSequence([6, 0])), 3000, 150)
    import torch
    from paper_1808_06194_amd import cfog
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    dP, dQ = torch.from_numpy(P).to(dev), torch.from_numpy(Q).to(dev)
    keep = torch.empty(len(P), dtype=torch.uint8, device=dev)
    res = torch.empty(27, dtype=torch.float64, device=dev)  # one cfog_reject_result (216 bytes)
    stream = torch.cuda.current_stream()
    for _ in range(args.warmup):
        cfog.reject_outliers(dP, dQ, 1.0, stream=stream, keep=keep, result=res, sync=False)
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    t0 = time.perf_counter()
    for e0, e1 in evs:
        e0.record(stream)
        cfog.reject_outliers(dP, dQ, 1.0, stream=stream, keep=keep, result=res, sync=False)
        e1.record(stream)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    kms = np.array([e0.elapsed_time(e1) for e0, e1 in evs])
    t = float(np.mean(kms)) * 1e-3
    info = cfog.reject_result_dict(res)
    iters = info["removed"] + 1
    # per iteration and kept point: 10 monomials (10 flops), the 55 + 20
    # normal-equation products and sums (150), the model evaluation and the
    # residual (45); the 10 x 10 Cholesky per iteration is negligible
    n = len(P)
    flops = sum((n - i) * 205.0 for i in range(iters))
    tfs = flops / t / 1e12
    FP64_PEAK_TFS = 78.6
    roof = dict(bound="alu", achieved=round(tfs, 5), peak=FP64_PEAK_TFS, unit="TFLOP/s",
                frac=round(tfs / FP64_PEAK_TFS, 6), kernel="reject_kernel (one workgroup per point set)",
                traffic=None, flops_per_launch=flops, iterations=iters,
                one_cu_peak_tfs=round(FP64_PEAK_TFS / 256, 4),
                one_cu_frac=round(tfs / (FP64_PEAK_TFS / 256), 4))
    out = {
        "metric": "outlier-rejection point sets/s (cubic model, Section IV) on 1 MI355X",
        "value": round(1.0 / t, 2), "unit": "point sets/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
        "config": {"workload": "reject_3000: 3000 matched points, 150 gross outliers, threshold 1 px",
                   "points": n, "removed": info["removed"], "rmse": info["rmse"]},
        "latency_ms": {"p50": round(float(np.percentile(kms, 50)), 4),
                       "p99": round(float(np.percentile(kms, 99)), 4)},
        "roofline": roof,
    }
    print(json.dumps(out), flush=True)


def run_serve(args):
    from concurrent.futures import ProcessPoolExecutor
    import multiprocessing as mp
    from paper_1808_06194_amd import synth
    n_pairs = args.serve_pairs
    sides = synth.SERVE_SIDES[:n_pairs] if n_pairs <= len(synth.SERVE_SIDES) else None
    if sides is None:
        raise SystemExit("--serve-pairs above 32")
    t_gen = time.perf_counter()
    # generated in forked workers before anything touches the GPU
    with ProcessPoolExecutor(max_workers=8, mp_context=mp.get_context("fork")) as ex:
        pairs = list(ex.map(synth.serve_pair, range(n_pairs)))
    print(f"[serve] generated {n_pairs} pairs in {time.perf_counter() - t_gen:.1f} s", file=sys.stderr, flush=True)

    import torch
    from paper_1808_06194_amd import cfog
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    imgs = [(torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev)) for A, B, _ in pairs]
    torch.cuda.synchronize()
    free, _ = torch.cuda.mem_get_info()
    budget = int(args.serve_budget_gib * (1 << 30)) if args.serve_budget_gib else int(free * 0.8)
    srv = cfog.Server(budget, n_slots=4, max_batch_cps=8192, max_batch_reqs=256)
    for a, b in imgs:
        srv.add_pair(a, b)
    # make every volume resident (first use extracts it)
    t_ext = time.perf_counter()
    warm = [srv.submit(j, np.array([[s // 2] * 4], np.int32), 40, 5) for j, s in enumerate(sides)]
    srv.wait(warm, timeout_s=300)
    print(f"[serve] {n_pairs} pairs resident in {time.perf_counter() - t_ext:.2f} s", file=sys.stderr, flush=True)

    def phase(rate, seconds, seed, keep=()):
        reqs = synth.serve_requests(max(1, int(rate * seconds)), rate, sides, seed=seed)
        t0 = time.monotonic_ns() + 20_000_000
        meta, done, i = {}, {}, 0
        while len(done) < len(reqs):
            now = time.monotonic_ns()
            while i < len(reqs) and t0 + int(reqs[i]["t"] * 1e9) <= now:
                q = reqs[i]
                rid = srv.submit(q["pair"], q["cps"], q["N"], q["r"])
                meta[rid] = (t0 + int(q["t"] * 1e9), i)
                i += 1
            for c in srv.poll(timeout_us=0 if i < len(reqs) else 2000):
                done[c.id] = c
            if i < len(reqs):
                gap = t0 + int(reqs[i]["t"] * 1e9) - time.monotonic_ns()
                if gap > 100_000:
                    time.sleep(min(gap, 1_000_000) * 1e-9)
        lat = np.array([(c.t_done - meta[k][0]) * 1e-6 for k, c in done.items()])
        t_end = max(c.t_done for c in done.values())
        ncp = sum(len(q["cps"]) for q in reqs)
        bad = sum(c.status != 0 for c in done.values())
        rec = dict(rate_req_s=rate, seconds=seconds, requests=len(reqs), cps=ncp, failed=bad,
                   cp_per_s=round(ncp / ((t_end - t0) * 1e-9), 1),
                   req_per_s=round(len(reqs) / ((t_end - t0) * 1e-9), 1),
                   p50_ms=round(float(np.percentile(lat, 50)), 3), p99_ms=round(float(np.percentile(lat, 99)), 3),
                   p999_ms=round(float(np.percentile(lat, 99.9)), 3),
                   mean_batch_reqs=round(float(np.mean([c.batch_reqs for c in done.values()])), 2))
        kept = {meta[k][1]: c for k, c in done.items() if meta[k][1] in keep}
        print(f"[serve] {rec}", file=sys.stderr, flush=True)
        return rec, reqs, kept

    phases, first = [], None
    sample = set(range(0, 10 ** 6, 37))
    for k, spec in enumerate(args.serve_rates.split(",")):
        rate, sec = (float(v) for v in spec.split(":"))
        rec, reqs, kept = phase(rate, sec, 1000 + k, keep=sample)
        phases.append(rec)
        if first is None:
            first = (rec, reqs, kept)
    # alone vs in the mix: the sampled requests of the first phase, one at a time
    rec0, reqs0, kept0 = first
    same = recovered = total = 0
    for i, c_mix in sorted(kept0.items())[:64]:
        q = reqs0[i]
        rid = srv.submit(q["pair"], q["cps"], q["N"], q["r"])
        c = srv.wait([rid])[rid]
        same += int(np.array_equal(c.out, c_mix.out))
        res = cfog.results_np(c.out)
        sx, sy = pairs[q["pair"]][2]
        recovered += int(np.sum(np.hypot(res["dx"] - sx, res["dy"] - sy) <= 1.5))
        total += len(q["cps"])
    n_alone = min(64, len(kept0))
    st = srv.stats()
    srv.close()
    best = max(phases, key=lambda p: p["cp_per_s"])
    out = {
        "metric": "CP matches/sec (CFOG+3DFFT SSD) on 1 MI355X; p50/p99 match latency",
        "value": best["cp_per_s"],
        "unit": "CP matches/s",
        "n_gpus": 1, "steps": len(phases), "warmup": n_pairs,
        "ms_per_step": None,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 (FP64 energies)", "data": "synthetic",
        "config": {"workload": f"serve: {n_pairs} resident pairs (8 each of 1024^2, 2048^2, 4096^2, 8192^2), "
                               "Poisson requests of 1-500 CPs, template 40-128, radius 5-32, m=9, sigma=0.8",
                   "path": "server (batched FFT, 4 slots)", "budget_bytes": budget},
        "latency_ms": {"p50": rec0["p50_ms"], "p99": rec0["p99_ms"], "p999": rec0["p999_ms"],
                       "at_req_per_s": rec0["rate_req_s"]},
        "phases": phases,
        "alone_vs_mix": {"requests": n_alone, "bit_identical": same},
        "recovered_1p5px": round(recovered / max(1, total), 4),
        "server": st,
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
