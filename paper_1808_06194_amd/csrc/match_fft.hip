// SSD template matching of control points in the frequency domain
// (Section III-G of Ye et al.: Eqs. 3-6 and 8-9), one workgroup per control
// point at a time, everything on chip.
//
// For control point (x, y) in A with search centre (bx, by) in B, template side
// N, radius r, h = N/2, K = 2r+1, Ws = N + 2r:
//   T_c  = D_A[c][y-h .. y-h+N)[x-h .. x-h+N)               (template)
//   S_c  = D_B[c][by-h-r .. +Ws)[bx-h-r .. +Ws)              (search window)
//   C(u) = sum_c sum_q T_c(q) S_c(q+u),  u in [0, 2r]^2        (correlation)
//   SSD(d) = E1 + E2(d) - 2 C(d + r)                          (Eq. 5)
// with E1, E2 from the FP64 summed-area tables and d = u - r the returned
// offset of B's window relative to the search centre.
//
// The orientation axis of Eq. 9's 3-D transform is only ever read back at
// zero orientation shift, where the orientation DFT / inverse DFT pair reduces
// (Parseval) to a plain sum over channels of 2-D spectral products.  So each
// channel goes through real 2-D FFTs of size P x P (P >= Ws):
//   x-pass: rows of T_c (or S_c), two real rows packed per complex FFT, the
//           two half-spectra separated via Z(k) and conj Z(-k);
//   y-pass: complex column FFTs of the half-spectrum kx in [0, P/2];
//   ACC(ky, kx) += conj(T^_c) * S^_c  in registers, T^_c parked in registers
//           between the T and S passes of the channel;
// then one inverse: column IFFTs (kept rows u_y < K) and a C2R row IFFT with
// two output rows packed per complex FFT (kept columns u_x < K), the SSD
// assembly in FP64, and a lexicographic argmin + second-best over (SSD, index).
//
// Two kernels share this scheme: this file's (windows up to 48, where one control
// point's transforms fit a few waves) and match_lane.hpp's (larger ones).
//
// Execution: every 1-D FFT of length P = R1 * R2 is owned by a group of
// G = max(R1, R2) lanes of one wave:
//   stage 1 (lane j < R2):  t[j R1 + k1] = sum_a x[j + R2 a] W_R1^{a k1}
//   stage 2 (lane k1 < R1): X[k1 + R1 k2] = sum_j W_P^{k1 j} t[j R1 + k1] W_R2^{j k2}
// with the small DFTs as unrolled register codelets (dft.hpp), the twiddles
// W_P^{k1 j} formed by recurrence from W_P^{k1}, and the exchange between
// stages through the FFT's own LDS row or column, with t at positions that
// keep a group's accesses in distinct banks (s1_pos, s1c).  Only the x -> y
// transposes need workgroup barriers (4 per channel).
#include <hip/hip_runtime.h>
#include <limits.h>
#include <algorithm>
#include <mutex>
#include <vector>
#include "dft.hpp"
#include "epilogue.hpp"
#include "kernels.hpp"
#include "match_lane.hpp"
#include "window.hpp"

namespace cfog {

// Orders the LDS accesses of one wave (the hardware keeps a wave's LDS
// operations in order; this stops the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// An integer the compiler must treat as computed here: addresses derived
// from it are rebuilt near their use instead of being hoisted out of the
// task loop and kept live (which costs registers).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <int P_, int R1_, int R2_, int NT_>
struct FftCfg {
  static constexpr int P = P_, R1 = R1_, R2 = R2_, NT = NT_;
  static_assert(P == R1 * R2, "P must equal R1 * R2");
  static_assert(NT % 64 == 0 && NT <= 1024, "bad workgroup size");
  static constexpr int PH = P / 2 + 1;
  static constexpr int G = R1 > R2 ? R1 : R2;  // lanes per FFT group
  static constexpr int GPW = 64 / G;           // groups per wave
  static constexpr int NW = NT / 64;
  static constexpr int NG = NW * GPW;          // groups per workgroup
  static constexpr int KF = (PH + NG - 1) / NG;  // column rounds per group
  static constexpr size_t LDS = sizeof(float2) * ((size_t)P * PH + P) + NW * 16;
};

// Lane identity within the FFT group layout.
template <class C>
struct Lane {
  int g;   // group index in the workgroup (>= NG for idle lanes)
  int li;  // lane index in the group
  __device__ __forceinline__ Lane() {
    const int lane = threadIdx.x & 63, gi = lane / C::G;
    li = lane - gi * C::G;
    g = gi < C::GPW ? (int)(threadIdx.x >> 6) * C::GPW + gi : INT_MAX / 2;
  }
};

// The inputs of a stage-2 DFT of lane k1: w[b] = get(b) W_P^{-k1 b} (INV:
// W_P^{+k1 b}).  The twiddles come by recurrence from W_P^{k1}: one LDS read
// instead of R2 - 1 (3% faster at P = 144, 15% at P = 192, when those sides took
// this layout), at most R2 - 2 more FP32 roundings in each.
template <class C, bool INV, class Get>
__device__ __forceinline__ void stage2_inputs(float2 (&w)[C::R2], const float2* tw, int k1, Get&& get) {
  float2 t1 = tw[C::R1 + k1];
  if (INV) t1.y = -t1.y;
  float2 t = t1;
  w[0] = get(0);
#pragma unroll
  for (int b = 1; b < C::R2; ++b) {
    if (b > 1) t = cmul(t, t1);
    w[b] = cmul(get(b), t);
  }
}

// Where lane j of an x-pass group leaves stage-1 output k in its pair's row
// buffer (2 PH = P + 2 slots), chosen so that neither the group's writes
// (fixed k) nor its stage-2 reads (fixed j) share LDS banks: j R1 + k plus
// j / 4 (unpadded, the stride R1 puts lanes j and j + 32 / R1 in one bank).
template <class C>
__device__ __forceinline__ int s1_pos(int j, int k) {
  static_assert((C::R2 - 1) / 4 <= 2, "the stage-1 outputs must fit the pair's two rows");
  return j * C::R1 + k + (j >> 2);
}

// Where lane j of a column FFT leaves its stage-1 output k: row k R2 + j of
// the column, i.e. back in the rows it read (j + R2 a), so stage 1 is in place
// per lane and consecutive lanes write consecutive rows; stage 2 then reads
// rows k1 R2 + b.  (The natural order, row j R1 + k, puts a group's writes
// R1 rows apart, in few LDS banks.)
template <class C>
__device__ __forceinline__ int s1c(int j, int k) { return k * C::R2 + j; }

// One set of rows for the x-pass: nrows x ncols real values at src (leading
// dim ld), transformed into X (row stride PH).
struct XRows {
  const float* src;
  int64_t ld;
  int nrows, ncols;
  float2* X;
};

// x-pass: forward FFTs of the rows, zero-padded to P, two rows per complex FFT;
// leaves the half-spectra of the rows in X as [row][kx], kx in [0, P/2].
template <class C>
__device__ __forceinline__ void xpass_fwd(const Lane<C>& L, const XRows& R, const float2* tw) {
  constexpr int R1 = C::R1, R2 = C::R2, PH = C::PH;
  const int total = (R.nrows + 1) >> 1;
  // each pair is loaded just before its transform: a group has one or two
  for (int q = L.g; q < total; q += C::NG) {
    float2* base = R.X + 2 * opaque(q) * PH;
    if (L.li < R2) {
      const int j = L.li;
      const float* r0 = R.src + (int64_t)(2 * q) * R.ld;
      const bool has1 = (2 * q + 1) < R.nrows;
      float2 v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) {
        const int xx = j + R2 * a;
        float re = 0.f, im = 0.f;
        if (xx < R.ncols) {
          re = ldg(r0 + xx);
          if (has1) im = ldg(r0 + R.ld + xx);
        }
        v[a] = make_float2(re, im);
      }
      dft<R1, -1>(v);
#pragma unroll
      for (int k = 0; k < R1; ++k) base[s1_pos<C>(j, k)] = v[k];
    }
    wave_sync();
    xpass_stage2<C>(L, base, q, R.nrows, tw);
  }
  // rows [2 ceil(nrows/2), P) are zero padding (an odd last row is zeroed by
  // its pair)
  for (int t = threadIdx.x; t < (C::P - 2 * total) * PH; t += C::NT) R.X[2 * total * PH + t] = make_float2(0.f, 0.f);
}

// Stage 2 of the row FFT of pair q at base (stage 1 done), then the
// separation of the two packed rows into their half-spectra.
template <class C>
__device__ __forceinline__ void xpass_stage2(const Lane<C>& L, float2* base, int q, int nrows, const float2* tw) {
  constexpr int P = C::P, R1 = C::R1, R2 = C::R2, PH = C::PH;
  {
    // stage 2 on every lane of the group (idle lanes duplicate lane R1-1 so the
    // cross-lane fetch below runs with the whole wave active)
    const int k1 = L.li < R1 ? L.li : R1 - 1;
    float2 v[R2];
    stage2_inputs<C, false>(v, tw, k1, [&](int b) { return base[s1_pos<C>(b, k1)]; });
    dft<R2, -1>(v);
    // separate the packed rows: 2 A(k) = Z(k) + conj Z(-k), 2 B(k) = (Z(k) - conj Z(-k)) / i
    // (the factor 2 of both spectra, 4 in their product, is taken out by the
    // inverse's normalisation: exact, being a power of two).
    // Z(-k) for k = k1 + R1 k2 is Z((R1-k1) + R1 (R2-1-k2)), i.e. register R2-1-k2 of
    // lane R1-k1 of the group (k1 > 0), or this lane's register (R2-k2) mod R2 (k1 = 0).
    const int lane = threadIdx.x & 63;
    const int msrc = lane - L.li + (k1 == 0 ? 0 : R1 - k1);
    // the value of lane R1 - k1 of the group: where the group is a DPP half row
    // (R1 = 8), a mirror within it and a shift by one lane (lane i then holds
    // lane R1 - i's value; lane 0's is not used), on the vector units; otherwise
    // an LDS permute
    auto from_mirror = [&](float x) -> float {
      if constexpr (C::G == R1 && R1 == 8) {
        const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, false);  // row_half_mirror
        return __int_as_float(__builtin_amdgcn_update_dpp(0, t, 0x111, 0xf, 0xf, false));  // row_shr:1
      } else {
        return __shfl(x, msrc, 64);
      }
    };
    const bool odd_pad = (2 * q + 1) >= nrows;  // second row of the pair is padding
    static_for<0, R2>([&](auto k2I) {
      constexpr int k2 = decltype(k2I)::value;
      const float2 far = make_float2(from_mirror(v[R2 - 1 - k2].x), from_mirror(v[R2 - 1 - k2].y));
      const float2 zm = (k1 == 0) ? v[(R2 - k2) % R2] : far;
      const int k = k1 + R1 * k2;
      if (L.li < R1 && k <= P / 2) {
        const float2 z = v[k2];
        base[k] = make_float2(z.x + zm.x, z.y - zm.y);
        base[PH + k] = odd_pad ? make_float2(0.f, 0.f) : make_float2(z.y + zm.y, zm.x - z.x);
      }
    });
    wave_sync();
  }
}

// y-pass: forward column FFTs of the half-spectrum (rows >= nrows were zeroed
// by the x-pass).
// Column kx = g + rnd * NG; lane k1 < R1 of its group ends up with
// ky = k1 + R1 k2 and hands each value to sink(rnd, k2, value).
template <class C, class Sink>
__device__ __forceinline__ void ypass_fwd(const Lane<C>& L, float2* X, const float2* tw, Sink&& sink) {
  constexpr int R1 = C::R1, R2 = C::R2, PH = C::PH;
  static_for<0, C::KF>([&](auto rndI) {
    constexpr int rnd = decltype(rndI)::value;
    const int kx = L.g + rnd * C::NG;
    if (kx < PH) {
      float2* col = X + opaque(kx);
      if (L.li < R2) {
        const int j = L.li;
        float2 v[R1];
#pragma unroll
        for (int a = 0; a < R1; ++a) v[a] = col[(j + R2 * a) * PH];
        dft<R1, -1>(v);
#pragma unroll
        for (int k = 0; k < R1; ++k) col[s1c<C>(j, k) * PH] = v[k];
      }
      wave_sync();
      if (L.li < R1) {
        const int k1 = L.li;
        float2 w[R2];
        stage2_inputs<C, false>(w, tw, k1, [&](int b) { return col[s1c<C>(b, k1) * PH]; });
        dft<R2, -1>(w);
        static_for<0, R2>([&](auto k2I) { sink(rndI, k2I, w[decltype(k2I)::value]); });
      }
    }
  });
}

// Control point cpi of job jd over the channels [c0, c1).  part == nullptr:
// the whole sum, finished by the epilogue; otherwise the partial correlation
// surface goes to part (item g of a split task; item 0 reports an
// out-of-bounds point).
template <class C>
__device__ __forceinline__ void match_one(const Lane<C>& L, const MatchJob& jd, int cpi, float2* X, const float2* tw,
                          ArgminState* red, int c0, int c1, float* __restrict__ part, int g) {
  constexpr int P = C::P, R1 = C::R1, R2 = C::R2, PH = C::PH, NT = C::NT, KF = C::KF;
  const int4 cp = jd.cps[cpi];
  const int N = jd.N, r = jd.r, K = 2 * r + 1, Ws = N + 2 * r;
  const CpBoxes bx = cp_boxes(cp.x, cp.y, cp.z, cp.w, N, r, jd.hA, jd.wA, jd.hB, jd.wB);
  if (!bx.inside) {
    if (g == 0) oob_result<NT>(jd, cpi);
    return;
  }
  const int tx0 = bx.tx0, ty0 = bx.ty0, sx0 = bx.sx0, sy0 = bx.sy0;

  float2 acc[KF][R2];
#pragma unroll
  for (int k = 0; k < KF; ++k)
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) acc[k][k2] = make_float2(0.f, 0.f);

  const size_t planeA = (size_t)jd.hA * jd.wA, planeB = (size_t)jd.hB * jd.wB;
  const float* tA = jd.volA + (size_t)ty0 * jd.wA + tx0;
  const float* sB = jd.volB + (size_t)sy0 * jd.wB + sx0;
  // T^ is parked in registers between the template's and the window's passes;
  // four barriers per channel
  for (int c = c0; c < c1; ++c) {
    float2 th[KF][R2];
    __syncthreads();  // previous readers of X are done
    xpass_fwd<C>(L, XRows{tA + c * planeA, jd.wA, N, N, X}, tw);
    __syncthreads();
    ypass_fwd<C>(L, X, tw, [&](auto rndI, auto k2I, float2 v) { th[decltype(rndI)::value][decltype(k2I)::value] = v; });
    __syncthreads();
    xpass_fwd<C>(L, XRows{sB + c * planeB, jd.wB, Ws, Ws, X}, tw);
    __syncthreads();
    ypass_fwd<C>(L, X, tw, [&](auto rndI, auto k2I, float2 v) {
      constexpr int rnd = decltype(rndI)::value, k2 = decltype(k2I)::value;
      acc[rnd][k2] = cmac_conj(acc[rnd][k2], th[rnd][k2], v);
    });
  }

  // ---- inverse along y: each group transforms its own columns in place and
  // keeps the rows u_y < K (no workgroup barrier: a column is group-private).
#pragma unroll
  for (int rnd = 0; rnd < KF; ++rnd) {
    const int kx = L.g + rnd * C::NG;
    if (kx < PH) {
      float2* col = X + opaque(kx);
      if (L.li < R1) {
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) col[(L.li + R1 * k2) * PH] = acc[rnd][k2];
      }
      wave_sync();
      if (L.li < R2) {
        const int j = L.li;
        float2 v[R1];
#pragma unroll
        for (int a = 0; a < R1; ++a) v[a] = col[(j + R2 * a) * PH];
        dft<R1, +1>(v);
#pragma unroll
        for (int k = 0; k < R1; ++k) col[s1c<C>(j, k) * PH] = v[k];
      }
      wave_sync();
      if (L.li < R1) {
        const int k1 = L.li;
        float2 w[R2];
        stage2_inputs<C, true>(w, tw, k1, [&](int b) { return col[s1c<C>(b, k1) * PH]; });
        dft<R2, +1>(w);
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
          const int uy = k1 + R1 * k2;
          if (uy < K) col[uy * PH] = w[k2];
        }
      }
    }
  }
  __syncthreads();

  // ---- inverse along x: C2R, two output rows per complex FFT, kept u_x < K.
  // A pair's stage-1 outputs overwrite its own two input rows (2 PH >= P
  // slots, read into registers by the same wave first); the correlation
  // C(u_y, u_x) goes to LDS behind all the pairs' rows.
  const int npair = (K + 1) >> 1;
  float* Cs = reinterpret_cast<float*>(X + 2 * npair * PH);
  // 1/P^2 of the inverse 2-D DFT and 1/4 for the doubled row spectra of T and S
  const float inv = 0.25f / ((float)P * (float)P);
  for (int p = L.g; p < npair; p += C::NG) {
    float2* sc = X + 2 * opaque(p) * PH;
    float2 v[R1];
    if (L.li < R2) {
      const int j = L.li;
      const float2* v1r = X + (2 * p) * PH;
      const bool has2 = 2 * p + 1 < K;
#pragma unroll
      for (int a = 0; a < R1; ++a) {
        const int kx = j + R2 * a;
        const bool lo = kx <= P / 2;
        const int kk = lo ? kx : P - kx;
        const float2 v1 = v1r[kk];
        const float2 v2 = has2 ? v1r[PH + kk] : make_float2(0.f, 0.f);
        v[a] = lo ? make_float2(v1.x - v2.y, v1.y + v2.x) : make_float2(v1.x + v2.y, v2.x - v1.y);
      }
    }
    wave_sync();  // every read of the pair's rows precedes the writes into them
    if (L.li < R2) {
      dft<R1, +1>(v);
#pragma unroll
      for (int k = 0; k < R1; ++k) sc[L.li * R1 + k] = v[k];
    }
    wave_sync();
    if (L.li < R1) {
      const int k1 = L.li;
      float2 w[R2];
      stage2_inputs<C, true>(w, tw, k1, [&](int b) { return sc[k1 + R1 * b]; });
      dft<R2, +1>(w);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) {
        const int ux = k1 + R1 * k2;
        if (ux < K) {
          Cs[(2 * p) * K + ux] = w[k2].x * inv;
          if (2 * p + 1 < K) Cs[(2 * p + 1) * K + ux] = w[k2].y * inv;
        }
      }
    }
  }
  __syncthreads();

  if (part) {
    for (int i = threadIdx.x; i < K * K; i += NT) stg(part + i, Cs[i]);
    return;
  }
  ssd_epilogue<NT>(jd, cpi, tx0, ty0, sx0, sy0, Cs, red);
}

// One kernel for both paths: with jobs == nullptr every task t is control
// point t of job0 (plain path); otherwise task t = tasks[t] = (job, cp) over the
// device job table (batched path).  Workgroups loop over tasks with a grid
// stride.
template <class C>
__global__ __launch_bounds__(C::NT) void match_fft_kernel(MatchJob job0, const MatchJob* __restrict__ jobs,
                                                          const int2* __restrict__ tasks, int n_tasks,
                                                          SplitArgs sp) {
  extern __shared__ float2 smem[];
  float2* X = smem;
  float2* tw = X + C::P * C::PH;
  ArgminState* red = reinterpret_cast<ArgminState*>(tw + C::P);
  // stage-2 twiddles W_P^{k1 b} stored lane-major, tw[b * R1 + k1] (stage 2
  // reads row b = 1 and forms the other powers)
  for (int i = threadIdx.x; i < C::P; i += C::NT) {
    const int b = i / C::R1, k1 = i - b * C::R1;
    double s, c;
    sincospi(2.0 * (double)((k1 * b) % C::P) / C::P, &s, &c);
    tw[i] = make_float2((float)c, (float)-s);
  }
  const Lane<C> L;
  const int n_items = split_items(n_tasks, sp);
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    __syncthreads();  // twiddles ready / previous task's reduction done
    int t = it, g = 0, G = 1;
    if (sp.G > 1 && it >= sp.n_whole) {  // an item of a split task
      const int s = it - sp.n_whole;
      t = sp.n_whole + s / sp.G;
      g = s - (t - sp.n_whole) * sp.G;
      G = sp.G;
    }
    MatchJob jd = job0;
    int cpi = t;
    if (jobs) {
      const int2 tk = tasks[t];
      jd = jobs[tk.x];
      cpi = tk.y;
    }
    float* part = G > 1 ? sp.part + (size_t)(it - sp.n_whole) * sp.slot : nullptr;
    match_one<C>(L, jd, cpi, X, tw, red, g * jd.m / G, (g + 1) * jd.m / G, part, g);
  }
}

// ------------------------------------------------------------------ plans
//  Group layout, G(P, R1, R2, NT): R1 >= R2 keeps the per-lane outputs of
//  stage 2 small; NT from measurement: as many waves as the registers allow,
//  in workgroups that fill a CU's wave slots.  P = 32..48 were level with the
//  lane layout (46-50, 55-60 and 67-71 against 49, 57 and 65 us per 1,024
//  points): there a point is a few waves' work on either.
//  Lane layout, L((P, R1, R2, RA, RB, I1, I2), full, spread), each a workgroup
//  (NT, PF, waves per SIMD, SEP): from 49 up, per 1,024 points of template N and
//  radius r, unsplit, before (the group layout) and after:
//    N, r     P   before  after     N, r     P   before  after
//    44,  8   60   127 ->  66 us    72, 12   96   311 -> 170 us
//    44,  9   64   116 ->  85       70, 15  100   290 -> 195
//    52, 10   72   249 ->  89       80, 14  108   319 -> 202
//    60, 10   80   228 -> 127       80, 20  120   362 -> 246
//    66, 12   90   251 -> 162      100, 20  144   494 -> 400
//                                  118, 20  160   707 -> 498
//                                  128, 32  192   882 -> 809
//  The factors keep the wave-sized pieces of each phase at a multiple of four
//  (a SIMD each) and the x2 items at one or two to a thread; up to P = 120 two
//  or more workgroups share a CU (16 waves at 128 VGPRs, so NT and WPE), above
//  it one has the plane to itself.  Spread is for launches that leave each
//  workgroup its CU, where a point's own waves are all there is to hide
//  latency (launch_lane).  768 threads at three waves per SIMD (168 VGPRs) do not
//  spill, where held to four they may (P = 120, 200 points: 95 us against 79;
//  P = 100: 74 us with 1,024 threads against 66).
//  P = 80 had factors 5 16 (x) and 5 16 (y), 256 threads at 49 spilled VGPRs to a
//  full workgroup: alone on a CU one took 106 us, so that 272 points were slower
//  than with the group layout (76 us; now 60).
#define CFOG_PLANS(G, L)                                         \
  G(16, 4, 4, 64)                                                \
  G(24, 6, 4, 128)                                               \
  G(32, 8, 4, 256)                                               \
  G(40, 8, 5, 256)                                               \
  G(48, 8, 6, 256)                                               \
  L((60, 6, 10, 15, 4, 10, 6), (192, 1, 4, 1), (512, 1, 4, 1))       \
  L((64, 8, 8, 8, 8, 8, 8), (256, 1, 4, 0), (512, 1, 4, 1))          \
  L((72, 6, 12, 9, 8, 9, 8), (256, 1, 4, 1), (512, 1, 4, 1))         \
  L((80, 10, 8, 10, 8, 10, 8), (512, 1, 2, 1), (768, 1, 3, 1))       \
  L((90, 9, 10, 9, 10, 10, 9), (512, 1, 4, 0), (768, 1, 4, 1))       \
  L((96, 8, 12, 12, 8, 12, 8), (512, 1, 4, 1), (768, 1, 3, 1))       \
  L((100, 10, 10, 5, 20, 10, 10), (512, 1, 4, 1), (768, 2, 3, 1))    \
  L((108, 9, 12, 9, 12, 12, 9), (512, 1, 4, 1), (1024, 1, 4, 0))     \
  L((120, 8, 15, 15, 8, 12, 10), (512, 1, 4, 0), (768, 1, 3, 0))     \
  L((144, 12, 12, 12, 12, 12, 12), (1024, 1, 4, 0), (1024, 1, 4, 0)) \
  L((160, 10, 16, 20, 8, 16, 10), (896, 0, 4, 0), (896, 0, 4, 0))    \
  L((192, 24, 8, 24, 8, 16, 12), (512, 0, 2, 1), (512, 0, 2, 1))

#define CFOG_ARGS(...) __VA_ARGS__
#define CFOG_LANE_CFG(PLAN, TEAM) LaneCfg<CFOG_ARGS PLAN, CFOG_ARGS TEAM>

template <class C>
static int launch_group(const MatchJob& job0, const MatchJob* jobs, const int2* tasks, int n_tasks, int n_blocks,
                        const SplitArgs& sp, bool, hipStream_t st) {
  hipLaunchKernelGGL(match_fft_kernel<C>, dim3(n_blocks), dim3(C::NT), C::LDS, st, job0, jobs, tasks, n_tasks, sp);
  return hipGetLastError() == hipSuccess ? 0 : -2;
}

// Workgroups of W that a CU holds (its registers allow W::WPE waves to a SIMD).
template <class W>
constexpr int resident() {
  return std::max(1, std::min((int)(kMaxLds / W::LDS), 4 * W::WPE / W::NW));
}

// Full or spread workgroups (takes_spread in split_plan.hpp).
template <class C, class W, bool WIDE>
static int launch_lane(const MatchJob& job0, const MatchJob* jobs, const int2* tasks, int n_tasks, int n_blocks,
                       const SplitArgs& sp, bool spread, hipStream_t st) {
  if (spread)
    hipLaunchKernelGGL((match_lane_kernel<W, WIDE>), dim3(n_blocks), dim3(W::NT), W::LDS, st, job0, jobs, tasks, n_tasks, sp);
  else
    hipLaunchKernelGGL((match_lane_kernel<C, WIDE>), dim3(n_blocks), dim3(C::NT), C::LDS, st, job0, jobs, tasks, n_tasks, sp);
  return hipGetLastError() == hipSuccess ? 0 : -2;
}

template <class C>
static constexpr FftPlan group_plan() {
  return FftPlan{C::P, C::R1, C::R2, C::NT, C::LDS, C::P, false, 0, false, launch_group<C>};
}
// WIDE: for images wider than kLaneMaxWidth.
template <class C, class W, bool WIDE>
static constexpr FftPlan lane_plan() {
  return FftPlan{C::P, C::R1, C::R2, C::NT, C::LDS, C::P == 144 ? 134 : C::P, true, resident<W>(), 2 * C::NT >= W::NT,
                 launch_lane<C, W, WIDE>};
}

#define CFOG_NO_PLAN(...)
static const FftPlan kPlans[] = {
#define CFOG_PLAN_ENTRY(...) group_plan<FftCfg<__VA_ARGS__>>(),
#define CFOG_LANE_ENTRY(PLAN, FULL, SPREAD) lane_plan<CFOG_LANE_CFG(PLAN, FULL), CFOG_LANE_CFG(PLAN, SPREAD), false>(),
#define CFOG_WIDE_ENTRY(PLAN, FULL, SPREAD) lane_plan<CFOG_LANE_CFG(PLAN, FULL), CFOG_LANE_CFG(PLAN, SPREAD), true>(),
    CFOG_PLANS(CFOG_PLAN_ENTRY, CFOG_LANE_ENTRY)
    CFOG_PLANS(CFOG_NO_PLAN, CFOG_WIDE_ENTRY)
#undef CFOG_PLAN_ENTRY
#undef CFOG_LANE_ENTRY
#undef CFOG_WIDE_ENTRY
};
#define CFOG_COUNT(...) + 1
constexpr int kNumPlans = CFOG_PLANS(CFOG_COUNT, CFOG_COUNT);  // those that are chosen by size, which come first
constexpr int kNumLane = CFOG_PLANS(CFOG_NO_PLAN, CFOG_COUNT);
#undef CFOG_COUNT
static_assert(sizeof(kPlans) / sizeof(kPlans[0]) == kNumPlans + kNumLane, "plans");

const FftPlan* wide_plan(const FftPlan* p) { return p->lane ? p + kNumLane : p; }

const FftPlan* fft_plans(int* count, bool with_wide) {
  *count = with_wide ? kNumPlans + kNumLane : kNumPlans;
  return kPlans;
}

bool plan_fits(const FftPlan* p, int N, int r) {
  if (N < 1 || r < 0 || N > kMaxSide || r > kMaxSide) return false;
  return p->P >= N + 2 * r && N <= p->t_rows && offsets_fit(p->P, 2 * r + 1);
}

const FftPlan* choose_fft_plan(int N, int r) {
  for (int i = 0; i < kNumPlans; ++i)
    if (plan_fits(&kPlans[i], N, r)) return &kPlans[i];
  return nullptr;
}

// Workgroups of each plan resident per CU, from the runtime's occupancy
// calculator (registers, LDS and waves); filled by init_match_fft_attributes.
static int g_plan_occupancy[64];

int plan_slots(const FftPlan* p, int num_cus) {
  const int i = (int)(p - kPlans);
  int per_cu = (i >= 0 && i < 64) ? g_plan_occupancy[i] : 0;
  if (per_cu <= 0) per_cu = std::max(1, std::min((int)(kMaxLds / p->lds), 32 / (p->NT / 64)));
  return num_cus * per_cu;
}

// Slots the channel split of a launch's last round is planned for.  Lane
// layout: two workgroups to a CU up to P = 72 and one above, the group
// layout's numbers, and not as many as fit, so that the same points are split
// into the same groups and their partial sums keep their roundings (see
// lane_inverse); the launches still fill every slot.
int plan_split_slots(const FftPlan* p, int num_cus) {
  return p->lane ? num_cus * (p->P <= 72 ? 2 : 1) : plan_slots(p, num_cus);
}

// One workgroup per split task: the sum of its G partial surfaces (in item
// order) into LDS, eight of an offset's partials in flight at a time, then the
// epilogue of the whole sum.  Bound by the latency of those reads, and past 256
// tasks by the rounds of workgroups: 52 SGPRs let two share a CU.  Summing as
// the epilogue goes took 106 (one to a CU), and with sub-pixel output read the
// neighbours' partials again: N = 16, r = 3, 272 points in both launches 22.2 us,
// with sub-pixel output 25.1; 20.3 and 21.1 so.
constexpr int SR_NT = 1024;
constexpr int SR_NG = 8;
__global__ __launch_bounds__(SR_NT) void split_reduce_kernel(
    MatchJob job0, const MatchJob* __restrict__ jobs, const int2* __restrict__ tasks, SplitArgs sp) {
  extern __shared__ float4 sr_lds[];
  ArgminState* red = reinterpret_cast<ArgminState*>(sr_lds);
  float* Cs = reinterpret_cast<float*>(red + SR_NT / 64);
  const int t = sp.n_whole + blockIdx.x;
  MatchJob jd = job0;
  int cpi = t;
  if (jobs) {
    const int2 tk = tasks[t];
    jd = jobs[tk.x];
    cpi = tk.y;
  }
  const int4 cp = jd.cps[cpi];
  const CpBoxes bx = cp_boxes(cp.x, cp.y, cp.z, cp.w, jd.N, jd.r, jd.hA, jd.wA, jd.hB, jd.wB);
  if (!bx.inside) return;  // reported by the task's first item
  const float* p = sp.part + (size_t)blockIdx.x * sp.G * sp.slot;
  const int KK = (2 * jd.r + 1) * (2 * jd.r + 1);
  for (int i = threadIdx.x; i < KK; i += SR_NT) {
    unsigned o = i;
    float s = ldg(p + o);
    for (int g = 1; g < sp.G; g += SR_NG) {
      float v[SR_NG];
#pragma unroll
      for (int u = 0; u < SR_NG; ++u) {
        if (g + u >= sp.G) break;
        o += sp.slot;
        v[u] = ldg(p + o);
      }
#pragma unroll
      for (int u = 0; u < SR_NG; ++u) {
        if (g + u >= sp.G) break;
        s += v[u];
      }
    }
    Cs[i] = s;
  }
  __syncthreads();
  ssd_epilogue<SR_NT, 1>(jd, cpi, bx.tx0, bx.ty0, bx.sx0, bx.sy0, Cs, red);
}

int launch_split_reduce(const MatchJob& job0, const MatchJob* d_jobs, const int2* d_tasks, int n_tasks,
                        const SplitArgs& sp, hipStream_t st) {
  if (sp.G <= 1 || n_tasks <= sp.n_whole) return 0;
  const size_t lds = sizeof(ArgminState) * (SR_NT / 64) + sizeof(float) * (size_t)sp.slot;
  if (lds > 64 * 1024) return -1;
  hipLaunchKernelGGL(split_reduce_kernel, dim3(n_tasks - sp.n_whole), dim3(SR_NT), lds, st, job0, d_jobs, d_tasks,
                     sp);
  return hipGetLastError() == hipSuccess ? 0 : -2;
}

int init_match_fft_attributes() {
  int idx = 0;
  auto allow = [&](auto* kernel, size_t lds) {
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
  };
  auto set = [&](auto* kernel, int nt, size_t lds) {
    if (!allow(kernel, lds)) return false;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, nt, lds) != hipSuccess) n = 0;
    g_plan_occupancy[idx++] = n;
    return true;
  };
#define CFOG_PLAN_ATTR(...) \
  if (!set(match_fft_kernel<FftCfg<__VA_ARGS__>>, FftCfg<__VA_ARGS__>::NT, FftCfg<__VA_ARGS__>::LDS)) return -2;
#define CFOG_LANE_ATTR_OF(PLAN, FULL, SPREAD, WIDE)                                                              \
  {                                                                                                              \
    using C = CFOG_LANE_CFG(PLAN, FULL);                                                                         \
    using W = CFOG_LANE_CFG(PLAN, SPREAD);                                                                       \
    if (!set(match_lane_kernel<C, WIDE>, C::NT, C::LDS) || !allow(match_lane_kernel<W, WIDE>, W::LDS)) return -2; \
  }
#define CFOG_LANE_ATTR(PLAN, FULL, SPREAD) CFOG_LANE_ATTR_OF(PLAN, FULL, SPREAD, false)
#define CFOG_WIDE_ATTR(PLAN, FULL, SPREAD) CFOG_LANE_ATTR_OF(PLAN, FULL, SPREAD, true)
  CFOG_PLANS(CFOG_PLAN_ATTR, CFOG_LANE_ATTR)
  CFOG_PLANS(CFOG_NO_PLAN, CFOG_WIDE_ATTR)
#undef CFOG_PLAN_ATTR
#undef CFOG_LANE_ATTR_OF
#undef CFOG_LANE_ATTR
#undef CFOG_WIDE_ATTR
  return 0;
}

int init_kernel_attributes() {
  static std::mutex mu;
  static std::vector<int> done;  // devices already set up
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -2;
  std::lock_guard<std::mutex> lock(mu);
  if (std::find(done.begin(), done.end(), dev) != done.end()) return 0;
  int rc = init_match_fft_attributes();
  if (rc == 0) rc = init_extract_attributes();
  if (rc == 0) rc = init_direct_attributes();
  if (rc == 0) rc = init_outlier_attributes();
  if (rc == 0) done.push_back(dev);
  return rc;
}

int launch_match_fft(const FftPlan* plan, const MatchJob& job0, const MatchJob* d_jobs, const int2* d_tasks,
                     int n_tasks, int n_blocks, const SplitArgs& sp, bool spread, hipStream_t st) {
  if (n_tasks <= 0) return 0;
  return plan->launch(job0, d_jobs, d_tasks, n_tasks, n_blocks, sp, spread, st);
}

}  // namespace cfog
