// Block-based Harris feature points (Section IV of Ye et al.): the reference
// image is divided into n x n cells; the chip (up to 64 x 64 pixels) centred
// on each cell is read and its k pixels with the largest Harris response
// become feature points, which are the control points the matcher takes.
//
// One workgroup per chip, its arrays in LDS (three chips per CU); the Gaussian
// radius is a template parameter (unrolled taps):
//   1. the chip (clipped to the image);
//   2. gradients by [-1, 0, 1] with the chip's borders replicated;
//   3. the structure tensor products gx^2, gx gy, gy^2 (formed on the fly)
//      smoothed by a normalised Gaussian (horizontal then vertical pass,
//      chip borders replicated) and the response R = det - kappa trace^2;
//   4. each wave's k largest responses (ties to the smallest row-major index),
//      and of these 4 k candidates the first k.
//
// What bounds it: LDS traffic and the vector units, about evenly; the image
// itself is read once.  So a thread takes four adjacent columns through the
// gradients and the horizontal pass (16-byte LDS accesses, the products of
// 4 + 2 R positions formed once for four sums) and 16 rows of a column through
// the vertical pass (16 + 2 R reads instead of 16 (2 R + 1)), and the responses
// stay in its registers: a round of the maximum is a wave's reduction without a
// barrier, and the candidates are ranked all at once.
//   64 x 64 chips of a 4096 x 4096 image, 4 points each, sigma 1: 175 us
//   with a thread per pixel in every pass and k workgroup reductions over the
//   responses in LDS, 80 us so.
#include <hip/hip_runtime.h>
#include <math.h>
#include <limits.h>
#include <algorithm>
#include "cfog.h"
#include "kernels.hpp"

namespace cfog {

constexpr int HR_NT = 256;
constexpr int HR_MAX_CHIP = 64;
constexpr int HR_MAX_K = 64;

struct HarrisArgs {
  const float* img;
  int64_t stride;
  int H, W, n, k, chip;
  float kappa;
  float w[kMaxGaussRadius + 1];  // w[|j|], j in [-R, R]
  cfog_cp* cps;
  float* resp;
};

constexpr int HR_NW = HR_NT / 64;
constexpr int HR_RPT = HR_MAX_CHIP / HR_NW;       // rows of a thread's column in the vertical pass
constexpr int HR_LDC = HR_MAX_CHIP;               // LDS row stride of the chip, later of sum gy^2
constexpr int HR_QR = HR_NT / (HR_MAX_CHIP / 4);  // rows that the workgroup covers with a quad of columns per thread

// Gradients (then sum gx^2 and sum gx gy) have the Gaussian's replicated
// columns on both sides: PAD, a multiple of 4.
template <int R>
struct HarrisLds {
  static constexpr int PAD = (R + 3) / 4 * 4;
  static constexpr int LD = HR_MAX_CHIP + 2 * PAD;
};
template <int R>
static size_t harris_lds_bytes(int chip) {
  // the candidates (HR_NW k values and indices) reuse the arrays
  return std::max((size_t)(2 * HarrisLds<R>::LD + HR_LDC) * chip, (size_t)HR_NW * HR_MAX_K * 2) * sizeof(float);
}

// The largest value of the wave, in every lane.
__device__ __forceinline__ float wave_max(float v) {
#define HR_DPP_MAX(ctrl, rows)                                                                                     \
  v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v),                   \
                                                                     __builtin_bit_cast(int, v), ctrl, rows, 0xf, false)))
  HR_DPP_MAX(0x111, 0xf);  // row_shr:1
  HR_DPP_MAX(0x112, 0xf);
  HR_DPP_MAX(0x114, 0xf);
  HR_DPP_MAX(0x118, 0xf);
  HR_DPP_MAX(0x142, 0xa);  // row_bcast:15
  HR_DPP_MAX(0x143, 0xc);  // row_bcast:31
#undef HR_DPP_MAX
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

template <int R>
__global__ __launch_bounds__(HR_NT) void harris_grid_kernel(HarrisArgs a) {
  extern __shared__ __attribute__((aligned(16))) float hsm[];
  constexpr int PAD = HarrisLds<R>::PAD, LD = HarrisLds<R>::LD, QN = 4 + 2 * PAD;
  float* gx = hsm + PAD;  // later sum gx^2
  float* gy = gx + LD * a.chip;  // later sum gx gy
  float* img = hsm + 2 * LD * a.chip;  // later sum gy^2
  const int cell = blockIdx.x, ci = cell / a.n, cj = cell - ci * a.n;
  // chip of cell (ci, cj): centred at ((2 cj + 1) W / 2n, (2 ci + 1) H / 2n), clipped
  const int cy = (int)(((int64_t)(2 * ci + 1) * a.H) / (2 * a.n));
  const int cx = (int)(((int64_t)(2 * cj + 1) * a.W) / (2 * a.n));
  const int y0 = max(0, cy - a.chip / 2), x0 = max(0, cx - a.chip / 2);
  const int h = min(a.H, cy - a.chip / 2 + a.chip) - y0, w = min(a.W, cx - a.chip / 2 + a.chip) - x0;
  const int x = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const bool col = x < w;
  float wt[R + 1];
#pragma unroll
  for (int j = 0; j <= R; ++j) wt[j] = a.w[j];

  {
    // all loads of the chip issued before the first LDS store
    float v[HR_RPT];
    const float* src = a.img + (int64_t)y0 * a.stride + x0 + x;
#pragma unroll
    for (int t = 0; t < HR_RPT; ++t) {
      const int y = wv + HR_NW * t;
      if (col && y < h) v[t] = src[(int64_t)y * a.stride];
    }
#pragma unroll
    for (int t = 0; t < HR_RPT; ++t) {
      const int y = wv + HR_NW * t;
      if (col && y < h) img[y * HR_LDC + x] = v[t];
    }
  }
  __syncthreads();
  // gradients: columns x4 .. x4 + 3 of the rows yq + HR_QR t; a row is one
  // wave's (the sixteen lanes of its quads) until the vertical pass
  const int x4 = (threadIdx.x & 15) * 4, yq = threadIdx.x >> 4;
  const int xl = max(x4 - 1, 0), xr = min(x4 + 4, w - 1);
  const bool last = x4 <= w - 1 && w - 1 < x4 + 4;  // the quad of the chip's last column
#pragma unroll
  for (int t = 0; t < HR_MAX_CHIP / HR_QR; ++t) {
    const int y = yq + HR_QR * t;
    if (x4 < w && y < h) {
      const float* row = img + y * HR_LDC;
      const float4 c4 = *reinterpret_cast<const float4*>(row + x4);
      const float4 d4 = *reinterpret_cast<const float4*>(img + min(y + 1, h - 1) * HR_LDC + x4);
      const float4 u4 = *reinterpret_cast<const float4*>(img + max(y - 1, 0) * HR_LDC + x4);
      const float c[6] = {row[xl], c4.x, c4.y, c4.z, c4.w, row[xr]};
      float g[4], e[4] = {d4.x - u4.x, d4.y - u4.y, d4.z - u4.z, d4.w - u4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) g[i] = (x4 + i < w - 1 ? c[i + 2] : c[i + 1]) - c[i];
      float* px = gx + y * LD + x4;
      float* py = gy + y * LD + x4;
      if (PAD > 0 && last) {  // the last column again, to the quad's end and past it
#pragma unroll
        for (int i = 1; i < 4; ++i)
          if (x4 + i > w - 1) {
            g[i] = g[i - 1];
            e[i] = e[i - 1];
          }
#pragma unroll
        for (int p = 4; p < 4 + PAD; p += 4) {
          *reinterpret_cast<float4*>(px + p) = make_float4(g[3], g[3], g[3], g[3]);
          *reinterpret_cast<float4*>(py + p) = make_float4(e[3], e[3], e[3], e[3]);
        }
      }
      if (PAD > 0 && x4 == 0) {
#pragma unroll
        for (int p = 4; p <= PAD; p += 4) {
          *reinterpret_cast<float4*>(px - p) = make_float4(g[0], g[0], g[0], g[0]);
          *reinterpret_cast<float4*>(py - p) = make_float4(e[0], e[0], e[0], e[0]);
        }
      }
      *reinterpret_cast<float4*>(px) = make_float4(g[0], g[1], g[2], g[3]);
      *reinterpret_cast<float4*>(py) = make_float4(e[0], e[1], e[2], e[3]);
    }
  }
  __syncthreads();
  // horizontal pass of the three products, in place
#pragma unroll
  for (int t = 0; t < HR_MAX_CHIP / HR_QR; ++t) {
    const int y = yq + HR_QR * t;
    const bool in = x4 < w && y < h;
    float4 sa, sb, sc;
    if (in) {
      float uu[QN], uv[QN], vv[QN];
#pragma unroll
      for (int q = 0; q < QN; q += 4) {
        const float4 u = *reinterpret_cast<const float4*>(gx + y * LD + x4 - PAD + q);
        const float4 v = *reinterpret_cast<const float4*>(gy + y * LD + x4 - PAD + q);
        const float us[4] = {u.x, u.y, u.z, u.w}, vs[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uu[q + i] = us[i] * us[i];
          uv[q + i] = us[i] * vs[i];
          vv[q + i] = vs[i] * vs[i];
        }
      }
      auto taps = [&](const float (&p)[QN]) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = -R; j <= R; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[i] = fmaf(wt[j < 0 ? -j : j], p[PAD + i + j], s[i]);
        return make_float4(s[0], s[1], s[2], s[3]);
      };
      sa = taps(uu);
      sb = taps(uv);
      sc = taps(vv);
    }
    // the row's sixteen lanes have read it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (in) {
      *reinterpret_cast<float4*>(gx + y * LD + x4) = sa;
      *reinterpret_cast<float4*>(gy + y * LD + x4) = sb;
      *reinterpret_cast<float4*>(img + y * HR_LDC + x4) = sc;
    }
  }
  __syncthreads();
  // vertical pass (rows clamped to the chip) and the response, of column x and
  // the rows yv .. yv + HR_RPT - 1; what is outside the chip is NaN
  const int yv = wv * HR_RPT;
  float rv[HR_RPT];
  {
    const int xc = min(x, w - 1);
    auto taps = [&](const float* p, int ld, float (&s)[HR_RPT]) {
      float win[HR_RPT + 2 * R];
#pragma unroll
      for (int t = 0; t < HR_RPT + 2 * R; ++t) win[t] = p[min(max(yv + t - R, 0), h - 1) * ld + xc];
#pragma unroll
      for (int t = 0; t < HR_RPT; ++t) {
        s[t] = 0.f;
#pragma unroll
        for (int j = -R; j <= R; ++j) s[t] = fmaf(wt[j < 0 ? -j : j], win[t + j + R], s[t]);
      }
    };
    float sa[HR_RPT], sb[HR_RPT], sc[HR_RPT];
    taps(gx, LD, sa);
    taps(gy, LD, sb);
    taps(img, HR_LDC, sc);
#pragma unroll
    for (int t = 0; t < HR_RPT; ++t) {
      const float tr = sa[t] + sc[t];
      const float r = sa[t] * sc[t] - sb[t] * sb[t] - a.kappa * tr * tr;
      rv[t] = col && yv + t < h ? r : NAN;
    }
  }
  __syncthreads();  // the arrays are dead: the candidates reuse them

  // this wave's k largest in order, as (value, row-major index); INT_MAX: none
  // left.  A taken response becomes NaN, which never wins.
  float* cv = hsm;
  int* cidx = reinterpret_cast<int*>(hsm + HR_NW * a.k);
  float bv;
  int bt;
  auto scan = [&] {
    bv = -INFINITY;
    bt = HR_RPT;
#pragma unroll
    for (int t = 0; t < HR_RPT; ++t)
      if (rv[t] > bv) {
        bv = rv[t];
        bt = t;
      }
  };
  scan();
  for (int q = 0; q < a.k; ++q) {
    const float mx = wave_max(bv);
    int bi = bt < HR_RPT && bv == mx ? (yv + bt) * w + x : INT_MAX;
    const int mine = bi;
    const uint64_t tied = __ballot(bi != INT_MAX);
    if (tied & (tied - 1)) {  // several columns hold it: the smallest index
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) bi = min(bi, __shfl_xor(bi, o, 64));
    } else if (tied) {
      bi = __builtin_amdgcn_readlane(bi, __builtin_ctzll(tied));
    }
    if (mine == bi && bi != INT_MAX) {
      cv[wv * a.k + q] = bv;
      cidx[wv * a.k + q] = bi;
      if (q + 1 < a.k) {
#pragma unroll
        for (int t = 0; t < HR_RPT; ++t)
          if (t == bt) rv[t] = NAN;
        scan();
      }
    }
    if (!tied) {
      if (x == 0) cidx[wv * a.k + q] = INT_MAX;
    }
  }
  __syncthreads();
  // the place of each candidate among all
  const int nc = HR_NW * a.k;
  if ((int)threadIdx.x < nc) {
    const int i = threadIdx.x, bi = cidx[i];
    const float v = cv[i];
    int before = 0, valid = 0;
    for (int u = 0; u < nc; ++u) {
      const int oi = cidx[u];
      const float ov = cv[u];
      valid += oi != INT_MAX;
      before += oi != INT_MAX && (ov > v || (ov == v && oi < bi));
    }
    if (bi != INT_MAX && before < a.k) {
      const int o = cell * a.k + before, yy = bi / w, xx = bi - yy * w;
      a.cps[o] = cfog_cp{x0 + xx, y0 + yy, x0 + xx, y0 + yy};
      if (a.resp) a.resp[o] = v;
    }
    if (i < a.k && i >= valid) {  // no finite response left (a non-finite chip)
      const int o = cell * a.k + i;
      a.cps[o] = cfog_cp{-1, -1, -1, -1};
      if (a.resp) a.resp[o] = NAN;
    }
  }
}

template <int R>
static int launch_harris(const HarrisArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(harris_grid_kernel<R>, dim3(a.n * a.n), dim3(HR_NT), harris_lds_bytes<R>(a.chip), st, a);
  return hipGetLastError() == hipSuccess ? 0 : -2;
}

}  // namespace cfog

extern "C" int cfog_harris_grid(cfog_ctx* ctx, const float* d_img, int32_t H, int32_t W, int64_t row_stride,
                                int32_t n, int32_t k, int32_t chip, float sigma, float kappa, cfog_cp* d_cps,
                                float* d_response, void* stream) {
  if (!ctx || !d_img || !d_cps || H < 1 || W < 1 || row_stride < W || n < 1 || k < 1 ||
      k > cfog::HR_MAX_K || chip < 1 || chip > cfog::HR_MAX_CHIP || !(sigma > 0.f) || !isfinite(sigma) ||
      !isfinite(kappa) || ((uintptr_t)d_cps % 16) != 0 || ((uintptr_t)d_response % 4) != 0)
    return CFOG_EINVAL;
  if ((int64_t)n * n > INT_MAX / k) return CFOG_EINVAL;
  const int R = (int)(4.0 * sigma + 0.5);
  if (R > cfog::kMaxGaussRadius) return CFOG_EUNSUPPORTED;
  // every chip must hold at least k pixels
  for (int i = 0; i < n; ++i) {
    const int cy = (int)(((int64_t)(2 * i + 1) * H) / (2 * n));
    const int h = std::min(H, cy - chip / 2 + chip) - std::max(0, cy - chip / 2);
    for (int j = 0; j < n; ++j) {
      const int cx = (int)(((int64_t)(2 * j + 1) * W) / (2 * n));
      const int w = std::min(W, cx - chip / 2 + chip) - std::max(0, cx - chip / 2);
      if (h < 1 || w < 1 || h * w < k) return CFOG_EINVAL;
    }
  }
  cfog::HarrisArgs a{};
  a.img = d_img;
  a.stride = row_stride;
  a.H = H;
  a.W = W;
  a.n = n;
  a.k = k;
  a.chip = chip;
  a.kappa = kappa;
  double ws[cfog::kMaxGaussRadius + 1], tot = 0.0;
  for (int j = 0; j <= R; ++j) {
    ws[j] = exp(-(double)j * j / (2.0 * (double)sigma * sigma));
    tot += (j ? 2.0 : 1.0) * ws[j];
  }
  for (int j = 0; j <= R; ++j) a.w[j] = (float)(ws[j] / tot);
  a.cps = d_cps;
  a.resp = d_response;
  hipStream_t st = (hipStream_t)stream;
  int rc = -2;
  switch (R) {
    case 0: rc = cfog::launch_harris<0>(a, st); break;
    case 1: rc = cfog::launch_harris<1>(a, st); break;
    case 2: rc = cfog::launch_harris<2>(a, st); break;
    case 3: rc = cfog::launch_harris<3>(a, st); break;
    case 4: rc = cfog::launch_harris<4>(a, st); break;
    case 5: rc = cfog::launch_harris<5>(a, st); break;
    case 6: rc = cfog::launch_harris<6>(a, st); break;
    case 7: rc = cfog::launch_harris<7>(a, st); break;
    case 8: rc = cfog::launch_harris<8>(a, st); break;
    default: return CFOG_EUNSUPPORTED;
  }
  return rc == 0 ? CFOG_OK : CFOG_EHIP;
}
