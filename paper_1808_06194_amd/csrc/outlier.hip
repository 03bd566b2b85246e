// Iterative outlier rejection of control points with a cubic polynomial
// mapping model (Section IV of Ye et al.): fit the model to all kept points by
// least squares, remove the point with the largest residual, and repeat until
// the RMSE falls below a threshold (or ten points, the model's size, remain).
//
// One workgroup per point set.  In FP64:
//   1. once, the 55 + 20 entries of the normal equations (ten monomials of
//      the normalised source coordinates; both target coordinates) summed
//      over all points (per-thread partials, wave shuffles, LDS);
//   per iteration:
//   2. a Cholesky solve of the 10 x 10 system for both right-hand sides;
//   3. residuals |model(p) - q| of the kept points, their squared sum and the
//      largest one (ties to the smaller index);
//   4. removal of that point, whose products are subtracted from the normal
//      equations (a rank-one downdate, so the sums need not be formed again).
//
// An iteration is a serial chain, so what counts is its length.  Sets of up to
// 4096 points (reject_small_kernel) are held in registers, and every wave
// solves the system by itself, a row to a lane, so that an iteration has one
// barrier.  Larger ones (reject_kernel) are held in LDS up to 8192 points and
// read from global memory above; one thread solves and downdates the system
// for all.  Both do the same operations in the same order: 1500 points, 60 of
// them gross errors, take 168 us in the one, 464 us in the other (an iteration
// of the one: 2.6 us, and 0.3 us per 1000 points).
#include <hip/hip_runtime.h>
#include <math.h>
#include <limits.h>
#include "cfog.h"
#include "root.hpp"

namespace cfog {

constexpr int RJ_NT = 512;
constexpr int RJ_NW = RJ_NT / 64;
constexpr int RJ_T = 10;                   // monomials of a bivariate cubic
constexpr int RJ_G = RJ_T * (RJ_T + 1) / 2;  // unique entries of the normal matrix
constexpr int RJ_V = RJ_G + 2 * RJ_T;      // plus the two right-hand sides
constexpr int RJ_LDS_POINTS = 8192;        // sets up to this size live in LDS

// Dynamic LDS of a set of n points: both coordinate arrays and the flags.
static size_t reject_lds_bytes(int n) {
  return n <= RJ_LDS_POINTS ? (size_t)n * (2 * sizeof(float2) + 1) : 0;
}

__device__ __forceinline__ void cubic_terms(double u, double v, double (&t)[RJ_T]) {
  t[0] = 1.0;
  t[1] = u;
  t[2] = v;
  t[3] = u * u;
  t[4] = u * v;
  t[5] = v * v;
  t[6] = u * u * u;
  t[7] = u * u * v;
  t[8] = u * v * v;
  t[9] = v * v * v;
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// RES: the set lives in LDS (n <= RJ_LDS_POINTS).  A compile-time choice, so
// that every point access has a known address space (LDS or global) instead
// of going through flat instructions.
template <bool RES>
__global__ __launch_bounds__(RJ_NT) void reject_kernel(const float2* __restrict__ src, const float2* __restrict__ dst,
                                                       int n, float thr, unsigned char* keep, cfog_reject_result* out) {
  extern __shared__ float2 rj_pts[];
  __shared__ double part[RJ_NW][RJ_V];
  __shared__ double sys[RJ_V];
  __shared__ double coef[RJ_T][2];
  __shared__ double rd[RJ_NW];
  __shared__ int ri[RJ_NW];
  __shared__ double ext[4];
  __shared__ int done, active, removed;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float2* ps = RES ? rj_pts : src;
  const float2* pd = RES ? rj_pts + n : dst;
  unsigned char* pk = RES ? reinterpret_cast<unsigned char*>(rj_pts + 2 * n) : keep;

  // points into LDS (resident sets); bounding box -> centre and half-extent per axis
  {
    double mn[2] = {INFINITY, INFINITY}, mx[2] = {-INFINITY, -INFINITY};
    for (int i = tid; i < n; i += RJ_NT) {
      const float2 p = src[i];
      if (RES) {
        rj_pts[i] = p;
        rj_pts[n + i] = dst[i];
      }
      mn[0] = fmin(mn[0], (double)p.x);
      mn[1] = fmin(mn[1], (double)p.y);
      mx[0] = fmax(mx[0], (double)p.x);
      mx[1] = fmax(mx[1], (double)p.y);
      pk[i] = 1;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      mn[0] = fmin(mn[0], __shfl_xor(mn[0], o, 64));
      mn[1] = fmin(mn[1], __shfl_xor(mn[1], o, 64));
      mx[0] = fmax(mx[0], __shfl_xor(mx[0], o, 64));
      mx[1] = fmax(mx[1], __shfl_xor(mx[1], o, 64));
    }
    if (lane == 0) {
      part[wv][0] = mn[0];
      part[wv][1] = mn[1];
      part[wv][2] = mx[0];
      part[wv][3] = mx[1];
    }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < RJ_NW; ++w) {
        mn[0] = fmin(mn[0], part[w][0]);
        mn[1] = fmin(mn[1], part[w][1]);
        mx[0] = fmax(mx[0], part[w][2]);
        mx[1] = fmax(mx[1], part[w][3]);
      }
      for (int a = 0; a < 2; ++a) {
        const double half = 0.5 * (mx[a] - mn[a]);
        ext[a] = 0.5 * (mn[a] + mx[a]);
        ext[2 + a] = half > 0.0 ? half : 1.0;
      }
      done = 0;
      active = n;
      removed = 0;
    }
    __syncthreads();
  }
  const double cx = ext[0], cy = ext[1], sx = ext[2], sy = ext[3];

  // 1. normal equations over all points (every point starts kept)
  {
    double acc[RJ_V];
#pragma unroll
    for (int e = 0; e < RJ_V; ++e) acc[e] = 0.0;
    for (int i = tid; i < n; i += RJ_NT) {
      const float2 p = ps[i], q = pd[i];
      double t[RJ_T];
      cubic_terms(((double)p.x - cx) / sx, ((double)p.y - cy) / sy, t);
      int e = 0;
#pragma unroll
      for (int a = 0; a < RJ_T; ++a)
#pragma unroll
        for (int b = a; b < RJ_T; ++b) acc[e++] += t[a] * t[b];
#pragma unroll
      for (int a = 0; a < RJ_T; ++a) {
        acc[RJ_G + 2 * a] += t[a] * (double)q.x;
        acc[RJ_G + 2 * a + 1] += t[a] * (double)q.y;
      }
    }
#pragma unroll
    for (int e = 0; e < RJ_V; ++e) {
      const double v = wave_sum(acc[e]);
      if (lane == 0) part[wv][e] = v;
    }
    __syncthreads();
    if (tid < RJ_V) {
      double v = 0.0;
      for (int w = 0; w < RJ_NW; ++w) v += part[w][tid];
      sys[tid] = v;
    }
    __syncthreads();
  }

  for (;;) {
    // 2. Cholesky solve (one thread: 10 x 10, every index fixed at compile
    // time so that the factor stays in registers)
    if (tid == 0) {
      // entry (a, b), a >= b, of the symmetric matrix held as the packed upper triangle
      auto A = [&](int a, int b) { return sys[b * RJ_T - b * (b - 1) / 2 + (a - b)]; };
      double L[RJ_T][RJ_T];
      bool ok = true;
#pragma unroll
      for (int j = 0; j < RJ_T; ++j) {
        double d = A(j, j);
#pragma unroll
        for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
        ok = ok && d > 0.0;
        const double ljj = sqrt(d > 0.0 ? d : 1.0);
        L[j][j] = ljj;
#pragma unroll
        for (int i = j + 1; i < RJ_T; ++i) {
          double t = A(i, j);
#pragma unroll
          for (int k = 0; k < j; ++k) t -= L[i][k] * L[j][k];
          L[i][j] = t / ljj;
        }
      }
      if (!ok) {
        done = 2;  // singular normal matrix (degenerate point layout)
      } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          double y[RJ_T], x[RJ_T];
#pragma unroll
          for (int i = 0; i < RJ_T; ++i) {
            double t = sys[RJ_G + 2 * i + c];
#pragma unroll
            for (int k = 0; k < i; ++k) t -= L[i][k] * y[k];
            y[i] = t / L[i][i];
          }
#pragma unroll
          for (int i = RJ_T - 1; i >= 0; --i) {
            double t = y[i];
#pragma unroll
            for (int k = i + 1; k < RJ_T; ++k) t -= L[k][i] * x[k];
            x[i] = t / L[i][i];
            coef[i][c] = x[i];
          }
        }
      }
    }
    __syncthreads();
    if (done == 2) break;
    // 3. residuals, RMSE, largest residual
    double ss = 0.0, best = -1.0;
    int bi = INT_MAX;
    for (int i = tid; i < n; i += RJ_NT) {
      if (!pk[i]) continue;
      const float2 p = ps[i], q = pd[i];
      double t[RJ_T];
      cubic_terms(((double)p.x - cx) / sx, ((double)p.y - cy) / sy, t);
      double mxv = 0.0, myv = 0.0;
#pragma unroll
      for (int a = 0; a < RJ_T; ++a) {
        mxv += t[a] * coef[a][0];
        myv += t[a] * coef[a][1];
      }
      const double ex = mxv - (double)q.x, ey = myv - (double)q.y;
      const double r2 = ex * ex + ey * ey;
      ss += r2;
      const double rr = sqrt(r2);
      if (rr > best || (rr == best && i < bi)) {
        best = rr;
        bi = i;
      }
    }
    ss = wave_sum(ss);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ob > best || (ob == best && oi < bi)) {
        best = ob;
        bi = oi;
      }
    }
    if (lane == 0) {
      part[wv][0] = ss;
      rd[wv] = best;
      ri[wv] = bi;
    }
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < RJ_NW; ++w) {
        s += part[w][0];
        if (rd[w] > best || (rd[w] == best && ri[w] < bi)) {
          best = rd[w];
          bi = ri[w];
        }
      }
      const double rmse = sqrt(s / active);
      if (bi == INT_MAX || !(rmse == rmse)) {
        done = 2;  // a non-finite residual: no point can be chosen
      } else if (rmse < (double)thr || active <= RJ_T) {
        done = 1;
        out->rmse = rmse;
      } else {
        // 4. remove the point and downdate the normal equations
        pk[bi] = 0;
        --active;
        ++removed;
        const float2 p = ps[bi], q = pd[bi];
        double t[RJ_T];
        cubic_terms(((double)p.x - cx) / sx, ((double)p.y - cy) / sy, t);
        int e = 0;
        for (int a = 0; a < RJ_T; ++a)
          for (int b = a; b < RJ_T; ++b) sys[e++] -= t[a] * t[b];
        for (int a = 0; a < RJ_T; ++a) {
          sys[RJ_G + 2 * a] -= t[a] * (double)q.x;
          sys[RJ_G + 2 * a + 1] -= t[a] * (double)q.y;
        }
      }
    }
    __syncthreads();
    if (done) break;
  }
  if (RES)
    for (int i = tid; i < n; i += RJ_NT) keep[i] = pk[i];
  if (tid == 0) {
    out->status = done == 1 ? 0 : 1;
    out->removed = removed;
    out->n_kept = active;
    if (done != 1) out->rmse = NAN;
    for (int a = 0; a < RJ_T; ++a) {
      out->coef[a][0] = done == 1 ? coef[a][0] : NAN;
      out->coef[a][1] = done == 1 ? coef[a][1] : NAN;
    }
    out->centre[0] = cx;
    out->centre[1] = cy;
    out->half_extent[0] = sx;
    out->half_extent[1] = sy;
  }
}

// ------------------------------------------------------------ small sets

constexpr int RS_NT = 256;                  // a wave to a SIMD
constexpr int RS_NW = RS_NT / 64;
constexpr int RS_PAIRS = 8;                 // points of a thread, in pairs
constexpr int RS_POINTS = 2 * RS_PAIRS * RS_NT;
// Of a thread's points tid + RS_NT k, those of even and of odd k are summed
// apart: as if by the threads of a workgroup of RJ_NT, wave by wave.
static_assert(2 * RS_NT == RJ_NT, "the two halves of the sums");

static size_t reject_small_lds_bytes(int n) { return (size_t)n * (sizeof(double2) + sizeof(float2)); }

struct Words {
  uint32_t lo, hi;
};
// a and b with the upper half of a's lanes exchanged for the lower half of
// b's; or, by rows of 16 lanes, the odd rows of a for the even rows of b.
template <int W>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
  Words x = __builtin_bit_cast(Words, a), y = __builtin_bit_cast(Words, b);
  if constexpr (W == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(x.lo, y.lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(x.hi, y.hi, false, false);
    x = Words{l[0], h[0]};
    y = Words{l[1], h[1]};
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(x.lo, y.lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(x.hi, y.hi, false, false);
    x = Words{l[0], h[0]};
    y = Words{l[1], h[1]};
  }
  a = __builtin_bit_cast(double, x);
  b = __builtin_bit_cast(double, y);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const Words x = __builtin_bit_cast(Words, v);
  return __builtin_bit_cast(double, Words{(uint32_t)__builtin_amdgcn_update_dpp(0, (int)x.lo, CTRL, 0xf, 0xf, false),
                                          (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x.hi, CTRL, 0xf, 0xf, false)});
}
// Op over the 16 lanes of each row, in the order of a butterfly of lane
// distances 8, 4, 2, 1 (after distance 8 a row repeats, so a rotation by 4 is
// that exchange).
template <class Op>
__device__ __forceinline__ double row_reduce(double v, Op op) {
  v = op(v, dpp<0x128>(v));  // row_ror:8
  v = op(v, dpp<0x124>(v));  // row_ror:4
  v = op(v, dpp<0x4e>(v));   // quad_perm 2, 3, 0, 1
  return op(v, dpp<0xb1>(v));  // quad_perm 1, 0, 3, 2
}
// Op over the wave, as a butterfly of distances 32, 16, 8, ...
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
  double w = v;
  lane_swap<32>(v, w);
  v = op(v, w);
  w = v;
  lane_swap<16>(v, w);
  return row_reduce(op(v, w), op);
}
// Lane i's value, in every lane.
__device__ __forceinline__ double lane_value(double v, int i) {
  const Words x = __builtin_bit_cast(Words, v);
  return __builtin_bit_cast(double, Words{(uint32_t)__builtin_amdgcn_readlane((int)x.lo, i),
                                          (uint32_t)__builtin_amdgcn_readlane((int)x.hi, i)});
}

__global__ __launch_bounds__(RS_NT, 1) void reject_small_kernel(const float2* __restrict__ src,
                                                                const float2* __restrict__ dst, int n, float thr,
                                                                unsigned char* keep, cfog_reject_result* out) {
  extern __shared__ double2 rs_uv[];  // the normalised source points, then the targets
  float2* rs_q = reinterpret_cast<float2*>(rs_uv + n);
  __shared__ double part[RJ_NW][RJ_V];
  __shared__ double sys[RJ_V];
  __shared__ double rss[2][RJ_NW], rd[2][RS_NW];  // by the parity of the iteration
  __shared__ int ri[2][RS_NW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const auto add = [](double a, double b) { return a + b; };
  const auto least = [](double a, double b) { return fmin(a, b); };
  const auto most = [](double a, double b) { return fmax(a, b); };

  double u[2 * RS_PAIRS], v[2 * RS_PAIRS];
  float2 q[2 * RS_PAIRS];
  uint32_t kept = 0;
  double cx, cy, sx, sy;
  // 0. the points; bounding box -> centre and half-extent per axis
  {
    double mn[2] = {INFINITY, INFINITY}, mx[2] = {-INFINITY, -INFINITY};
    float2 p[2 * RS_PAIRS];
#pragma unroll
    for (int k = 0; k < 2 * RS_PAIRS; ++k) {
      const int i = tid + RS_NT * k;
      u[k] = v[k] = 0.0;
      q[k] = make_float2(0.f, 0.f);
      if (i < n) {
        p[k] = src[i];
        q[k] = dst[i];
        kept |= 1u << k;
      }
    }
#pragma unroll
    for (int k = 0; k < 2 * RS_PAIRS; ++k)
      if (kept >> k & 1) {
        mn[0] = fmin(mn[0], (double)p[k].x);
        mn[1] = fmin(mn[1], (double)p[k].y);
        mx[0] = fmax(mx[0], (double)p[k].x);
        mx[1] = fmax(mx[1], (double)p[k].y);
      }
    for (int a = 0; a < 2; ++a) {
      mn[a] = wave_reduce(mn[a], least);
      mx[a] = wave_reduce(mx[a], most);
      if (lane == 0) {
        part[wv][a] = mn[a];
        part[wv][2 + a] = mx[a];
      }
    }
    __syncthreads();
    double c[2], e[2];
    for (int a = 0; a < 2; ++a) {
      for (int w = 0; w < RS_NW; ++w) {
        mn[a] = fmin(mn[a], part[w][a]);
        mx[a] = fmax(mx[a], part[w][2 + a]);
      }
      const double half = 0.5 * (mx[a] - mn[a]);
      c[a] = 0.5 * (mn[a] + mx[a]);
      e[a] = half > 0.0 ? half : 1.0;
    }
    cx = c[0], cy = c[1], sx = e[0], sy = e[1];
#pragma unroll
    for (int k = 0; k < 2 * RS_PAIRS; ++k)
      if (kept >> k & 1) {
        u[k] = ((double)p[k].x - cx) / sx;
        v[k] = ((double)p[k].y - cy) / sy;
        rs_uv[tid + RS_NT * k] = make_double2(u[k], v[k]);
        rs_q[tid + RS_NT * k] = q[k];
      }
    __syncthreads();
  }

  // 1. normal equations over all points
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    double acc[(RJ_V + 3) / 4 * 4];
#pragma unroll
    for (int e = 0; e < (RJ_V + 3) / 4 * 4; ++e) acc[e] = 0.0;
#pragma unroll 1
    for (int i = tid + half * RS_NT; i < n; i += RJ_NT) {
      const double2 p = rs_uv[i];
      const float2 g = rs_q[i];
      double t[RJ_T];
      cubic_terms(p.x, p.y, t);
      int e = 0;
#pragma unroll
      for (int a = 0; a < RJ_T; ++a)
#pragma unroll
        for (int b = a; b < RJ_T; ++b) acc[e++] += t[a] * t[b];
#pragma unroll
      for (int a = 0; a < RJ_T; ++a) {
        acc[RJ_G + 2 * a] += t[a] * (double)g.x;
        acc[RJ_G + 2 * a + 1] += t[a] * (double)g.y;
      }
    }
    // four entries at a time: the first exchange leaves two to a half of the
    // wave, the second one to a row: entries e, e + 2, e + 1, e + 3
#pragma unroll
    for (int e = 0; e < RJ_V; e += 4) {
      lane_swap<32>(acc[e], acc[e + 1]);
      lane_swap<32>(acc[e + 2], acc[e + 3]);
      double x = acc[e] + acc[e + 1], y = acc[e + 2] + acc[e + 3];
      lane_swap<16>(x, y);
      x = row_reduce(x + y, add);
      const int row = lane >> 4, mine = e + (row >> 1) + 2 * (row & 1);
      if ((lane & 15) == 0 && mine < RJ_V) part[half * RS_NW + wv][mine] = x;
    }
  }
  __syncthreads();
  if (tid < RJ_V) {
    double s = 0.0;
    for (int w = 0; w < RJ_NW; ++w) s += part[w][tid];
    sys[tid] = s;
  }
  __syncthreads();

  // Row `lane` of the normal matrix, in lanes 10 and 11 the right-hand sides.
  double M[RJ_T];
#pragma unroll
  for (int k = 0; k < RJ_T; ++k) {
    const int a = min(lane, k), b = max(lane, k);
    M[k] = lane < RJ_T ? sys[a * RJ_T - a * (a - 1) / 2 + (b - a)] : lane < RJ_T + 2 ? sys[RJ_G + 2 * k + lane - RJ_T] : 0.0;
  }

  int active = n, done = 0;
  double rmse = NAN, coef[RJ_T][2];
  for (int it = 0; !done; ++it) {
    // 2. Cholesky: column by column, the rows below in their lanes.  The
    // right-hand sides are rows of the same elimination, which turns them into
    // the solution of the lower triangle.
    double L[RJ_T], diag[RJ_T], rcp[RJ_T];
#pragma unroll
    for (int k = 0; k < RJ_T; ++k) L[k] = M[k];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < RJ_T; ++j) {
      const double d = lane_value(L[j], j);
      ok = ok && d > 0.0;
      const double p = d > 0.0 ? d : 1.0;
      diag[j] = sqrt_rcp(p, __builtin_amdgcn_rsq(p), rcp[j]);
      L[j] = quotient(L[j], diag[j], rcp[j]);
#pragma unroll
      for (int k = j + 1; k < RJ_T; ++k) L[k] -= L[j] * lane_value(L[j], k);
    }
    if (!ok) {
      done = 2;  // singular normal matrix (degenerate point layout)
      break;
    }
    {
      double x[RJ_T];
#pragma unroll
      for (int i = RJ_T - 1; i >= 0; --i) {
        double t = L[i];
#pragma unroll
        for (int k = i + 1; k < RJ_T; ++k) t -= lane_value(L[i], k) * x[k];
        x[i] = quotient(t, diag[i], rcp[i]);
        coef[i][0] = lane_value(x[i], RJ_T);
        coef[i][1] = lane_value(x[i], RJ_T + 1);
      }
    }
    // 3. residuals, RMSE, largest residual
    double ss[2] = {0.0, 0.0}, r2[2 * RS_PAIRS], best2 = -1.0;
#pragma unroll
    for (int kk = 0; kk < RS_PAIRS; ++kk) {
      r2[2 * kk] = r2[2 * kk + 1] = -1.0;
      if (kk * RJ_NT < n) {
#pragma unroll
        for (int k = 2 * kk; k < 2 * kk + 2; ++k) {
          double t[RJ_T];
          cubic_terms(u[k], v[k], t);
          double mxv = 0.0, myv = 0.0;
#pragma unroll
          for (int a = 0; a < RJ_T; ++a) {
            mxv += t[a] * coef[a][0];
            myv += t[a] * coef[a][1];
          }
          const double ex = mxv - (double)q[k].x, ey = myv - (double)q[k].y;
          const double r = ex * ex + ey * ey;
          if (kept >> k & 1) {
            ss[k & 1] += r;
            r2[k] = r;
            best2 = fmax(best2, r);
          }
        }
      }
    }
    lane_swap<32>(ss[0], ss[1]);
    double s = ss[0] + ss[1], s2 = s;
    lane_swap<16>(s, s2);
    s = row_reduce(s + s2, add);
    best2 = wave_reduce(best2, most);
    // The largest residual is a square root, and the smallest index of those
    // equal to it counts: roots are equal only if their squares are within 2
    // ulp, so the roots are formed only where several are that close.
    const double rbest = best2 >= 0.0 ? sqrt(best2) : -1.0;
    const double close = best2 * (1.0 - 1e-15);
    int near = 0, bi = INT_MAX;
    if (best2 >= 0.0) {
#pragma unroll
      for (int k = 0; k < 2 * RS_PAIRS; ++k)
        if (r2[k] >= close) {
          ++near;
          bi = tid + RS_NT * k;
        }
      const uint64_t lanes = __ballot(near > 0);
      const int first = __builtin_ctzll(lanes);
      if ((lanes & (lanes - 1)) == 0 && __builtin_amdgcn_readlane(near, first) == 1) {
        bi = __builtin_amdgcn_readlane(bi, first);
      } else {
        bi = INT_MAX;
#pragma unroll
        for (int k = 2 * RS_PAIRS - 1; k >= 0; --k)
          if (r2[k] >= close && sqrt(r2[k]) == rbest) bi = tid + RS_NT * k;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) bi = min(bi, __shfl_xor(bi, o, 64));
      }
    }
    const int par = it & 1;
    if ((lane & 31) == 0) rss[par][wv + (lane ? RS_NW : 0)] = s;
    if (lane == 0) {
      rd[par][wv] = rbest;
      ri[par][wv] = bi;
    }
    // The next write of this parity's values comes after the next barrier.
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int w = 0; w < RJ_NW; ++w) s += rss[par][w];
    double best = rd[par][0];
    bi = ri[par][0];
#pragma unroll
    for (int w = 1; w < RS_NW; ++w)
      if (rd[par][w] > best || (rd[par][w] == best && ri[par][w] < bi)) {
        best = rd[par][w];
        bi = ri[par][w];
      }
    bi = __builtin_amdgcn_readfirstlane(bi);
    const double e = sqrt(s / active);
    if (bi == INT_MAX || !(e == e)) {
      done = 2;  // a non-finite residual: no point can be chosen
    } else if (e < (double)thr || active <= RJ_T) {
      done = 1;
      rmse = e;
    } else {
      // 4. remove the point and downdate the normal equations
      --active;
      if ((bi & (RS_NT - 1)) == tid) kept &= ~(1u << (bi / RS_NT));
      const double2 p = rs_uv[bi];
      const float2 g = rs_q[bi];
      double t[RJ_T];
      cubic_terms(p.x, p.y, t);
      double f = lane == RJ_T ? (double)g.x : (double)g.y;
#pragma unroll
      for (int k = 0; k < RJ_T; ++k) f = lane == k ? t[k] : f;
#pragma unroll
      for (int k = 0; k < RJ_T; ++k) M[k] -= f * t[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 2 * RS_PAIRS; ++k)
    if (tid + RS_NT * k < n) keep[tid + RS_NT * k] = kept >> k & 1;
  if (tid == 0) {
    out->status = done == 1 ? 0 : 1;
    out->removed = n - active;
    out->n_kept = active;
    out->rmse = rmse;
#pragma unroll
    for (int a = 0; a < RJ_T; ++a) {
      out->coef[a][0] = done == 1 ? coef[a][0] : NAN;
      out->coef[a][1] = done == 1 ? coef[a][1] : NAN;
    }
    out->centre[0] = cx;
    out->centre[1] = cy;
    out->half_extent[0] = sx;
    out->half_extent[1] = sy;
  }
}

int init_outlier_attributes() {
  return hipFuncSetAttribute((const void*)reject_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)reject_lds_bytes(RJ_LDS_POINTS)) == hipSuccess &&
                 hipFuncSetAttribute((const void*)reject_small_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)reject_small_lds_bytes(RS_POINTS)) == hipSuccess
             ? 0
             : -2;
}

}  // namespace cfog

extern "C" int cfog_reject_outliers(cfog_ctx* ctx, const float* d_src, const float* d_dst, int32_t n, float threshold,
                                    unsigned char* d_keep, cfog_reject_result* d_result, void* stream) {
  if (!ctx || !d_src || !d_dst || !d_keep || !d_result || n < 10 || n > (1 << 20) || !(threshold >= 0.f) ||
      ((uintptr_t)d_src % 8) != 0 || ((uintptr_t)d_dst % 8) != 0 || ((uintptr_t)d_result % 8) != 0)
    return CFOG_EINVAL;
  const float2* src = reinterpret_cast<const float2*>(d_src);
  const float2* dst = reinterpret_cast<const float2*>(d_dst);
  if (n <= cfog::RS_POINTS)
    hipLaunchKernelGGL(cfog::reject_small_kernel, dim3(1), dim3(cfog::RS_NT), cfog::reject_small_lds_bytes(n),
                       (hipStream_t)stream, src, dst, n, threshold, d_keep, d_result);
  else if (n <= cfog::RJ_LDS_POINTS)
    hipLaunchKernelGGL(cfog::reject_kernel<true>, dim3(1), dim3(cfog::RJ_NT), cfog::reject_lds_bytes(n),
                       (hipStream_t)stream, src, dst, n, threshold, d_keep, d_result);
  else
    hipLaunchKernelGGL(cfog::reject_kernel<false>, dim3(1), dim3(cfog::RJ_NT), 0, (hipStream_t)stream, src, dst, n,
                       threshold, d_keep, d_result);
  return hipGetLastError() == hipSuccess ? CFOG_OK : CFOG_EHIP;
}
