// The FFT matcher's second kernel: the correlation of match_fft.hip (the
// notation there), with the 2-D transforms laid out one lane per column or row
// instead of one group of lanes per transform.
//
// A channel's samples are real, so along y only half of the spectrum is formed:
// with P = RA RB and ky = k1 + RA k2, the first stage is a real transform of
// RA values, and its outputs k1 = 0..RA/2 are the only ones taken further.  The
// rows ky of the plane so formed, with weight 2 where -ky is not among them,
// carry the whole correlation:
//   C(u) = Re sum_{rows ky} w(ky) sum_kx ACC(ky, kx) W^{-(ky u_y + kx u_x)}.
// k1 = 0 is real itself (RB/2 + 1 rows), k1 = 1..RA/2 take RB rows each, so
// the plane has about P/2 rows of P complex values.
//
// Per channel, for the template and then for the window, four phases, each
// ended by a workgroup barrier (P = R1 R2 along x):
//   y1  item (column x, j < RB): real DFT_RA of the rows j + RB a of the volume
//       (lanes along x: one contiguous run per load and wave), twiddle;
//   y2  item (x, k1): DFT_RB over j, in place;
//   x1  item (row, j < R2), lanes along the rows: DFT_R1 in place;
//   x2  item (row, k1 < R1): DFT_R2 into registers, kx = k1 + R1 k2: T^ stays
//       there until the window's x2 accumulates conj(T^) S^.
// All exchanges go through the plane X[row][column] in LDS.  Its row stride is
// odd, so lanes along a row and lanes along a column both fall in distinct
// banks, and every access of an item is its base plus a constant.
//
// What bounds it: the vector units, through the phases' ends.  At P = 144
// (N = 100, r = 20) a point issues 165K wave instructions where the group
// layout issues 211K, with the vector units busy 68% of the time; a phase's
// own instructions fill 75-80% of it, the rest is LDS latency at its start and
// the barrier at its end.  Against the group layout it has no separation of
// packed real rows (24 LDS permutes and as many extra LDS writes per row
// pair), no 48-byte pieces of rows to load, no idle lanes in the groups and
// half the plane, so that up to P = 120 two workgroups share a CU: 447 us per
// 1,024 points against 546 at P = 144, 285 against 403 at P = 120, 105 against
// 263 at P = 72 (the plan table in match_fft.hip has every size).
// Measured and not taken: two channels as one complex signal over all ky
// (twice the plane: at P >= 144 in two classes of ky with every volume row
// read twice; 642 us at P = 144, 1206 at P = 192); loads of two or three
// y1 items in flight together (447 -> 450-485 us); touching the next set's
// cache lines a phase ahead (slower at every size).
#pragma once
#include <hip/hip_runtime.h>
#include "dft.hpp"
#include "epilogue.hpp"
#include "kernels.hpp"
#include "window.hpp"

namespace cfog {

constexpr int gcd_of(int a, int b) { return b ? gcd_of(b, a % b) : a; }

// PF: y1 items of a thread whose loads are issued during the x2 phase before.
// WPE: waves per SIMD that the registers are held to.
// Coprime R1, R2 use the prime-factor map (DftPfa in dft.hpp): no twiddles
// between the x stages.  Column x = (R2 a + R1 b) mod P of the plane is then
// kept at position a R2 + b, so that the accesses are those of the
// common-factor case, where position and column are the same.
template <int P_, int R1_, int R2_, int RA_, int RB_, int NT_, int PF_ = 0, int WPE_ = 0>
struct LaneCfg {
  static constexpr int P = P_, R1 = R1_, R2 = R2_, RA = RA_, RB = RB_, NT = NT_, PF = PF_;
  static constexpr int WPE = WPE_ ? WPE_ : (NT + 255) / 256;  // waves per SIMD the registers must allow
  static_assert(P == R1 * R2 && P == RA * RB, "factors");
  static_assert(NT % 64 == 0 && NT <= 1024, "bad workgroup size");
  static constexpr bool PFA = gcd_of(R1, R2) == 1;
  static constexpr int LD = P | 1;
  static constexpr int KH = RA / 2;          // k1 = 1..KH
  static constexpr int ROW1 = RB / 2 + 1;    // rows of k1 = 0; k1 >= 1 starts at ROW1 + (k1 - 1) RB
  static constexpr int ROWS = ROW1 + KH * RB;
  static_assert(NT >= ROWS, "a row per thread");
  static constexpr int KS1 = (ROWS * R2 + NT - 1) / NT;  // x1 items per thread
  static constexpr int KS2 = (ROWS * R1 + NT - 1) / NT;  // x2 items per thread
  static constexpr int NW = NT / 64;
  static_assert(KS2 <= 8, "accumulators");
  static constexpr int NTW = KH * RB + (PFA ? 0 : P);
  // plane, twiddles, column positions, the surface's rows, argmin scratch
  static constexpr size_t LDS =
      (sizeof(float2) * ((size_t)ROWS * LD + NTW) + 2 * sizeof(short) * P + 15) / 16 * 16 + sizeof(ArgminState) * NW;
  static_assert(LDS <= kMaxLds, "LDS");
};

// The tables of a plan, formed at compile time and copied to LDS by each
// workgroup (forming them there took a small call's workgroups 2 us).
template <class C>
struct LaneTables {
  float2 tw[C::NTW];          // y twiddles W_P^{k1 j} at (k1 - 1) RB + j, then x twiddles W_P^{k j} at k R2 + j
  unsigned short pos[C::P];   // position of column x in the plane
  unsigned short row[C::P];   // offset in floats / 2 | component << 15 of the surface's row u_y (lane_inverse)
};

template <class C>
constexpr LaneTables<C> make_lane_tables() {
  LaneTables<C> t{};
  for (int k = 1; k <= C::KH; ++k)
    for (int j = 0; j < C::RB; ++j) {
      t.tw[(k - 1) * C::RB + j].x = (float)cos2pi(k * j, C::P);
      t.tw[(k - 1) * C::RB + j].y = (float)-sin2pi(k * j, C::P);
    }
  if (!C::PFA)
    for (int k = 0; k < C::R1; ++k)
      for (int j = 0; j < C::R2; ++j) {
        t.tw[C::KH * C::RB + k * C::R2 + j].x = (float)cos2pi(k * j, C::P);
        t.tw[C::KH * C::RB + k * C::R2 + j].y = (float)-sin2pi(k * j, C::P);
      }
  const int ta = inv_mod(C::R2 % C::R1, C::R1), tb = inv_mod(C::R1 % C::R2, C::R2);
  for (int x = 0; x < C::P; ++x) {
    t.pos[x] = (unsigned short)(C::PFA ? (x * ta) % C::R1 * C::R2 + (x * tb) % C::R2 : x);
    // u_y = n2 + RB n1; the values of one n2 share the slots of its column
    const int n1 = x / C::RB, n2 = x % C::RB;
    const int slot = n1 == 0 ? n2 / 2 : C::ROW1 + (n1 - 1) / 2 * C::RB + n2, part = n1 == 0 ? n2 % 2 : (n1 - 1) % 2;
    t.row[x] = (unsigned short)(slot | part << 15);
  }
  return t;
}

template <class C>
__device__ const LaneTables<C> kLaneTables = make_lane_tables<C>();

// The wave-uniform pointer p in scalar registers.
template <class T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const T*>((uint64_t)hi << 32 | lo);
}

// One set of samples: n x n values at src, row stride ld (all wave-uniform, in
// scalar registers: they make buffer descriptors).
struct LaneSet {
  const float* src;
  int ld, n;
};

// Item i of a set as (j, x): i = j n + x.  (Formed where it is used, not kept
// across the channel loop.)
__device__ __forceinline__ int2 lane_item(int n, int i) {
  asm volatile("" : "+v"(i));
  const int j = (int)(((float)i + 0.5f) * (1.0f / (float)n));
  return make_int2(j, i - j * n);
}

// Rows j + RB a (a < RA) of column x of the set; zero past the set.
// Buffer loads: the per-row offset is a scalar, and the descriptor's range
// check (offset of the lane >= size - scalar offset) makes rows past the set
// read as zero.  The scalar offset is held to the size, past which that
// difference would wrap.
template <class C>
__device__ __forceinline__ void lane_load(const LaneSet& S, int j, int x, float (&v)[C::RA]) {
  const int size = ((S.n - 1) * S.ld + S.n) * 4, ld4 = S.ld * 4;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(S.src), 0, size, 0x00027000);
  const int vo = j * ld4 + x * 4;
#pragma unroll
  for (int a = 0; a < C::RA; ++a) {
    const int off = C::RB * a * ld4;
    v[a] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, off < size ? off : size, 0));
  }
}

// The part of y1 after the loads.
template <class C>
__device__ __forceinline__ void lane_y1(int j, int x, const float (&u)[C::RA], float2* X, const float2* twy,
                                        const unsigned short* pos) {
  constexpr int RB = C::RB, LD = C::LD;
  const int p = C::PFA ? pos[x] : x;
  float2 v[C::KH + 1];
  rdft<C::RA>(u, v);
  // k1 = 0 is real: its RB values share RB/2 slots of the column
  reinterpret_cast<float*>(X)[((j >> 1) * LD + p) * 2 + (j & 1)] = v[0].x;
  float2* dst = X + (C::ROW1 + j) * LD + p;
  const float2* tw = twy + j;
  static_for<1, C::KH + 1>([&](auto kI) {
    constexpr int k = decltype(kI)::value;
    const float2 t = tw[(k - 1) * RB];
    if constexpr (2 * k == C::RA) dst[(k - 1) * RB * LD] = make_float2(v[k].x * t.x, v[k].x * t.y);  // real
    else dst[(k - 1) * RB * LD] = cmul(v[k], t);
  });
}

// Phases y1 and y2 of one set.  u: this thread's first PF items, loaded.
// Ends before the closing barrier.
template <class C>
__device__ __forceinline__ void lane_ypass(const LaneSet& S, float (&u)[C::PF ? C::PF : 1][C::RA], float2* X,
                                           const float2* twy, const unsigned short* pos) {
  constexpr int RB = C::RB, LD = C::LD, NT = C::NT, P = C::P;
  const int n = S.n, total = n * RB;
  if constexpr (C::PF > 0) {
#pragma unroll
    for (int s = 0; s < C::PF; ++s) {
      const int2 it = lane_item(n, threadIdx.x + s * NT);
      if ((int)threadIdx.x + s * NT < total) lane_y1<C>(it.x, it.y, u[s], X, twy, pos);
    }
  }
#pragma unroll 1
  for (int i = threadIdx.x + C::PF * NT; i < total; i += NT) {
    float w[C::RA];
    const int2 it = lane_item(n, i);
    lane_load<C>(S, it.x, it.y, w);
    lane_y1<C>(it.x, it.y, w, X, twy, pos);
  }
  __syncthreads();
  const float inv = 1.0f / (float)n;
#pragma unroll 1
  for (int i = threadIdx.x; i < n * (C::KH + 1); i += NT) {
    const int k1 = (int)(((float)i + 0.5f) * inv), x = i - k1 * n, p = C::PFA ? pos[x] : x;
    if (k1 == 0) {
      float2* col = X + p;
      float r[RB + 1];
      float2 v[RB / 2 + 1];
#pragma unroll
      for (int t = 0; t < (RB + 1) / 2; ++t) {
        const float2 z = col[t * LD];
        r[2 * t] = z.x;
        r[2 * t + 1] = z.y;
      }
      rdft<RB>(r, v);
#pragma unroll
      for (int k = 0; k < RB / 2 + 1; ++k) col[k * LD] = v[k];
    } else {
      float2* col = X + (C::ROW1 + (k1 - 1) * RB) * LD + p;
      float2 v[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b) v[b] = col[b * LD];
      dft<RB, -1>(v);
#pragma unroll
      for (int b = 0; b < RB; ++b) col[b * LD] = v[b];
    }
  }
  // the columns past the set are zero (the x stages of the set before wrote
  // them): a thread stays in its row
  constexpr int ROWS = C::ROWS, NC = NT / ROWS;
  const int c = threadIdx.x / ROWS;
  if (c < NC) {
    float2* r = X + (threadIdx.x - c * ROWS) * LD;
#pragma unroll 1
    for (int x = n + c; x < P; x += NC) r[C::PFA ? pos[x] : x] = make_float2(0.f, 0.f);
  }
}

// Phase x1: DFT_R1 of every row in place.
template <class C>
__device__ __forceinline__ void lane_x1(float2* X, const float2* twx) {
  constexpr int R1 = C::R1, R2 = C::R2, ROWS = C::ROWS;
#pragma unroll
  for (int s = 0; s < C::KS1; ++s) {
    if (s && C::WPE > 2) __builtin_amdgcn_sched_barrier(0);  // one item's values in registers at a time
    const int i = threadIdx.x + s * C::NT;
    if (C::KS1 * C::NT == ROWS * R2 || i < ROWS * R2) {
      const int j = i / ROWS, row = i - j * ROWS;
      float2* p = X + row * C::LD + j;
      float2 v[R1];
#pragma unroll
      for (int a = 0; a < R1; ++a) v[a] = p[a * R2];
      dft<R1, -1>(v);
#pragma unroll
      for (int k = 0; k < R1; ++k) p[k * R2] = (C::PFA || k == 0) ? v[k] : cmul(v[k], twx[k * R2 + j]);
    }
  }
}

// Phase x2: DFT_R2 of every row into registers, handed to sink(slot, values).
template <class C, class Sink>
__device__ __forceinline__ void lane_x2(const float2* X, Sink&& sink) {
  constexpr int R1 = C::R1, R2 = C::R2, ROWS = C::ROWS;
  static_for<0, C::KS2>([&](auto sI) {
    constexpr int s = decltype(sI)::value;
    if constexpr (s > 0 && C::WPE > 2) __builtin_amdgcn_sched_barrier(0);
    const int i = threadIdx.x + s * C::NT;
    if (C::KS2 * C::NT == ROWS * R1 || i < ROWS * R1) {
      const int k1 = i / ROWS, row = i - k1 * ROWS;
      const float2* p = X + row * C::LD + k1 * R2;
      float2 v[R2];
#pragma unroll
      for (int b = 0; b < R2; ++b) v[b] = p[b];
      dft<R2, -1>(v);
      sink(sI, v);
    }
  });
}

// The inverse of the accumulators, weighted, for the columns u_x < K.  Ends
// before the closing barrier.
template <class C>
__device__ __forceinline__ void lane_inverse(float2* X, float2 (&acc)[C::KS2][C::R2], const float2* twy,
                                             const float2* twx, const unsigned short* pos, int K) {
  constexpr int R1 = C::R1, R2 = C::R2, RA = C::RA, RB = C::RB, LD = C::LD, NT = C::NT, ROWS = C::ROWS;
  constexpr int KH = C::KH, ROW1 = C::ROW1;
  auto conj_tw = [](float2 t) { return make_float2(t.x, -t.y); };
  static_for<0, C::KS2>([&](auto sI) {
    constexpr int s = decltype(sI)::value;
    if constexpr (s > 0 && C::WPE > 2) __builtin_amdgcn_sched_barrier(0);
    const int i = threadIdx.x + s * NT;
    if (C::KS2 * NT == ROWS * R1 || i < ROWS * R1) {
      const int k1 = i / ROWS, row = i - k1 * ROWS;
      float2* p = X + row * LD + k1 * R2;
      // rows whose -ky is a row too (or the row itself) count once
      const bool once = row == 0 || (RB % 2 == 0 && row == RB / 2) || (RA % 2 == 0 && row >= ROW1 + (KH - 1) * RB);
      const float w = once ? 1.0f / ((float)C::P * C::P) : 2.0f / ((float)C::P * C::P);
      float2 v[R2];
#pragma unroll
      for (int k = 0; k < R2; ++k) v[k] = cscale(acc[s][k], w);
      dft<R2, +1>(v);
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) p[n2] = (C::PFA || n2 == 0) ? v[n2] : cmul(v[n2], conj_tw(twx[k1 * R2 + n2]));
    }
  });
  __syncthreads();
#pragma unroll 1
  for (int i = threadIdx.x; i < ROWS * R2; i += NT) {
    const int n2 = i / ROWS, row = i - n2 * ROWS;
    float2* p = X + row * LD + n2;
    float2 v[R1];
#pragma unroll
    for (int k = 0; k < R1; ++k) v[k] = p[k * R2];
    dft<R1, +1>(v);
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) p[n1 * R2] = v[n1];
  }
  __syncthreads();
  const float inv = 1.0f / (float)K;
#pragma unroll 1
  for (int i = threadIdx.x; i < K * (KH + 1); i += NT) {
    const int k1 = (int)(((float)i + 0.5f) * inv), ux = i - k1 * K, p = C::PFA ? pos[ux] : ux;
    float2* col = X + (k1 ? ROW1 + (k1 - 1) * RB : 0) * LD + p;
    float2 v[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) v[b] = (b < ROW1 || k1) ? col[b * LD] : make_float2(0.f, 0.f);
    dft<RB, +1>(v);
    if (k1 == 0) {  // only the real parts count: two to a slot
#pragma unroll
      for (int t = 0; t < (RB + 1) / 2; ++t) col[t * LD] = make_float2(v[2 * t].x, 2 * t + 1 < RB ? v[2 * t + 1].x : 0.f);
    } else {
#pragma unroll
      for (int n2 = 0; n2 < RB; ++n2) col[n2 * LD] = cmul(v[n2], conj_tw(twy[(k1 - 1) * RB + n2]));
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int i = threadIdx.x; i < K * RB; i += NT) {
    const int n2 = (int)(((float)i + 0.5f) * inv), ux = i - n2 * K, p = C::PFA ? pos[ux] : ux;
    float* r0 = reinterpret_cast<float*>(X) + ((n2 >> 1) * LD + p) * 2 + (n2 & 1);
    float2* col = X + (ROW1 + n2) * LD + p;
    float2 v[RA];
    v[0] = make_float2(*r0, 0.f);
#pragma unroll
    for (int k = 1; k < RA; ++k) v[k] = k <= KH ? col[(k - 1) * RB * LD] : make_float2(0.f, 0.f);
    dft<RA, +1>(v);
    *r0 = v[0].x;
#pragma unroll
    for (int t = 0; t < KH; ++t) col[t * RB * LD] = make_float2(v[1 + 2 * t].x, 2 + 2 * t < RA ? v[2 + 2 * t].x : 0.f);
  }
}

// Control point cpi of job jd over the channels [c0, c1): as match_one in
// match_fft.hip.
template <class C>
__device__ __forceinline__ void lane_match_one(const MatchJob& jd, int cpi, float2* X, const float2* twy,
                                               const float2* twx, const unsigned short* pos, const unsigned short* rows,
                                               ArgminState* red, int c0, int c1, float* __restrict__ part, int g) {
  constexpr int NT = C::NT, KS2 = C::KS2, R2 = C::R2;
  const int4 cp = jd.cps[cpi];
  const int K = 2 * jd.r + 1;
  const CpBoxes bx = cp_boxes(cp.x, cp.y, cp.z, cp.w, jd.N, jd.r, jd.hA, jd.wA, jd.hB, jd.wB);
  if (!bx.inside) {
    if (g == 0) oob_result<NT>(jd, cpi);
    return;
  }
  {
    const size_t planeA = (size_t)jd.hA * jd.wA, planeB = (size_t)jd.hB * jd.wB;
    const float* tA = jd.volA + c0 * planeA + (size_t)bx.ty0 * jd.wA + bx.tx0;
    const float* sB = jd.volB + c0 * planeB + (size_t)bx.sy0 * jd.wB + bx.sx0;
    LaneSet T{uniform_ptr(tA), __builtin_amdgcn_readfirstlane(jd.wA), __builtin_amdgcn_readfirstlane(jd.N)};
    LaneSet S{uniform_ptr(sB), __builtin_amdgcn_readfirstlane(jd.wB),
              __builtin_amdgcn_readfirstlane(jd.N + 2 * jd.r)};
    float2 acc[KS2][R2], th[KS2][R2];
#pragma unroll
    for (int s = 0; s < KS2; ++s)
#pragma unroll
      for (int k = 0; k < R2; ++k) acc[s][k] = make_float2(0.f, 0.f);
    float u[C::PF ? C::PF : 1][C::RA];
    auto preload = [&](const LaneSet& set) {
#pragma unroll
      for (int s = 0; s < C::PF; ++s)
        if (s == 0 || s * NT < set.n * C::RB) {
          const int2 it = lane_item(set.n, threadIdx.x + s * NT);
          lane_load<C>(set, it.x, it.y, u[s]);
        }
    };
    preload(T);
#pragma unroll 1
    for (int c = __builtin_amdgcn_readfirstlane(c1 - c0); c > 0; --c) {
      lane_ypass<C>(T, u, X, twy, pos);
      __syncthreads();
      lane_x1<C>(X, twx);
      __syncthreads();
      preload(S);
      lane_x2<C>(X, [&](auto sI, const float2 (&v)[R2]) {
        constexpr int s = decltype(sI)::value;
#pragma unroll
        for (int k = 0; k < R2; ++k) th[s][k] = v[k];
      });
      __syncthreads();
      lane_ypass<C>(S, u, X, twy, pos);
      __syncthreads();
      lane_x1<C>(X, twx);
      __syncthreads();
      T.src = uniform_ptr(T.src + planeA);
      S.src = uniform_ptr(S.src + planeB);
      if (c > 1) preload(T);
      lane_x2<C>(X, [&](auto sI, const float2 (&v)[R2]) {
        constexpr int s = decltype(sI)::value;
#pragma unroll
        for (int k = 0; k < R2; ++k) acc[s][k] = cmac_conj(acc[s][k], th[s][k], v[k]);
      });
      __syncthreads();
    }
    lane_inverse<C>(X, acc, twy, twx, pos, K);
    __syncthreads();
  }
  const float* Xf = reinterpret_cast<const float*>(X);
  auto corr = [&](int, int uy, int ux) -> float {
    const int row = rows[uy];
    return Xf[((row & 0x7fff) * C::LD + (C::PFA ? pos[ux] : ux)) * 2 + (row >> 15)];
  };
  if (part) {
    for (int i = threadIdx.x; i < K * K; i += NT) {
      const int uy = i / K;
      stg(part + i, corr(i, uy, i - uy * K));
    }
    return;
  }
  ssd_epilogue<NT>(jd, cpi, bx.tx0, bx.ty0, bx.sx0, bx.sy0, corr, red);
}

// The kernel: arguments and work items as match_fft_kernel.
template <class C>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE))) void match_lane_kernel(MatchJob job0, const MatchJob* __restrict__ jobs,
                                                           const int2* __restrict__ tasks, int n_tasks, SplitArgs sp) {
  extern __shared__ float2 smem[];
  float2* X = smem;
  float2* tw = X + (size_t)C::ROWS * C::LD;
  const float2* twx = tw + C::KH * C::RB;
  unsigned short* pos = reinterpret_cast<unsigned short*>(tw + C::NTW);
  unsigned short* rows = pos + C::P;
  ArgminState* red = reinterpret_cast<ArgminState*>(reinterpret_cast<char*>(smem) + C::LDS - sizeof(ArgminState) * C::NW);
  for (int i = threadIdx.x; i < C::NTW; i += C::NT) tw[i] = kLaneTables<C>.tw[i];
  for (int i = threadIdx.x; i < C::P; i += C::NT) {
    pos[i] = kLaneTables<C>.pos[i];
    rows[i] = kLaneTables<C>.row[i];
  }
  const int n_items = split_items(n_tasks, sp);
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    __syncthreads();  // tables ready / previous item's reduction done
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
    lane_match_one<C>(jd, cpi, X, tw, twx, pos, rows, red, g * jd.m / G, (g + 1) * jd.m / G, part, g);
  }
}

}  // namespace cfog
