// The FFT matcher's second kernel: the correlation of match_fft.hip (the
// notation there), with the 2-D transforms laid out one lane per column or row
// instead of one group of lanes per transform.
//
// A channel's samples are real, so along y only half of the spectrum is formed:
// with P = RA RB and ky = k1 + RA k2, the first stage is a real transform of
// RA values, and its outputs k1 = 0..RA/2 are the only ones taken further.  The
// rows ky of the plane so formed carry the whole correlation, the others being
// their conjugates.
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
// layout issued 211K, with the vector units busy 53% of the time and LDS 37%; the
// rest is latency at each phase's start and the barrier at its end.  Against the
// group layout it has no separation of packed real rows (24 LDS permutes and as
// many extra LDS writes per row pair), no 48-byte pieces of rows to load, no idle
// lanes in the groups and half the plane, so that up to P = 120 two workgroups
// share a CU: 400 us per 1,024 points against 494 at P = 144, 246 against 362 at
// P = 120, 89 against 249 at P = 72 (the plan table in match_fft.hip has every
// size).  It loses by up to 4% where a template is far smaller than its window and
// the points are fewer than CUs (N = 20, r = 26 and 30), as the x stages transform
// the template's zero columns too.
// Measured and not taken: two channels as one complex signal over all ky
// (twice the plane: at P >= 144 in two classes of ky with every volume row
// read twice; 642 us at P = 144, 1206 at P = 192); loads of two or three
// y1 items in flight together (447 -> 450-485 us); touching the next set's
// cache lines a phase ahead (slower at every size); no zero columns written and
// x1 testing its columns instead (4% slower at P = 72 and 100, 8 to 10% at P = 60,
// 80, 96 and 144, 27% at P = 192); the zero columns written four at a time (up to
// 4% slower).
#pragma once
#include <hip/hip_runtime.h>
#include "dft.hpp"
#include "epilogue.hpp"
#include "kernels.hpp"
#include "window.hpp"

namespace cfog {

constexpr int gcd_of(int a, int b) { return b ? gcd_of(b, a % b) : a; }

// Offsets K per axis that a side takes: those whose K x K correlation the group
// layout has room for behind the rows of its inverse's row pairs.
constexpr bool offsets_fit(int P, int K) { return K * K <= 2 * (P - 2 * ((K + 1) / 2)) * (P / 2 + 1); }
constexpr int max_offsets(int P) {
  int K = 1;
  while (offsets_fit(P, K + 2)) K += 2;
  return K;
}

// PF: y1 items of a thread whose loads are issued during the x2 phase before.
// WPE: waves per SIMD that the registers are held to.
// SEP: the real items of y2 are the last threads', so that no wave has both a
// real and a complex transform to run one after the other; else the first ones',
// which takes fewer registers.
// Coprime R1, R2 use the prime-factor map (DftPfa in dft.hpp): no twiddles
// between the x stages.  Column x = (R2 a + R1 b) mod P of the plane is then
// kept at position a R2 + b, so that the accesses are those of the
// common-factor case, where position and column are the same.
template <int P_, int R1_, int R2_, int RA_, int RB_, int I1_, int I2_, int NT_, int PF_, int WPE_, int SEP_>
struct LaneCfg {
  static constexpr int P = P_, R1 = R1_, R2 = R2_, RA = RA_, RB = RB_, I1 = I1_, I2 = I2_, NT = NT_, PF = PF_;
  static constexpr int WPE = WPE_;
  static constexpr bool SEP = SEP_ != 0;
  static_assert(P == R1 * R2 && P == RA * RB && P == I1 * I2, "factors");
  static constexpr int PH = P / 2 + 1;
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
  // the inverse (lane_inverse): whether its DC and Nyquist columns are one
  // complex column, its row pairs at the largest K the side takes, and the
  // items of a thread
  static constexpr bool PACK = P == 120 || P == 192;
  static constexpr int NCOL = PACK ? P / 2 : PH;
  static constexpr int MAXK = max_offsets(P);
  static constexpr int KP2 = ((MAXK + 1) / 2 * I2 + NT - 1) / NT;
  static constexpr int LDP = P | 1;
  static_assert(P * PH <= ROWS * LD && (MAXK + 1) / 2 * LDP + (MAXK * MAXK + 1) / 2 <= ROWS * LD, "inverse in the plane");
  static constexpr int NTW = KH * RB + (PFA ? 0 : P) + I1;
  // plane, twiddles, column positions, argmin scratch
  static constexpr size_t LDS =
      (sizeof(float2) * ((size_t)ROWS * LD + NTW) + sizeof(short) * P + 15) / 16 * 16 + sizeof(ArgminState) * NW;
  static_assert(LDS <= kMaxLds, "LDS");
};

// The tables of a plan, formed at compile time and copied to LDS by each
// workgroup.
template <class C>
struct LaneTables {
  float2 tw[C::NTW];         // y twiddles W_P^{k1 j} at (k1 - 1) RB + j, x twiddles W_P^{k j} at k R2 + j, W_P^k, k < I1
  unsigned short pos[C::P];  // position of column x in the plane
};

template <class C>
constexpr LaneTables<C> make_lane_tables() {
  LaneTables<C> t{};
  int n = 0;
  auto put = [&](int e) {
    t.tw[n].x = (float)cos2pi(e, C::P);
    t.tw[n++].y = (float)-sin2pi(e, C::P);
  };
  for (int k = 1; k <= C::KH; ++k)
    for (int j = 0; j < C::RB; ++j) put(k * j);
  if (!C::PFA)
    for (int k = 0; k < C::R1; ++k)
      for (int j = 0; j < C::R2; ++j) put(k * j);
  for (int k = 0; k < C::I1; ++k) put(k);
  const int ta = inv_mod(C::R2 % C::R1, C::R1), tb = inv_mod(C::R1 % C::R2, C::R2);
  for (int x = 0; x < C::P; ++x)
    t.pos[x] = (unsigned short)(C::PFA ? (x * ta) % C::R1 * C::R2 + (x * tb) % C::R2 : x);
  return t;
}

template <class C>
__device__ const LaneTables<C> kLaneTables = make_lane_tables<C>();

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
// Where a window's byte offsets fit 31 bits, buffer loads: the per-row offset is a scalar, and the descriptor's range
// check (offset of the lane >= size - scalar offset) makes rows past the set
// read as zero.  The scalar offset is held to the size, past which that
// difference would wrap.  WIDE images: 64-bit addresses, and the rows tested.
template <class C, bool WIDE>
__device__ __forceinline__ void lane_load(const LaneSet& S, int j, int x, float (&v)[C::RA]) {
  if constexpr (WIDE) {
    const float* p = S.src + (int64_t)j * S.ld + x;
#pragma unroll
    for (int a = 0; a < C::RA; ++a) {
      v[a] = 0.f;
      if (j + C::RB * a < S.n) v[a] = ldg(p);
      p += (int64_t)C::RB * S.ld;
    }
    return;
  }
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
template <class C, bool WIDE>
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
    lane_load<C, WIDE>(S, it.x, it.y, w);
    lane_y1<C>(it.x, it.y, w, X, twy, pos);
  }
  __syncthreads();
  // The real transform of column x's k1 = 0 values, and the complex one of the
  // values at col.
  auto real = [&](float2* col) {
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
  };
  auto complex = [&](float2* col) {
    float2 v[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) v[b] = col[b * LD];
    dft<RB, -1>(v);
#pragma unroll
    for (int b = 0; b < RB; ++b) col[b * LD] = v[b];
  };
  constexpr int FIRST = C::SEP ? 1 : 0;  // the k1 of item 0
  const float inv = 1.0f / (float)n;
#pragma unroll 1
  for (int i = threadIdx.x; i < n * (C::KH + 1 - FIRST); i += NT) {
    const int q = (int)(((float)i + 0.5f) * inv), x = i - q * n, k1 = q + FIRST;
    float2* col = X + (C::PFA ? pos[x] : x);
    if (!C::SEP && k1 == 0) real(col);
    else complex(col + (C::ROW1 + (k1 - 1) * RB) * LD);
  }
  if constexpr (C::SEP) {
#pragma unroll 1
    for (int x = NT - 1 - (int)threadIdx.x; x < n; x += NT) real(X + (C::PFA ? pos[x] : x));
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

// The inputs of a stage-2 DFT of the inverse: w[b] = get(b) W^{+k1 b}, the
// powers by recurrence from t1 = W^{-k1}.
template <int R2, class Get>
__device__ __forceinline__ void inverse_stage2(float2 (&w)[R2], float2 t1, Get&& get) {
  t1.y = -t1.y;
  float2 t = t1;
  w[0] = get(0);
#pragma unroll
  for (int b = 1; b < R2; ++b) {
    if (b > 1) t = cmul(t, t1);
    w[b] = cmul(get(b), t);
  }
}

// The inverse of the accumulators: returns the correlation as [u_y K + u_x], in
// the plane.
//
// Its order of operations is the group layout's (match_fft.hip: columns
// kx <= P/2 in two stages of I1 I2, then two real rows per complex FFT), and
// not the one that would suit the plane best.  All K x K values are close to
// their mean, which enters in the last stages, so it is the roundings there
// that decide between offsets whose SSDs are equal to rounding: with another
// order, 8 of 135,000 points of ordinary scenes returned another offset than
// the group layout does.
template <class C>
__device__ __forceinline__ const float* lane_inverse(float2* X, float2 (&acc)[C::KS2][C::R2], const float2* twi, int K) {
  constexpr int P = C::P, PH = C::PH, R1 = C::R1, R2 = C::R2, I1 = C::I1, I2 = C::I2, NT = C::NT;
  constexpr int RA = C::RA, RB = C::RB, ROWS = C::ROWS, ROW1 = C::ROW1, KH = C::KH, LDP = C::LDP;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // no index of the inverse is kept across the channel loop
  // the accumulators as the half plane X[ky][kx <= P/2] (Hermitian symmetry)
  static_for<0, C::KS2>([&](auto sI) {
    constexpr int s = decltype(sI)::value;
    const int i = tid + s * NT;
    if (C::KS2 * NT == ROWS * R1 || i < ROWS * R1) {
      const int k1 = i / ROWS, row = i - k1 * ROWS;
      const int q = row < ROW1 ? 0 : (row - ROW1) / RB + 1;
      const int ky = row < ROW1 ? RA * row : q + RA * (row - ROW1 - (q - 1) * RB);
      // rows whose -ky is a row too (or the row itself)
      const bool once = row == 0 || (RB % 2 == 0 && row == RB / 2) || (RA % 2 == 0 && q == KH);
      static_for<0, R2>([&](auto kI) {
        constexpr int k2 = decltype(kI)::value;
        int kx = k1 + R1 * k2;
        if constexpr (C::PFA) {
          constexpr int ta = inv_mod(R2 % R1, R1), tb = inv_mod(R1 % R2, R2);
          kx = (R2 * ta * k1 + R1 * tb * k2) % P;
        }
        if (2 * kx <= P) X[ky * PH + kx] = acc[s][k2];
        if (!once && (2 * kx >= P || kx == 0)) X[(P - ky) * PH + (kx ? P - kx : 0)] = make_float2(acc[s][k2].x, -acc[s][k2].y);
      });
    }
  });
  __syncthreads();
  // columns, in place: u_y = k1 + I1 k2 ends up in row k1 I2 + k2.  The DC and
  // Nyquist columns are real: where PACK, they are the real and the imaginary
  // part of one.
#pragma unroll 1
  for (int i = tid; i < C::NCOL * I2; i += NT) {
    const int j = i / C::NCOL, kx = i - j * C::NCOL;
    float2* col = X + j * PH + kx;
    float2 v[I1];
#pragma unroll
    for (int a = 0; a < I1; ++a) {
      v[a] = col[a * I2 * PH];
      if (C::PACK && kx == 0) {
        const float2 n = col[a * I2 * PH + P / 2];
        v[a] = make_float2(v[a].x - n.y, v[a].y + n.x);
      }
    }
    dft<I1, +1>(v);
#pragma unroll
    for (int k = 0; k < I1; ++k) col[k * I2 * PH] = v[k];
  }
  __syncthreads();
#pragma unroll 1
  for (int i = tid; i < C::NCOL * I1; i += NT) {
    const int k1 = i / C::NCOL, kx = i - k1 * C::NCOL;
    float2* col = X + k1 * I2 * PH + kx;
    float2 w[I2];
    inverse_stage2<I2>(w, twi[k1], [&](int b) { return col[b * PH]; });
    dft<I2, +1>(w);
#pragma unroll
    for (int k2 = 0; k2 < I2; ++k2) {
      if (C::PACK && kx == 0) {
        col[k2 * PH] = make_float2(w[k2].x, 0.f);
        col[k2 * PH + P / 2] = make_float2(w[k2].y, 0.f);
      } else {
        col[k2 * PH] = w[k2];
      }
    }
  }
  __syncthreads();
  // rows 2p and 2p + 1 as one complex row.  Once every thread holds its
  // inputs, the stage-1 outputs go to the start of the plane, pair by pair, and
  // the surface behind them.
  const int npair = (K + 1) >> 1;
  float2 v[C::KP2][I1];
  static_for<0, C::KP2>([&](auto sI) {
    constexpr int s = decltype(sI)::value;
    const int i = tid + s * NT, p = i / I2, j = i - p * I2;
    if (p < npair) {
      const float2* r1 = X + (2 * p % I1 * I2 + 2 * p / I1) * PH;
      const float2* r2 = X + ((2 * p + 1) % I1 * I2 + (2 * p + 1) / I1) * PH;
      const bool has2 = 2 * p + 1 < K;
#pragma unroll
      for (int a = 0; a < I1; ++a) {
        const int kx = j + I2 * a;
        const bool lo = kx <= P / 2;
        const int kk = lo ? kx : P - kx;
        const float2 v1 = r1[kk];
        const float2 v2 = has2 ? r2[kk] : make_float2(0.f, 0.f);
        v[s][a] = lo ? make_float2(v1.x - v2.y, v1.y + v2.x) : make_float2(v1.x + v2.y, v2.x - v1.y);
      }
    }
  });
  __syncthreads();
  static_for<0, C::KP2>([&](auto sI) {
    constexpr int s = decltype(sI)::value;
    const int i = tid + s * NT, p = i / I2, j = i - p * I2;
    if (p < npair) {
      float2* r = X + p * LDP + j;
      dft<I1, +1>(v[s]);
#pragma unroll
      for (int k = 0; k < I1; ++k) r[k * I2] = v[s][k];
    }
  });
  __syncthreads();
  float* Cs = reinterpret_cast<float*>(X + npair * LDP);
  const float norm = 1.0f / ((float)P * (float)P);
#pragma unroll 1
  for (int i = tid; i < npair * I1; i += NT) {
    const int p = i / I1, k1 = i - p * I1;
    const float2* r = X + p * LDP + k1 * I2;
    float2 w[I2];
    inverse_stage2<I2>(w, twi[k1], [&](int b) { return r[b]; });
    dft<I2, +1>(w);
    float* c = Cs + 2 * p * K + k1;
#pragma unroll
    for (int k2 = 0; k2 < I2; ++k2) {
      if (k1 + I1 * k2 < K) {
        c[I1 * k2] = w[k2].x * norm;
        if (2 * p + 1 < K) c[K + I1 * k2] = w[k2].y * norm;
      }
    }
  }
  __syncthreads();
  return Cs;
}

// Control point cpi of job jd over the channels [c0, c1): as match_one in
// match_fft.hip.
template <class C, bool WIDE>
__device__ __forceinline__ void lane_match_one(const MatchJob& jd, int cpi, float2* X, const float2* twy,
                                               const float2* twx, const float2* twi, const unsigned short* pos,
                                               ArgminState* red, int c0, int c1, float* __restrict__ part, int g) {
  constexpr int NT = C::NT, KS2 = C::KS2, R2 = C::R2;
  const int4 cp = jd.cps[cpi];
  const int K = 2 * jd.r + 1;
  const CpBoxes bx = cp_boxes(cp.x, cp.y, cp.z, cp.w, jd.N, jd.r, jd.hA, jd.wA, jd.hB, jd.wB);
  if (!bx.inside) {
    if (g == 0) oob_result<NT>(jd, cpi);
    return;
  }
  const float* Cs;
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
          lane_load<C, WIDE>(set, it.x, it.y, u[s]);
        }
    };
    preload(T);
#pragma unroll 1
    for (int c = __builtin_amdgcn_readfirstlane(c1 - c0); c > 0; --c) {
      lane_ypass<C, WIDE>(T, u, X, twy, pos);
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
      lane_ypass<C, WIDE>(S, u, X, twy, pos);
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
    Cs = lane_inverse<C>(X, acc, twi, K);
  }
  if (part) {
    for (int i = threadIdx.x; i < K * K; i += NT) stg(part + i, Cs[i]);
    return;
  }
  ssd_epilogue<NT>(jd, cpi, bx.tx0, bx.ty0, bx.sx0, bx.sy0, Cs, red);
}

// The kernel: arguments and work items as match_fft_kernel.
template <class C, bool WIDE>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(C::WPE))) void match_lane_kernel(MatchJob job0, const MatchJob* __restrict__ jobs,
                                                           const int2* __restrict__ tasks, int n_tasks, SplitArgs sp) {
  extern __shared__ float2 smem[];
  float2* X = smem;
  float2* tw = X + (size_t)C::ROWS * C::LD;
  const float2* twx = tw + C::KH * C::RB;
  const float2* twi = tw + C::NTW - C::I1;
  unsigned short* pos = reinterpret_cast<unsigned short*>(tw + C::NTW);
  ArgminState* red = reinterpret_cast<ArgminState*>(reinterpret_cast<char*>(smem) + C::LDS - sizeof(ArgminState) * C::NW);
  for (int i = threadIdx.x; i < C::NTW; i += C::NT) tw[i] = kLaneTables<C>.tw[i];
  for (int i = threadIdx.x; i < C::P; i += C::NT) pos[i] = kLaneTables<C>.pos[i];
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
    lane_match_one<C, WIDE>(jd, cpi, X, tw, twx, twi, pos, red, g * jd.m / G, (g + 1) * jd.m / G, part, g);
  }
}

}  // namespace cfog
