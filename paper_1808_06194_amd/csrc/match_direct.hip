// Direct (spatial) evaluation of the correlation term of Eq. 5 (Ye et al.,
// Section III-G) as BF16 MFMA GEMMs with FP32 accumulation: the precision
// alternative to the FP32 FFT path.  The energies and the SSD assembly are the
// same FP64 summed-area-table epilogue as the FFT path.
//
// With T_c the template and S_c the search window of channel c,
//   C(u_y, u_x) = sum_c sum_s sum_tx  S_c(s, tx + u_x) * T_c(s - u_y, tx)
// is one GEMM per control point with
//   M = u_x  (rows of a Hankel matrix built from search row s),
//   N = u_y  (template row s - u_y, zero outside the template),
//   K = (c, s, tx)  (all channels, all search rows, the template columns),
// so every output tile of C accumulates in MFMA registers with no scatter.
// v_mfma_f32_16x16x32_bf16 tiles: M and N are padded to 16, the template
// width to 32.  Every wave keeps all (2r+1)^2 outputs in registers (up to 5 x 5
// tiles) and takes every 8th search row s; the waves' partial sums are added in
// wave order at the end (deterministic).  Operand fragments:
//   A (lane l, u_x block m): 8 bf16 of search row s from column
//      32kc + 8(l/16) + 16m + l%16, read as 5 aligned dwords and realigned by a
//      byte shift (chunk kc + 1 shares all but two of chunk kc's);
//   B (lane l, u_y block n): 8 bf16 of template row s - 16n - l%16, columns
//      32kc + 8(l/16) .. +7, one aligned 16-byte LDS read.
// A search row is used by one wave only, which brings it in by itself, two rows
// ahead: from memory to registers, rounded into a pair of rows of LDS of its own.
// The template (bf16, with 15 zero rows above and below) is shared; where two
// fit LDS, the next channel's is brought in a row at a time meanwhile, so that
// loads and MFMAs overlap and a channel has one barrier (direct_launch says where
// one is taken).
//
// What bounds it: the matrix cores.  N = 128, r = 32 (65 offsets in 80), 1,000
// points: 1.61 ms, 2.18 where each channel's rows were staged before its MFMAs and
// all fragments read per chunk.  That executes 1.28 PFLOP/s at the 2.0 to 2.1 GHz
// that the clock then has, of which 0.77 are not padding; a large library product
// reaches 1.24.  (Steps, in a loop of launches of their own: 2407 us staged; 2195
// with shared fragments, the next chunk's read ahead; 1995 without the moves and
// address arithmetic of that; 1884 with rows brought in by their waves.)
// A body without tests for rows that meet all blocks spills and is slower.
// Precision: inputs are rounded to BF16 (round to nearest, 8 significant bits,
// unit roundoff u = 2^-8), products are exact in FP32, so
//   |C_bf16 - C| <= [(2u + u^2) + gamma_L (1 + u)^2] sum |T S|,
// with gamma_L = L 2^-24 / (1 - L 2^-24) for the longest chain of L FP32
// additions into one output: m channels x ceil(Ws / 8) search rows of a wave x
// ceil(N / 32) chunks of MFMAs of 32 products each, plus the 8 wave partials.
// As sum |T S| <= sqrt(E1 E2) <= (E1 + E2) / 2 and SSD = E1 + E2 - 2C, the
// SSD surface is within [(2u + u^2) + gamma_L (1 + u)^2 + 2^-23] (E1 + E2(d))
// of the exact one (the last term is its own FP32 rounding): about 2^-7, or
// 0.0095 at N = 128, r = 32, m = 9, against ~1e-6 for the FP32 FFT path.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <utility>
#include "cfog.h"
#include "epilogue.hpp"
#include "kernels.hpp"
#include "window.hpp"

namespace cfog {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D_NB = 5;            // max 16-wide blocks of u_x (and u_y): 2r+1 <= 80
constexpr int D_NW = 8;            // waves per workgroup
constexpr int D_NT = 64 * D_NW;
constexpr int D_TPAD = 15;         // zero template rows above and below
constexpr int D_KC = 6;            // most 32-column chunks of a template row (N <= 192)
constexpr int D_RB = 12;           // template rows of a wave staged per batch of loads
constexpr int D_PW = 4;            // waves whose partial correlations are summed together

struct DirectGeom {
  int N, r, K, nblk, NP, Ws;
  int TROWS;  // template rows staged: N + 2 * D_TPAD (row tr holds template row tr - D_TPAD)
  int TLD;    // template row stride in dwords, NP/2 + 4: an odd multiple of 4, so the
              // 16 rows one B fragment reads start in 16 different 4-bank groups
  int SLD;    // dwords of a search row (NP + 16 nblk + 2 bf16: the fragment over-read)
  int tbufs;  // template buffers
  size_t t_bytes, lds;
};

// tbufs: at most that many template buffers.
static DirectGeom direct_geom(int N, int r, int tbufs = 2) {
  DirectGeom g;
  g.N = N;
  g.r = r;
  g.K = 2 * r + 1;
  g.nblk = (g.K + 15) / 16;
  g.NP = (N + 31) / 32 * 32;
  g.Ws = N + 2 * r;
  g.TROWS = N + 2 * D_TPAD;
  g.TLD = g.NP / 2 + 4;
  g.SLD = (g.NP + 16 * g.nblk + 2) / 2;
  g.t_bytes = (size_t)g.TROWS * g.TLD * 4;
  const size_t sb = (size_t)2 * D_NW * g.SLD * 4;
  g.tbufs = tbufs * g.t_bytes + sb <= kMaxLds ? tbufs : 1;
  // after the channels: Cs (K x K) and D_PW partial surfaces; the epilogue's
  // argmin scratch sits behind Cs once the partials are summed
  const size_t c = (size_t)g.K * g.K * 4 * (1 + D_PW) + 16 * D_NW;
  g.lds = std::max(g.tbufs * g.t_bytes + sb, c);
  return g;
}

__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
  const __bf16 a = (__bf16)lo, b = (__bf16)hi;
  return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}

// A row's values 2 (lane + 64 i) and the next, i < NX, of the `bytes` at src
// (wave-uniform); zero past them.  The row is a buffer of its own, whose range
// check gives the zeros.  odd: the last pair straddles the end, so two loads each;
// PAIRS: only the whole pairs.
template <int NX, bool PAIRS>
__device__ __forceinline__ void load_row(const float* src, int bytes, bool odd, int lane, float2 (&v)[NX]) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(uniform_ptr(src)), 0,
                                                                      PAIRS ? bytes & ~7 : bytes, 0x00027000);
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int o = 8 * lane + 512 * i;
    if (!PAIRS && odd) {
      v[i].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0));
      v[i].y = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, o + 4, 0, 0));
    } else {
      v[i] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0));
    }
  }
}
// An odd row's last value, in all lanes.
__device__ __forceinline__ float load_last(const float* src, int bytes) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(uniform_ptr(src)), 0, bytes, 0x00027000);
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, 0, bytes ? bytes - 4 : 0, 0));
}
template <int NX>
__device__ __forceinline__ void put_last(int n, int lane, float last, float2 (&v)[NX]) {
#pragma unroll
  for (int i = 0; i < NX; ++i)
    if (lane + 64 * i == n / 2) v[i].x = last;
}
// Those as packed bf16 pairs, the first w dwords, to dst.
template <int NX>
__device__ __forceinline__ void store_row(unsigned* dst, int w, int lane, const float2 (&v)[NX]) {
#pragma unroll
  for (int i = 0; i < NX; ++i)
    if (lane + 64 * i < w) dst[lane + 64 * i] = pack_bf16x2(v[i].x, v[i].y);
}

// LAST (odd N only): rows as their whole pairs and the last value by itself, which
// halves the loads for more registers and the selection.
template <int NB, int NKC, bool LAST>
__global__ __launch_bounds__(D_NT) void match_direct_kernel(MatchJob jd, DirectGeom g) {
  extern __shared__ unsigned char dsm[];
  constexpr int SX = (16 * NKC + 8 * NB + 1 + 63) / 64;  // dwords of a search row per lane
  constexpr int TX = (16 * NKC + 63) / 64;               // and of a template row
  float* Cs = reinterpret_cast<float*>(dsm);                                    // K x K, after the channels
  ArgminState* red = reinterpret_cast<ArgminState*>(dsm + (size_t)g.K * g.K * 4);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: scalar loop control
  const int l16 = lane & 15, kg = lane >> 4;
  const int N = g.N, r = g.r, K = g.K, NP = g.NP, Ws = g.Ws;
  const size_t planeA = (size_t)jd.hA * jd.wA, planeB = (size_t)jd.hB * jd.wB;
  const bool odd = N & 1;
  unsigned* const T0 = reinterpret_cast<unsigned*>(dsm);          // template buffers, TROWS x TLD dwords
  const int tstep = g.tbufs == 2 ? (int)(g.t_bytes / 4) : 0;      // to the other buffer
  unsigned* const Sw = T0 + g.tbufs * (g.t_bytes / 4) + 2 * wv * g.SLD;  // this wave's two search rows

  for (int cpi = blockIdx.x; cpi < jd.n_cps; cpi += gridDim.x) {
    const int4 cp = jd.cps[cpi];
    const CpBoxes bx = cp_boxes(cp.x, cp.y, cp.z, cp.w, N, r, jd.hA, jd.wA, jd.hB, jd.wB);
    __syncthreads();  // the previous point's epilogue is done with LDS
    if (!bx.inside) {
      oob_result<D_NT>(jd, cpi);
      continue;
    }
    const int tx0 = bx.tx0, ty0 = bx.ty0, sx0 = bx.sx0, sy0 = bx.sy0;
    // acc[m][n]: u_x block m, u_y block n; lane element q is
    // u_x = 16 m + 4 (lane / 16) + q, u_y = 16 n + lane % 16
    f32x4 acc[NB][NB];
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    const float* tsrc = jd.volA + (size_t)ty0 * jd.wA + tx0;
    const float* ssrc = jd.volB + (size_t)sy0 * jd.wB + sx0;
    // the zero rows around the template
    for (int i = threadIdx.x; i < D_TPAD * g.TLD; i += D_NT)
      for (int b = 0; b < g.tbufs; ++b) {
        T0[b * tstep + i] = 0;
        T0[b * tstep + (D_TPAD + N) * g.TLD + i] = 0;
      }
    // this wave's template rows of channel c into buffer Tc
    auto stage_template = [&](int c, unsigned* Tc) {
#pragma unroll 1
      for (int n0 = wv; n0 < N; n0 += D_NW * D_RB) {
        float2 v[D_RB][TX];
#pragma unroll
        for (int u = 0; u < D_RB; ++u) {
          const int n = n0 + u * D_NW;
          load_row<TX, LAST>(tsrc + c * planeA + (size_t)min(n, N - 1) * jd.wA, n < N ? N * 4 : 0, odd, lane, v[u]);
        }
#pragma unroll
        for (int u = 0; u < D_RB; ++u) {
          const int n = n0 + u * D_NW;
          if (n < N) store_row<TX>(Tc + (D_TPAD + n) * g.TLD, NP / 2, lane, v[u]);
        }
      }
      const int n = wv + D_NW * lane;  // the rows' last values, a row per lane, over the zeros just stored
      if (LAST && n < N)
        Tc[(D_TPAD + n) * g.TLD + N / 2] = pack_bf16x2(ldg(tsrc + c * planeA + (size_t)n * jd.wA + N - 1), 0.f);
    };
    // This wave's search rows are s = wv, wv + NW, ... of every channel, one
    // after the other; it alone reads them, so it brings them in by itself: row
    // t + 2 of that sequence is on its way to registers and row t + 1 in LDS while
    // row t is used.
    float2 sv[SX];
    float slast;
    int lc = 0, ls = wv;  // the next row to load
    auto next_row = [&] {
      const bool more = ls < Ws && lc < jd.m;
      const float* src = ssrc + (more ? lc * planeB + (size_t)ls * jd.wB : 0);
      load_row<SX, LAST>(src, more ? Ws * 4 : 0, odd, lane, sv);
      if (LAST) slast = load_last(src, more ? Ws * 4 : 0);
      ls += D_NW;
      if (ls >= Ws) {
        ls = wv;
        ++lc;
      }
    };
    unsigned* srow = Sw;  // the row in use; the other of the two is the next one's
    if (wv < Ws) {
      next_row();
      if (LAST) put_last<SX>(Ws, lane, slast, sv);
      store_row<SX>(Sw, g.SLD, lane, sv);
      next_row();
    }
    stage_template(0, T0);
    __syncthreads();

    unsigned* Tl = T0;
    for (int c = 0; c < jd.m; ++c) {
      // the next channel's template goes into the other buffer, a row of each
      // wave per search row
      const bool ahead = g.tbufs == 2 && c + 1 < jd.m;
      unsigned* const Tn = T0 + (Tl == T0 ? tstep : 0);
      const float* tnext = tsrc + (c + 1) * planeA;
      float2 tv[TX];
      float tlast;
      const unsigned sh = (l16 & 1) * 2;  // e & 1 for every m
      // fragment j: 8 bf16 of a search row from column 16 j + 8 kg + lane % 16;
      // chunk kc takes j = 2 kc + m for block m, so two in a row share all but two
      const int alo = (8 * kg + l16) >> 1;
      auto load_a = [&](const unsigned* row, int j, unsigned (&raw)[5]) {
#pragma unroll
        for (int i = 0; i < 5; ++i) raw[i] = row[8 * j + alo + i];
      };
      auto align = [&](const unsigned (&raw)[5]) {
        unsigned av[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) av[i] = __builtin_amdgcn_alignbyte(raw[i + 1], raw[i], sh);
        return __builtin_bit_cast(bf16x8, av);
      };
      // template row s - 16 n - lane % 16, columns 32 kc + 8 kg .. + 7 (for a
      // block that row s does not meet some other row, not used)
      const unsigned* tb = Tl + (D_TPAD - l16) * g.TLD + 4 * kg;
      auto load_b = [&](int s, int kc, uint4 (&bw)[NB]) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
          bw[n] = *reinterpret_cast<const uint4*>(tb + min(max(s - 16 * n, 0), N + D_TPAD - 1) * g.TLD + 16 * kc);
      };
      constexpr int NEW = NB < 2 ? NB : 2;  // fragments that the next chunk does not share
      bf16x8 A[NB];
      uint4 B[NB];
      if (wv < Ws) {
        unsigned raw[NB][5];
#pragma unroll
        for (int m = 0; m < NB; ++m) load_a(srow, m, raw[m]);
        load_b(wv, 0, B);
#pragma unroll
        for (int m = 0; m < NB; ++m) A[m] = align(raw[m]);
      }
#pragma unroll 1
      for (int s = wv; s < Ws; s += D_NW) {
        // for row s the u_y blocks n whose template rows s - u_y meet [0, N) are
        // those with 0 <= s - 16 n <= N + 14
        const int nhi = min(NB - 1, s >> 4);
        const int nlo = max(0, (s - N + 1) >> 4);
        const int sn = min(s + D_NW, Ws - 1);  // the next row (at the end any: not used)
        unsigned* const snext = Sw + (srow == Sw ? g.SLD : 0);
        if (LAST) put_last<SX>(Ws, lane, slast, sv);
        store_row<SX>(snext, g.SLD, lane, sv);
        if (ahead && s > wv && s - D_NW < N) {
          if (LAST) put_last<TX>(N, lane, tlast, tv);
          store_row<TX>(Tn + (D_TPAD + s - D_NW) * g.TLD, NP / 2, lane, tv);
        }
        next_row();
        if (ahead && s < N) {
          load_row<TX, LAST>(tnext + (size_t)s * jd.wA, N * 4, odd, lane, tv);
          if (LAST) tlast = load_last(tnext + (size_t)s * jd.wA, N * 4);
        }
        // the wave's lanes read each other's parts of the row
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
          // the next chunk's operands are on their way while this one's are used
          const bool row_end = kc + 1 == NKC;
          unsigned raw[NB][5];
          uint4 Bn[NB];
#pragma unroll
          for (int m = row_end ? 0 : NB - NEW; m < NB; ++m)
            load_a(row_end ? snext : srow, row_end ? m : 2 * (kc + 1) + m, raw[m]);
          load_b(row_end ? sn : s, row_end ? 0 : kc + 1, Bn);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int n = 0; n < NB; ++n) {
            if (n >= nlo && n <= nhi) {
#pragma unroll
              for (int m = 0; m < NB; ++m)
                acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m], __builtin_bit_cast(bf16x8, B[n]), acc[m][n], 0, 0, 0);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int m = 0; m < NB; ++m) {
            if (!row_end && m + 2 < NB) A[m] = A[m + 2];
            else A[m] = align(raw[m]);
          }
#pragma unroll
          for (int n = 0; n < NB; ++n) B[n] = Bn[n];
        }
        srow = snext;
      }
      if (ahead) {
        // the last template row, where the loop ended before storing it
        const int sl = wv + (Ws - 1 - wv) / D_NW * D_NW;
        if (wv < Ws && sl < N) {
          if (LAST) put_last<TX>(N, lane, tlast, tv);
          store_row<TX>(Tn + (D_TPAD + sl) * g.TLD, NP / 2, lane, tv);
        }
      } else if (c + 1 < jd.m) {
        __syncthreads();  // MFMA reads of this channel are done
        stage_template(c + 1, Tn);
      }
      __syncthreads();  // the next channel's template is whole, this one's no longer read
      Tl = Tn;
    }
    __syncthreads();  // all MFMA reads of T/S are done: Cs and the partials may overwrite them
    // sum the waves' partial correlations in wave order (deterministic): D_PW
    // waves at a time store theirs side by side behind Cs, then every thread
    // adds the D_PW values of its elements into Cs.  (Adding wave by wave into
    // Cs serialised each wave's read-modify-writes: about 8% of a point's
    // time at K = 65.)
    const int KK = K * K;
    float* part = Cs + KK;
    for (int w0 = 0; w0 < D_NW; w0 += D_PW) {
      if (wv >= w0 && wv < w0 + D_PW) {
        float* mine = part + (size_t)(wv - w0) * KK;
        int lx = 4 * kg, ly = l16;  // (formed here, not kept across the points)
        asm volatile("" : "+v"(lx), "+v"(ly));
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
          for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int ux = 16 * m + lx + q, uy = 16 * n + ly;
              if (ux < K && uy < K) mine[uy * K + ux] = acc[m][n][q];
            }
      }
      __syncthreads();
      for (int i = threadIdx.x; i < KK; i += D_NT) {
        float s = w0 == 0 ? 0.f : Cs[i];
#pragma unroll
        for (int w = 0; w < D_PW; ++w) s += part[(size_t)w * KK + i];
        Cs[i] = s;
      }
      __syncthreads();
    }
    ssd_epilogue<D_NT>(jd, cpi, tx0, ty0, sx0, sy0, Cs, red);
  }
}

size_t direct_workspace_bytes(const cfog_job*, int, int, int) { return 0; }

using DirectKernel = void (*)(MatchJob, DirectGeom);

template <int NB, int... KC>
static constexpr DirectKernel direct_kernel(int nkc, std::integer_sequence<int, KC...>) {
  DirectKernel k = nullptr;
  ((nkc == KC + 1 ? void(k = match_direct_kernel<NB, KC + 1, false>) : void()), ...);
  return k;
}
// The kernel of nblk blocks of offsets and nkc chunks of template columns.
static DirectKernel direct_kernel(int nblk, int nkc) {
  constexpr std::make_integer_sequence<int, D_KC> kcs;
  switch (nblk) {
    case 1: return direct_kernel<1>(nkc, kcs);
    case 2: return direct_kernel<2>(nkc, kcs);
    case 3: return direct_kernel<3>(nkc, kcs);
    case 4: return direct_kernel<4>(nkc, kcs);
    default: return direct_kernel<5>(nkc, kcs);
  }
}
// How a launch of n points runs: two template buffers where they fit, but one
// where two would leave each CU one workgroup although it has registers for two
// and there are points for two (one or two blocks, 118 <= N <= 128 mostly).  There
// odd rows count, and get kernels of their own.  1,000 points, r = 5, two
// buffers against one: N = 118 369 and 344 us, N = 121 392 and 358 (one buffer and
// loads of single values: 392).  A launch with a CU for each point keeps two
// buffers: N = 118, 200 points 95 and 112 us.
static DirectKernel direct_launch(int N, int r, int n, int num_cus, DirectGeom* g) {
  *g = direct_geom(N, r);
  const int nkc = g->NP / 32;
  const bool registers = g->nblk == 1 || (g->nblk == 2 && nkc <= 4);
  if (n > num_cus && registers && 2 * g->lds > kMaxLds) {
    const DirectGeom one = direct_geom(N, r, 1);
    if (2 * one.lds <= kMaxLds) {
      *g = one;
      if (N % 2 && nkc == 4) return g->nblk == 1 ? match_direct_kernel<1, 4, true> : match_direct_kernel<2, 4, true>;
    }
  }
  return direct_kernel(g->nblk, nkc);
}

int init_direct_attributes() {
  for (int nb = 1; nb <= D_NB; ++nb)
    for (int kc = 1; kc <= D_KC; ++kc)
      if (hipFuncSetAttribute((const void*)direct_kernel(nb, kc), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)kMaxLds) != hipSuccess)
        return -2;
  for (const DirectKernel k : {match_direct_kernel<1, 4, true>, match_direct_kernel<2, 4, true>})
    if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds) != hipSuccess)
      return -2;
  return 0;
}

int launch_match_direct(const cfog_job* jobs, int n_jobs, int m, int obj, void*, int num_cus, hipStream_t st) {
  for (int i = 0; i < n_jobs; ++i)
    if (!direct_supported(jobs[i].N, jobs[i].r)) return -1;
  for (int i = 0; i < n_jobs; ++i) {
    const cfog_job& j = jobs[i];
    if (j.n_cps == 0) continue;
    DirectGeom g;
    const DirectKernel kernel = direct_launch(j.N, j.r, j.n_cps, num_cus, &g);
    MatchJob d{};
    d.volA = j.volA; d.satA = j.satA; d.hA = j.hA; d.wA = j.wA;
    d.volB = j.volB; d.satB = j.satB; d.hB = j.hB; d.wB = j.wB;
    d.cps = reinterpret_cast<const int4*>(j.cps);
    d.n_cps = j.n_cps; d.N = j.N; d.r = j.r; d.m = m;
    d.out = reinterpret_cast<Result*>(j.out);
    d.surfaces = j.surfaces;
    d.subpix = reinterpret_cast<float2*>(j.subpix);
    d.obj = obj;
    const int per_cu = std::max(1, (int)(kMaxLds / g.lds));
    const int blocks = std::min(j.n_cps, num_cus * per_cu);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(D_NT), g.lds, st, d, g);
    if (hipGetLastError() != hipSuccess) return -2;
  }
  return 0;
}

bool direct_supported(int N, int r) {
  if (N < 1 || r < 0 || N > kMaxSide || r > kMaxSide) return false;
  const DirectGeom g = direct_geom(N, r);
  // the sizes that are taken: those whose template and whole search window fit LDS.
  // The kernel no longer holds a window; the limit is kept so that the sizes taken
  // stay the same.
  return g.nblk <= D_NB && g.lds <= kMaxLds && g.t_bytes + (size_t)g.Ws * g.SLD * 4 <= kMaxLds;
}

}  // namespace cfog
