// backward_f32.hip - the bidirectional gradients of fp32 inputs, features split
// over the waves.
//
// The notation is backward.hip's. A workgroup has M / 32 waves; wave w owns
// features 32 w .. 32 w + 31 and holds its operands of every product in registers:
// W'' (projection), its rows of the aggregate, and W^T (and for dV the aggregate's
// value columns). A 16-row block is then one pass: each wave forms its features'
// part of the gradient, the parts meet in LDS and are added in wave order. fp32
// matrix products take 32 cycles per 2048 FLOP, so the work per row is set by
// them; what a launch of few rows (B2 H8 L1024: 1024 row blocks) needs is all CUs
// at work and no chain of feature steps. Walking a 256-row tile per workgroup with
// the operand tables in LDS, 128 features at a time, took 2 x 39 us (dQ) and 2 x
// 48 us (dK, dV) there on 64 workgroups. (Calls of M <= 128 with enough rows to give
// every CU full tiles take that form all the same: f32_tiles in backward.hip.)
// A block's rows are loaded while the block before is worked on, each tensor's once
// that block's fragments of it are dead: loaded together after them, one third of the
// block before their use, many rows took longer (forward and backward of B8 H8 L4096
// cos M256 1220 us, now 1180; B2 H8 L1024 123.0, now 123.6).
#include <type_traits>

#include "favor_common.hpp"
#include "kernels.hpp"
#include "tile_common.hpp"

namespace favor {

namespace {
using Pf = Mma<float>;
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // rows of 65 floats

// Eight consecutive floats at any 4-byte address as a fragment.
__device__ __forceinline__ f32x8 load8_a4(const float *p) {
  const f32x4 a = *reinterpret_cast<const f32x4_a4 *>(p);
  const f32x4 b = *reinterpret_cast<const f32x4_a4 *>(p + 4);
  return Pf::pack(a, b);
}

// The lane, for the offsets formed once per head. They depend on the lane alone and
// the compiler would keep them over the loop of heads, in scratch (28-248 bytes per
// lane, read again for every head); so it is not told that the lane stays the same.
// Training step of B2 H8 L1024 M256 132 -> 121 us, B40 H4 L200 M64 132 -> 117.
__device__ __forceinline__ int head_lane() {
  int l = lane_id();
  asm volatile("" : "+v"(l));
  return l;
}

// This wave's W'' fragments and seeds, its rows of an aggregate S [M][65] (A
// operand: lane row = feature, k = value columns in loaded order) with their last
// column, and W^T (A operand: lane row = input column 16 kb + lane % 16, k = the 32
// features in chained order). The columns stay in natural order: sixteen lanes
// load (and, of the result, four lane groups store) 64 contiguous bytes.
struct RowOps {
  f32x8 wf[2][2], sa[2][2], wt[4];
  f32x4 bx[2], sz[2];
};
__device__ __forceinline__ void load_row_ops(RowOps &o, const f32x8 *__restrict__ wfr_h,
                                             const float *__restrict__ bq_h,
                                             const float *__restrict__ Wh,
                                             const float *__restrict__ S, int w, int Mr,
                                             float wts) {
  const int l = head_lane();
  const int g = l >> 4;
  const int c16 = l & 15;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int mb = 2 * w + hh;
    o.wf[hh][0] = wfr_h[(size_t)mb * 128 + l];
    o.wf[hh][1] = wfr_h[(size_t)mb * 128 + 64 + l];
    o.bx[hh] = *reinterpret_cast<const f32x4 *>(bq_h + 16 * mb + 4 * g);
    const float *row = S + (size_t)(16 * mb + c16) * 65 + 8 * g;
    o.sa[hh][0] = load8_a4(row);
    o.sa[hh][1] = load8_a4(row + 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) o.sz[hh][j] = S[(size_t)(16 * mb + 4 * g + j) * 65 + 64];
  }
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int m = 32 * w + 16 * (i >> 2) + 4 * g + (i & 3);
      const float x = Wh[min(m, Mr - 1) * kD + 16 * kb + c16];
      v[i] = m < Mr ? x : 0.f;   // padding rows are zero
    }
    o.wt[kb] = Pf::from_f32(v, wts);
  }
}

// Rows t (lane % 16) of a [L][64] tensor, zero past L.
__device__ __forceinline__ void load_rows16(f32x8 (&f)[2], const float *__restrict__ X, int t,
                                            int L) {
  const int g = lane_id() >> 4;
  f[0] = f[1] = Pf::splat(0.f);
  if (t < L) {
    f[0] = load_frag<float>(X + (size_t)t * kD + 8 * g);
    f[1] = load_frag<float>(X + (size_t)t * kD + 32 + 8 * g);
  }
}
__device__ __forceinline__ float row_sum(float v) {   // over the four lane groups
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
__device__ __forceinline__ float dot_rows(const f32x8 (&a)[2], const f32x8 (&b)[2]) {
  float n = 0.f;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int i = 0; i < 8; ++i) n = fmaf(a[k][i], b[k][i], n);
  return row_sum(n);
}
// Columns 16 kb + 4 g .. + 3 of row t.
__device__ __forceinline__ f32x4 load_quad(const float *__restrict__ X, int t, int L, int kb) {
  return t < L ? *reinterpret_cast<const f32x4 *>(X + (size_t)t * kD + 16 * kb +
                                                  4 * (lane_id() >> 4))
               : f32x4{0.f, 0.f, 0.f, 0.f};
}
}  // namespace

constexpr int f32_waves(int M) { return M / 32; }

// Items: 16-row blocks, walked over XCD-local ranges. g~ . q-hat of cos features is
// summed over the features of the very g~ and q-hat that the product with W^T takes.
// For a renormalised row it is (dout . out) eps in units of q-hat, exactly 0 without a
// stabiliser, but the sum's errors cancel part of the other term's and the closed form's
// cannot: dQ's error against 64 bits, B2 H8 L2048, M 192 / 256: 1.094e-6 / 1.030e-6
// summed, 1.111e-6 / 1.057e-6 with the closed form (relative 2-norms).
template <int M, int KN, bool RN>
__global__ __launch_bounds__(64 * f32_waves(M), 2) void k_bwd_dq_f32(
    const float *__restrict__ Q, const float *__restrict__ dout, const float *__restrict__ out,
    const float *__restrict__ rsave, const f32x8 *__restrict__ wfr,
    const float *__restrict__ bqg, const float *__restrict__ W, const float *__restrict__ buf1,
    float *__restrict__ dQ, float2 *__restrict__ aux, int H, int L, float s, int Mr, float cM,
    float wts, int ntiles, int nitems) {
  constexpr int NW = f32_waves(M);
  constexpr bool kDot = KN == kCos;
  constexpr float sgn = KN == kCos ? -1.f : 1.f;
  __shared__ f32x4 red[2][NW][4][64];
  __shared__ float dots[2][NW][16];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float s2half = 0.5f * s * s;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  int begin, end;
  xcd_range(blockIdx.x, gridDim.x, nitems, begin, end);
  for (int first = begin, last; first < end; first = last) {   // the items of one head
    const int bh = first / ntiles;
    const int h = bh % H;
    last = min(end, (bh + 1) * ntiles);
    const int l = head_lane();
    const int g = l >> 4;
    const int c16 = l & 15;
    RowOps op;
    load_row_ops(op, wfr + (size_t)h * (M / 16) * 128, bqg + (size_t)h * M,
                 W + (size_t)h * Mr * kD, buf1 + (size_t)bh * M * 65, w, Mr, wts);
    // a block's rows are loaded while the block before is worked on, each tensor's as
    // soon as that block's fragments are read for the last time
    f32x8 qf[2], df[2], of[2];
    float rs = 0.f;
    auto load_out = [&](int item) __attribute__((always_inline)) {
      const int t = (item - bh * ntiles) * 16 + c16;
      if constexpr (RN) {
        load_rows16(of, out + (size_t)bh * L * kD, t, L);
        rs = t < L ? rsave[(size_t)bh * L + t] : 0.f;
      }
    };
    load_out(first);
    load_rows16(df, dout + (size_t)bh * L * kD, (first - bh * ntiles) * 16 + c16, L);
    load_rows16(qf, Q + (size_t)bh * L * kD, (first - bh * ntiles) * 16 + c16, L);
    for (int item = first; item < last; ++item) {
      const int t = (item - bh * ntiles) * 16 + c16;
      const int buf = item & 1;
      const bool more = item + 1 < last;
      float alpha = 1.f, ud = 0.f, cx = 0.f;   // cx: s^2 g~ . q-hat
      if constexpr (RN) {
        alpha = rs;
        ud = -dot_rows(df, of);
        if (more) load_out(item + 1);
      }
      f32x4 G[2];
      float dot = 0.f;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        G[hh] = Pf::mma(op.sa[hh][0], df[0], zero4);
        G[hh] = Pf::mma(op.sa[hh][1], df[1], G[hh]);
      }
      if (more) load_rows16(df, dout + (size_t)bh * L * kD, t + 16, L);
      if constexpr (KN == kCos && !RN) alpha = cM * expf(s2half * dot_rows(qf, qf));
      f32x4 p[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        p[hh] = Pf::mma(op.wf[hh][0], qf[0], op.bx[hh]);
        p[hh] = Pf::mma(op.wf[hh][1], qf[1], p[hh]);
      }
      if (more) load_rows16(qf, Q + (size_t)bh * L * kD, t + 16, L);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float gj = fmaf(op.sz[hh][j], ud, G[hh][j]);
          if constexpr (kDot) dot = fmaf(gj, feature<KN, Pf>(p[hh][j], op.bx[hh][j]), dot);
          G[hh][j] = sgn * gj * feature_slope<KN, Pf>(p[hh][j], op.bx[hh][j]);
        }
      // the columns of x this wave's sums are finished with
      constexpr int NU = NW >= 4 ? 1 : 4 / NW;
      f32x4 q4[NU];
      if constexpr (kDot) {
#pragma unroll
        for (int k = 0; k < NU; ++k)
          q4[k] = load_quad(Q + (size_t)bh * L * kD, t, L, (w + k * NW) & 3);
      }
      const f32x8 gb = Pf::pack(G[0], G[1]);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) red[buf][w][kb][l] = Pf::mma(op.wt[kb], gb, zero4);
      if constexpr (kDot) {
        dot = row_sum(dot);
        if (g == 0) dots[buf][w][c16] = dot;
      }
      __syncthreads();   // the other buffer's readers are past their sums
      if constexpr (kDot) {
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) d += dots[buf][k][c16];
        cx = s * s * d;
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int kb = w + u * NW;
        if (kb >= 4) break;
        f32x4 v = red[buf][0][kb][l];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += red[buf][k][kb][l];
        if (t < L) {
          if constexpr (kDot) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(cx, q4[u][e], v[e]);
          }
          store4(dQ + ((size_t)bh * L + t) * kD + 16 * kb + 4 * g, v * alpha);
        }
      }
      if (w == 0 && g == 0 && t < L) aux[(size_t)bh * L + t] = make_float2(alpha, alpha * ud);
    }
  }
}

// dK and dV of a 16-row block of keys with the aggregate R = dBuf1.
template <int M, int KN>
__global__ __launch_bounds__(64 * f32_waves(M), 2) void k_bwd_dkv_f32(
    const float *__restrict__ K, const float *__restrict__ V, const f32x8 *__restrict__ wfr,
    const float *__restrict__ bqg, const float *__restrict__ W, const float *__restrict__ dbuf1,
    float *__restrict__ dK, float *__restrict__ dV, int H, int L, float s, int Mr, float cM,
    float wts, int ntiles, int nitems) {
  constexpr int NW = f32_waves(M);
  constexpr float sgn = KN == kCos ? -1.f : 1.f;
  __shared__ f32x4 red[2][NW][8][64];   // input columns, value columns
  __shared__ float dots[2][NW][16];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float s2half = 0.5f * s * s;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  int begin, end;
  xcd_range(blockIdx.x, gridDim.x, nitems, begin, end);
  for (int first = begin, last; first < end; first = last) {   // the items of one head
    const int bh = first / ntiles;
    const int h = bh % H;
    last = min(end, (bh + 1) * ntiles);
    const int l = head_lane();
    const int g = l >> 4;
    const int c16 = l & 15;
    const float *R = dbuf1 + (size_t)bh * M * 65;
    RowOps op;
    f32x8 rb[4];   // R^T: lane row = value column 16 nb + c16, k = features
    load_row_ops(op, wfr + (size_t)h * (M / 16) * 128, bqg + (size_t)h * M,
                 W + (size_t)h * Mr * kD, R, w, Mr, wts);
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          v[i] = R[(size_t)(32 * w + 16 * (i >> 2) + 4 * g + (i & 3)) * 65 + 16 * nb + c16];
        rb[nb] = Pf::from_f32(v, 1.f);
      }
    // a block's rows are loaded as k_bwd_dq_f32 does
    f32x8 kf[2], vf[2];
    load_rows16(vf, V + (size_t)bh * L * kD, (first - bh * ntiles) * 16 + c16, L);
    load_rows16(kf, K + (size_t)bh * L * kD, (first - bh * ntiles) * 16 + c16, L);
    for (int item = first; item < last; ++item) {
      const int t = (item - bh * ntiles) * 16 + c16;
      const int buf = item & 1;
      const bool more = item + 1 < last;
      f32x4 kh[2], G[2];
      float dot = 0.f;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        G[hh] = Pf::mma(op.sa[hh][0], vf[0], op.sz[hh]);
        G[hh] = Pf::mma(op.sa[hh][1], vf[1], G[hh]);
      }
      if (more) load_rows16(vf, V + (size_t)bh * L * kD, t + 16, L);
      float D = 1.f;
      if constexpr (KN == kCos) D = cM * expf(s2half * dot_rows(kf, kf));
      f32x4 p[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        p[hh] = Pf::mma(op.wf[hh][0], kf[0], op.bx[hh]);
        p[hh] = Pf::mma(op.wf[hh][1], kf[1], p[hh]);
      }
      if (more) load_rows16(kf, K + (size_t)bh * L * kD, t + 16, L);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          kh[hh][j] = feature<KN, Pf>(p[hh][j], op.bx[hh][j]);
          dot = fmaf(G[hh][j], kh[hh][j], dot);
          G[hh][j] = sgn * G[hh][j] * feature_slope<KN, Pf>(p[hh][j], op.bx[hh][j]);
        }
      // the columns of k this wave's sums are finished with
      constexpr int NU = 8 / NW;
      constexpr int NQ = NW >= 4 ? 1 : 4 / NW;
      f32x4 k4[NQ];
      if constexpr (KN == kCos) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          k4[q] = load_quad(K + (size_t)bh * L * kD, t, L, (w + q * NW) & 3);
      }
      const f32x8 gb = Pf::pack(G[0], G[1]);
      const f32x8 kb8 = Pf::pack(kh[0], kh[1]);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        red[buf][w][kb][l] = Pf::mma(op.wt[kb], gb, zero4);
        red[buf][w][4 + kb][l] = Pf::mma(rb[kb], kb8, zero4);
      }
      if constexpr (KN == kCos) {
        dot = row_sum(dot);
        if (g == 0) dots[buf][w][c16] = dot;
      }
      __syncthreads();   // the other buffer's readers are past their sums
#pragma unroll
      for (int q = 0; q < NU; ++q) {
        const int u = w + q * NW;   // input columns (u < 4) or value columns
        const int kb = u & 3;
        f32x4 v = red[buf][0][u][l];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += red[buf][k][u][l];
        if (t < L) {
          if (KN == kCos && u < 4) {
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < NW; ++k) d += dots[buf][k][c16];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(s * s * d, k4[q % NQ][e], v[e]);
          }
          store4((u < 4 ? dK : dV) + ((size_t)bh * L + t) * kD + 16 * kb + 4 * g, v * D);
        }
      }
    }
  }
}

// ------------------------------------------------------------ launchers
// One workgroup of eight waves per CU at M = 256; smaller M has fewer waves per
// workgroup and as many more of them.
static int f32_grid(int M, int nitems) {
  const int most = 256 * (256 / M);
  return nitems < most ? nitems : most;
}

#define FAVOR_F32_DISPATCH_M(M_, ...)                                \
  switch (M_) {                                                     \
    case 64: { constexpr int MM = 64; __VA_ARGS__; } break;          \
    case 128: { constexpr int MM = 128; __VA_ARGS__; } break;        \
    case 256: { constexpr int MM = 256; __VA_ARGS__; } break;        \
    default: return hipErrorInvalidValue;                           \
  }

template <int KN, bool RN>
static hipError_t dq_f32(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  const float wts = sh.kernel == 1 ? sh.s / sqrtf((float)sh.Mr) : sh.s;
  const int ntiles = (sh.L + 15) / 16;
  const int nitems = ntiles * sh.BH;
  FAVOR_F32_DISPATCH_M(
      sh.M, hipLaunchKernelGGL((k_bwd_dq_f32<MM, KN, RN>), dim3(f32_grid(MM, nitems)),
                               dim3(64 * f32_waves(MM)), 0, st, (const float *)a.Q,
                               (const float *)a.dout, (const float *)a.out, a.rsave,
                               (const f32x8 *)a.wfr, a.bq, a.W, a.state, (float *)a.dQ, a.aux,
                               sh.H, sh.L, sh.s, sh.Mr, feature_norm(sh), wts, ntiles, nitems));
  return hipGetLastError();
}

hipError_t launch_bwd_dq_f32(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  if (sh.kernel == 1)
    return sh.renorm ? dq_f32<kRelu, true>(sh, a, st) : dq_f32<kRelu, false>(sh, a, st);
  return sh.renorm ? dq_f32<kCos, true>(sh, a, st) : dq_f32<kCos, false>(sh, a, st);
}

template <int KN>
static hipError_t dkv_f32(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  const float wts = sh.kernel == 1 ? sh.s / sqrtf((float)sh.Mr) : sh.s;
  const int ntiles = (sh.L + 15) / 16;
  const int nitems = ntiles * sh.BH;
  FAVOR_F32_DISPATCH_M(
      sh.M, hipLaunchKernelGGL((k_bwd_dkv_f32<MM, KN>), dim3(f32_grid(MM, nitems)),
                               dim3(64 * f32_waves(MM)), 0, st, (const float *)a.K,
                               (const float *)a.V, (const f32x8 *)a.wfr, a.bq, a.W, a.state,
                               (float *)a.dK, (float *)a.dV, sh.H, sh.L, sh.s, sh.Mr,
                               feature_norm(sh), wts, ntiles, nitems));
  return hipGetLastError();
}

hipError_t launch_bwd_dkv_f32(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  return sh.kernel == 1 ? dkv_f32<kRelu>(sh, a, st) : dkv_f32<kCos>(sh, a, st);
}

}  // namespace favor
