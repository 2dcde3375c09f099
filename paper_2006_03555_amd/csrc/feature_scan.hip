// feature_scan.hip - the causal output and the causal gradients of bf16 inputs:
// chunk scans with the features split over the waves.
//
// The notation is backward.hip's. One workgroup per (head, segment of the
// forward plan) walks 64-token chunks, for the output and dQ forwards with the
// aggregate S = G^PS, for dK and dV backwards with R, the aggregate of the rows
// after the chunk. Wave w owns M / NW features (NW = 8 waves; 4 at M = 64): its W''
// fragments, its slice of the aggregate (fp32 accumulators) and the chunk's
// features of the other side never leave its registers, and every row fragment
// it reads from LDS meets all of its features. What the waves exchange through
// LDS is bf16 and small: the rows of the chunk, the masked intra-chunk matrix
// P (no feature dimension: formed once, by blocks) and the products that the
// last contraction, over all features, takes in another split.
#include <type_traits>

#include "favor_common.hpp"
#include "kernels.hpp"
#include "tile_common.hpp"

namespace favor {

constexpr int scan_waves(int M) { return M == 256 ? 8 : 4; }
// M = 256 fills a CU's LDS: rows are double-buffered and W^T is read from LDS.
// Smaller M holds the rows once and W^T in registers, which leaves room for two
// workgroups per CU.
constexpr bool scan_wide(int M) { return M == 256; }

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // rows of 65 floats

// Offset of element 8 s of row r in a staged tile of 64 rows. Wide: the eight
// 16-byte slots of a row are permuted by its pair number, so that a fragment load
// (16 rows, one slot per lane group) meets all banks evenly without padding, which
// the wide kernels' LDS has no room for. Else rows of 72 elements: the addresses
// of all loads then differ by constants, which saves the registers.
template <bool WIDE>
__device__ __forceinline__ int tile_at(int r, int s) {
  return WIDE ? r * kD + 8 * (s ^ ((r >> 1) & 7)) : r * (kD + kKsPad) + 8 * s;
}
template <bool WIDE> constexpr int tile_size() { return 64 * (kD + (WIDE ? 0 : kKsPad)); }

// Sum over the eight lanes of an aligned group (DPP: pairs, quads, half-rows).
__device__ __forceinline__ float oct_sum_f32(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, false));
  return v;
}

// x . y over eight bf16 pairs, fp32 accumulation (dot2: exact products).
__device__ __forceinline__ float dot8(bf16x8 x, bf16x8 y) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  struct Pairs { bf16x2 p[4]; };
  const Pairs a = __builtin_bit_cast(Pairs, x), b = __builtin_bit_cast(Pairs, y);
  float n = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) n = __builtin_amdgcn_fdot2_f32_bf16(a.p[i], b.p[i], n, false);
  return n;
}

// Selection fragment in loaded k order: B[k][c] = (k == 8 (c / 4) + 4 half + c % 4):
// moves value column perm_col(2 kh + half, c) of a row fragment of k-step kh into
// lane c.
__device__ __forceinline__ bf16x8 scan_select(int half) {
  const int l = lane_id();
  const int c = l & 15;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (8 * (l >> 4) + i == 8 * (c >> 2) + 4 * half + (c & 3)) ? 1.f : 0.f;
  return Mma<bf16>::from_f32(v, 1.f);
}

// Four floats as four bf16 in one 8-byte store: slots 4 h .. 4 h + 3 of a fragment.
__device__ __forceinline__ void store_half_frag(bf16x8 *f, int h, f32x4 v) {
  store4(reinterpret_cast<bf16 *>(f) + 4 * h, v);
}

// One chunk's rows and row weights. X: the rows whose gradient is taken and Y
// their partners (dQ: queries and output gradients; dK: keys and values); Z, U
// the other side (dQ: keys and values; dK: queries and output gradients).
template <bool WIDE>
struct ScanTile {
  bf16 X[tile_size<WIDE>()], Y[tile_size<WIDE>()], Z[tile_size<WIDE>()], U[tile_size<WIDE>()];   // see tile_at
  float wz[64];   // weight of a z row: D~ (keys) or alpha (queries)
  float ez[64];   // its last column: D~ or alpha u_d
  float uy[64];   // last column of an x row's partner: u_d (dQ) or 1 (dK)
  bf16x8 EF[2][4];   // ez in chained row order, one fragment per lane group
};

template <int M>
struct ScanSmem {
  ScanTile<scan_wide(M)> tile[scan_wide(M) ? 2 : 1];
  bf16x8 UF[4][2][64];          // (w U)^T: row = value column (permuted), k = z rows
  bf16x8 PF[4][2][64];          // P of x block, z half: B operand, k = 32 z rows
  bf16x8 GF[4][M / 32][64];     // gradient of the projections: lane = x row, k = features
  float dots[scan_waves(M)][64];   // g~ . xf of each wave's features (cos)
  bf16x8 WT[scan_wide(M) ? 4 : 1][M / 32][64];   // W^T: lane = input column (permuted), k = features
  float sz[M];                  // last column of the aggregate before the chunk
  float ox[2][64];              // factor of an x row's gradient, by chunk parity: alpha (dQ) or D~ (dK)
  // else, to save registers: the selection fragments and b''
  bf16x8 sel[scan_wide(M) ? 1 : 2][64];
  float bq[scan_wide(M) ? 4 : M];
};

// dQ (KEY false) or dK (KEY true). With a = the aggregate before (dQ: prefix S; dK:
// suffix R) and zf, xf the features of the z and x rows:
//   P[z][x] = w_z (u_z . y_x) + e_z uy_x   for z <= x (dQ), z >= x (dK)
//   g~[m][x] = a y + zf^T P + a_d uy       (one accumulation)
//   grad x = ox (W^T (g~ o slope) + s^2 (g~ . xf) x)      (cos features)
//   a += zf (x) [w u, e]
// The dot product g~ . xf of cos features is summed over the features of the very
// g~ and xf that the first term takes: their bf16 errors then cancel in part. The
// closed forms (u . Buf2 of a renormalised row: exactly 0 without a stabiliser; dK:
// v . (R^T k-hat)[:d] + (R^T k-hat)[d] from the dV pass) save the cosines but are
// further from 64 bits: B2 H8 L2048 M256 dQ 4.9e-3 against 4.5e-3, dK 4.6e-3 against
// 4.3e-3 (relative 2-norms).
// Wide: two barriers per chunk: P, (w U)^T and the next tile are formed while the
// previous chunk's gradient is contracted; g~, the fold into the aggregate and
// the staging of the next tile follow the first barrier, the contraction with W
// (each wave: one 16-row block, half of the input columns, all features) the
// second.
template <int M, int KN, bool RN, bool KEY, bool ACC>
__global__ __launch_bounds__(64 * scan_waves(M), scan_wide(M) ? 1 : 2) void k_bwd_row_scan(
    const bf16 *__restrict__ Q, const bf16 *__restrict__ K, const bf16 *__restrict__ V,
    const bf16 *__restrict__ dout, const bf16 *__restrict__ out, const float *__restrict__ rsave,
    const bf16x8 *__restrict__ wfr, const float *__restrict__ bqg, const float *__restrict__ W,
    const float *__restrict__ states, bf16 *__restrict__ dX, float2 *__restrict__ aux,
    int H, int L, int seg_len, int nseg, float s, int Mr, float cM, float wts) {
  constexpr bool kDot = KN == kCos;
  constexpr int NW = scan_waves(M);
  constexpr int FB = M / 16 / NW;      // 16-feature blocks per wave
  constexpr int NS = M / 32;           // feature steps of the last contraction
  constexpr bool kWide = scan_wide(M);
  constexpr int RPT = 8 / NW;          // rows a thread stages (eighths of a row)
  constexpr float sgn = KN == kCos ? -1.f : 1.f;
  using P = Mma<bf16>;
  using frag = bf16x8;
  __shared__ ScanSmem<M> sm;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int bh = item / nseg;
  const int seg = item - bh * nseg;
  const int h = bh % H;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int g = l >> 4;
  const int c16 = l & 15;
  const float s2half = 0.5f * s * s;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  const int r0 = seg * seg_len;
  const int r1 = min(L, r0 + seg_len);
  if (r0 >= r1) return;
  const int nch = (r1 - r0 + 63) / 64;

  const bf16 *Xh = (KEY ? K : Q) + (size_t)bh * L * kD;
  const bf16 *Yh = (KEY ? V : dout) + (size_t)bh * L * kD;
  const bf16 *Zh = (KEY ? Q : K) + (size_t)bh * L * kD;
  const bf16 *Uh = (KEY ? dout : V) + (size_t)bh * L * kD;
  const bf16 *Oh = KEY ? nullptr : out + (size_t)bh * L * kD;
  const float *rsh = KEY ? nullptr : rsave + (size_t)bh * L;
  float2 *auh = aux + (size_t)bh * L;

  // the chunk's rows in registers until staged: row sr, columns 8 (tid % 8) ..
  struct Regs {
    frag x, y, z, u, o;
    float rs;
    float2 a;
  };
  Regs rg[RPT];
  auto load_rows = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int t = t0 + (tid >> 3) + 8 * NW * k;
      const size_t off = (size_t)t * kD + 8 * (tid & 7);
      const frag z8 = P::splat(0.f);
      rg[k].x = rg[k].y = rg[k].z = rg[k].u = rg[k].o = z8;
      rg[k].rs = 0.f;
      rg[k].a = make_float2(0.f, 0.f);
      if (t < r1) {
        rg[k].x = load_frag<bf16>(Xh + off);
        rg[k].y = load_frag<bf16>(Yh + off);
        rg[k].z = load_frag<bf16>(Zh + off);
        rg[k].u = load_frag<bf16>(Uh + off);
        if constexpr (KEY) {
          rg[k].a = auh[t];
        } else if constexpr (RN) {
          rg[k].o = load_frag<bf16>(Oh + off);
          rg[k].rs = rsh[t];
        }
      }
    }
  };
  auto stage_rows = [&](ScanTile<kWide> &tl, int t0, int par) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int r = (tid >> 3) + 8 * NW * k;
      const int at = tile_at<kWide>(r, tid & 7);
      const int t = t0 + r;
      store_frag<bf16>(&tl.X[at], rg[k].x);
      store_frag<bf16>(&tl.Y[at], rg[k].y);
      store_frag<bf16>(&tl.Z[at], rg[k].z);
      store_frag<bf16>(&tl.U[at], rg[k].u);
      // D~ of the key row
      float D = 1.f;
      if constexpr (KN == kCos) {
        const frag &kr = KEY ? rg[k].x : rg[k].z;
        D = cM * expf(s2half * oct_sum_f32(dot8(kr, kr)));
      }
      D = t < r1 ? D : 0.f;
      float wz, ez, uy, ox;
      if constexpr (KEY) {
        wz = rg[k].a.x;
        ez = rg[k].a.y;
        uy = 1.f;
        ox = D;
      } else {
        wz = D;
        ez = D;
        if constexpr (RN) {
          ox = rg[k].rs;
          uy = -oct_sum_f32(dot8(rg[k].y, rg[k].o));
        } else {
          float a = 1.f;
          if constexpr (KN == kCos) a = cM * expf(s2half * oct_sum_f32(dot8(rg[k].x, rg[k].x)));
          ox = t < r1 ? a : 0.f;
          uy = 0.f;
        }
        if ((tid & 7) == 0 && t < r1) auh[t] = make_float2(ox, ox * uy);
      }
      if ((tid & 7) == 0) {
        tl.wz[r] = wz;
        tl.ez[r] = ez;
        tl.uy[r] = uy;
        sm.ox[par][r] = ox;
        reinterpret_cast<bf16 *>(&tl.EF[r >> 5][(r >> 2) & 3])[4 * ((r >> 4) & 1) + (r & 3)] =
            (bf16)ez;
      }
    }
  };
  auto chunk_t0 = [&](int c) { return r0 + 64 * (KEY ? nch - 1 - c : c); };
  load_rows(chunk_t0(0));

  // W'' of this wave's features (both orientations of the projection), b'' per
  // result row and column, and W^T of the last contraction's columns
  frag wf[FB][2];
  f32x4 bx[FB];
  float bz[FB];
#pragma unroll
  for (int mb = 0; mb < FB; ++mb) {
    const int mbg = w * FB + mb;
    const frag *wp = wfr + ((size_t)h * (M / 16) + mbg) * 2 * 64 + l;
    wf[mb][0] = wp[0];
    wf[mb][1] = wp[64];
    const float *bp = bqg + (size_t)h * M + 16 * mbg;
    bx[mb] = *reinterpret_cast<const f32x4 *>(bp + 4 * g);
    bz[mb] = bp[c16];
  }
  // W^T for the last contraction. Wide: in LDS, columns in store order; wave w
  // takes x block w % 4 and column blocks 2 (w / 4), 2 (w / 4) + 1. Else: wave w
  // holds the 16 columns 16 w .. and takes every x block.
  frag wt[kWide ? 1 : NS];
  {
    const float *Wh = W + (size_t)h * Mr * kD;
    if constexpr (kWide) {
      // a thread takes four columns (lanes 4 a .. 4 a + 3) of eight features
      static_assert(4 * NS * 16 == 64 * NW, "one unit per thread");
      const int a4 = tid & 3, gg = (tid >> 2) & 3, ks = (tid >> 4) % NS, kb = tid / (16 * NS);
      f32x4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int m = 32 * ks + 16 * (i >> 2) + 4 * gg + (i & 3);
        v[i] = m < Mr ? *reinterpret_cast<const f32x4 *>(Wh + m * kD + perm_col(kb, 4 * a4)) : zero4;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float col[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) col[i] = v[i][q];
        sm.WT[kb][ks][16 * gg + 4 * a4 + q] = P::from_f32(col, wts);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < NS; ++ks) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int m = 32 * ks + 16 * (i >> 2) + 4 * g + (i & 3);
          v[i] = m < Mr ? Wh[m * kD + 16 * w + c16] : 0.f;   // padding rows are zero
        }
        wt[ks] = P::from_f32(v, wts);
      }
    }
  }
  // a^T: acc[nb][mb] rows = value column perm_col(nb, 4 g + j) (block 4: the last
  // column, replicated), lane = feature 16 (w FB + mb) + lane % 16
  f32x4 acc[5][FB];
  {
    const float *S = states + ((size_t)bh * nseg + seg) * M * 65;
#pragma unroll
    for (int mb = 0; mb < FB; ++mb) {
      const float *row = S + (size_t)(16 * (w * FB + mb) + c16) * 65;
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
        acc[nb][mb] = *reinterpret_cast<const f32x4_a4 *>(row + perm_col(nb, 4 * g));
      const float e = row[64];
      acc[4][mb] = f32x4{e, e, e, e};
    }
  }
  if (!kWide && w == 0) {
    sm.sel[0][l] = scan_select(0);
    sm.sel[kWide ? 0 : 1][l] = scan_select(1);
  }
  if (!kWide && tid < M) sm.bq[tid] = bqg[(size_t)h * M + tid];
  stage_rows(sm.tile[0], chunk_t0(0), 0);
  if (nch > 1) load_rows(chunk_t0(1));
  __syncthreads();

  for (int c = 0; c < nch; ++c) {
    const int t0 = chunk_t0(c);
    const ScanTile<kWide> &tl = sm.tile[kWide ? c & 1 : 0];
    // (w U)^T, one 16-row block and 32 columns per wave and unit
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int tb = w & 3;
      const int kh = (w >> 2) + k;
      const frag u = load_frag<bf16>(&tl.U[tile_at<kWide>(16 * tb + c16, 4 * kh + g)]);
      const f32x4 wz = *reinterpret_cast<const f32x4 *>(&tl.wz[16 * tb + 4 * g]);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const f32x4 t = P::mma(u, kWide ? scan_select(half) : sm.sel[kWide ? 0 : half][l], zero4);
        store_half_frag(&sm.UF[2 * kh + half][tb >> 1][l], tb & 1, t * wz);
      }
    }
    // P of x block w % 4, z rows 32 zs .. 32 zs + 31
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int ib = w & 3;
      const int zs = (w >> 2) + k;
      if (KEY ? 2 * zs + 1 < ib : 2 * zs > ib) continue;   // wholly masked
      const frag y0 = load_frag<bf16>(&tl.Y[tile_at<kWide>(16 * ib + c16, g)]);
      const frag y1 = load_frag<bf16>(&tl.Y[tile_at<kWide>(16 * ib + c16, 4 + g)]);
      const float uy = tl.uy[16 * ib + c16];
      f32x4 pt[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int zb = 2 * zs + q;
        const frag u0 = load_frag<bf16>(&tl.U[tile_at<kWide>(16 * zb + c16, g)]);
        const frag u1 = load_frag<bf16>(&tl.U[tile_at<kWide>(16 * zb + c16, 4 + g)]);
        f32x4 t = P::mma(u0, y0, zero4);
        t = P::mma(u1, y1, t);
        const f32x4 wz = *reinterpret_cast<const f32x4 *>(&tl.wz[16 * zb + 4 * g]);
        const f32x4 ez = *reinterpret_cast<const f32x4 *>(&tl.ez[16 * zb + 4 * g]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int z = 16 * zb + 4 * g + j, x = 16 * ib + c16;
          pt[q][j] = (KEY ? z >= x : z <= x) ? fmaf(wz[j], t[j], ez[j] * uy) : 0.f;
        }
      }
      sm.PF[ib][zs][l] = P::pack(pt[0], pt[1]);
    }
    // features of the z rows (A operand: row = feature, k = z rows)
    frag zt[FB][2];
#pragma unroll
    for (int zs = 0; zs < 2; ++zs) {
      f32x4 f[FB][2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const frag z0 = load_frag<bf16>(&tl.Z[tile_at<kWide>(32 * zs + 16 * q + c16, g)]);
        const frag z1 = load_frag<bf16>(&tl.Z[tile_at<kWide>(32 * zs + 16 * q + c16, 4 + g)]);
#pragma unroll
        for (int mb = 0; mb < FB; ++mb) {
          f32x4 p = P::mma(z0, wf[mb][0], f32x4{bz[mb], bz[mb], bz[mb], bz[mb]});
          p = P::mma(z1, wf[mb][1], p);
#pragma unroll
          for (int j = 0; j < 4; ++j) f[mb][q][j] = feature<KN, P>(p[j], bz[mb]);
        }
      }
#pragma unroll
      for (int mb = 0; mb < FB; ++mb) zt[mb][zs] = P::pack(f[mb][0], f[mb][1]);
    }
    // the aggregate before the chunk as A operand (row = feature, k = value columns)
    frag sa[FB][2];
#pragma unroll
    for (int mb = 0; mb < FB; ++mb) {
      sa[mb][0] = P::pack(acc[0][mb], acc[1][mb]);
      sa[mb][1] = P::pack(acc[2][mb], acc[3][mb]);
      if (g == 0) sm.sz[16 * (w * FB + mb) + c16] = acc[4][mb][0];
    }
    __syncthreads();

    // g~ of this wave's features, 16 x rows at a time
    f32x4 szv[FB];
#pragma unroll
    for (int mb = 0; mb < FB; ++mb)
      szv[mb] = *reinterpret_cast<const f32x4 *>(&sm.sz[16 * (w * FB + mb) + 4 * g]);
    // operands of one x block (wide: loaded a block ahead; else the other
    // workgroup of the CU covers their latency)
    struct XOps {
      frag x[2], y[2], pf[2];
      float uy;
    };
    auto load_x = [&](XOps &o, int tb) __attribute__((always_inline)) {
      o.x[0] = load_frag<bf16>(&tl.X[tile_at<kWide>(16 * tb + c16, g)]);
      o.x[1] = load_frag<bf16>(&tl.X[tile_at<kWide>(16 * tb + c16, 4 + g)]);
      o.y[0] = load_frag<bf16>(&tl.Y[tile_at<kWide>(16 * tb + c16, g)]);
      o.y[1] = load_frag<bf16>(&tl.Y[tile_at<kWide>(16 * tb + c16, 4 + g)]);
      if (KEY ? tb < 2 : true) o.pf[0] = sm.PF[tb][0][l];
      if (KEY ? true : tb >= 2) o.pf[1] = sm.PF[tb][1][l];
      o.uy = KEY ? 1.f : tl.uy[16 * tb + c16];
    };
    XOps xo[2];
    if (kWide) load_x(xo[0], 0);
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      if (!kWide)
        load_x(xo[tb & 1], tb);
      else if (tb + 1 < 4)
        load_x(xo[(tb + 1) & 1], tb + 1);
      const XOps &o = xo[tb & 1];
      const bool p0 = KEY ? tb < 2 : true, p1 = KEY ? true : tb >= 2;   // halves not masked
      const frag x0 = o.x[0], x1 = o.x[1], y0 = o.y[0], y1 = o.y[1];
      const float uy = o.uy;
      const frag(&pf)[2] = o.pf;
      f32x4 G[2];
      float dot = 0.f;
#pragma unroll
      for (int mb = 0; mb < FB; ++mb) {
        const f32x4 sd =
            kWide ? bx[mb] : *reinterpret_cast<const f32x4 *>(&sm.bq[kWide ? 0 : 16 * (w * FB + mb) + 4 * g]);
        f32x4 p = P::mma(wf[mb][0], x0, sd);
        p = P::mma(wf[mb][1], x1, p);
        f32x4 t = P::mma(sa[mb][0], y0, KEY ? szv[mb] : zero4);
        t = P::mma(sa[mb][1], y1, t);
        if (p0) t = P::mma(zt[mb][0], pf[0], t);
        if (p1) t = P::mma(zt[mb][1], pf[1], t);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float gj = KEY ? t[j] : fmaf(szv[mb][j], uy, t[j]);
          if constexpr (kDot) dot = fmaf(gj, feature<KN, P>(p[j], sd[j]), dot);
          G[mb][j] = sgn * gj * feature_slope<KN, P>(p[j], sd[j]);
        }
      }
      if constexpr (FB == 2)
        sm.GF[tb][w][l] = P::pack(G[0], G[1]);
      else
        store_half_frag(&sm.GF[tb][w >> 1][l], w & 1, G[0]);
      if constexpr (kDot) {
        dot += __shfl_xor(dot, 16);
        dot += __shfl_xor(dot, 32);
        if (g == 0) sm.dots[w][16 * tb + c16] = dot;
      }
    }
    // fold the chunk's z rows into the aggregate
#pragma unroll
    for (int zs = 0; zs < 2; ++zs) {
#pragma unroll
      for (int nb = 0; nb < 5; ++nb) {
        const frag u = nb < 4 ? sm.UF[nb][zs][l] : tl.EF[zs][g];
#pragma unroll
        for (int mb = 0; mb < FB; ++mb) acc[nb][mb] = P::mma(u, zt[mb][zs], acc[nb][mb]);
      }
    }
    if constexpr (kWide) {   // the next rows into the other buffer
      if (c + 1 < nch) {
        stage_rows(sm.tile[(c + 1) & 1], chunk_t0(c + 1), (c + 1) & 1);
        if (c + 2 < nch) load_rows(chunk_t0(c + 2));
      }
    }
    // the rows the gradient is finished with
    constexpr int NT = kWide ? 1 : 4;   // x blocks per wave
    bf16x4 xr[NT][kWide ? 2 : 1];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int x = 16 * (kWide ? w & 3 : q) + c16;
      const bf16 *xp = &tl.X[kWide ? tile_at<kWide>(x, 4 * (w >> 2) + g) : tile_at<kWide>(x, 2 * w + (g >> 1)) + 4 * (g & 1)];
      xr[q][0] = *reinterpret_cast<const bf16x4 *>(xp);
      if constexpr (kWide) xr[q][1] = *reinterpret_cast<const bf16x4 *>(xp + 4);
    }
    __syncthreads();

    // rows of the result = input columns, lane = x row
    constexpr int NA = kWide ? 2 : 4;
    f32x4 da[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) da[q] = zero4;
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) {
      if constexpr (kWide) {
        const frag gf = sm.GF[w & 3][ks][l];
#pragma unroll
        for (int q = 0; q < 2; ++q) da[q] = P::mma(sm.WT[2 * (w >> 2) + q][ks][l], gf, da[q]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) da[q] = P::mma(wt[ks], sm.GF[q][ks][l], da[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int x = 16 * (kWide ? w & 3 : q) + c16;
      const float ox = sm.ox[c & 1][x];
      float cx = 0.f;   // factor of the row itself: s^2 g~ . xf
      if constexpr (kDot) {
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) d += sm.dots[k][x];
        cx = s * s * d;
      }
      if (t0 + x >= r1) continue;
      bf16 *dst = dX + ((size_t)bh * L + t0 + x) * kD + (kWide ? 32 * (w >> 2) + 8 * g : 16 * w + 4 * g);
      f32x4 v[2];
#pragma unroll
      for (int hh = 0; hh < (kWide ? 2 : 1); ++hh) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[hh][e] = ox * fmaf(cx, (float)xr[q][hh][e], da[kWide ? hh : q][e]);
        if constexpr (ACC) {
          const bf16x4 old = *reinterpret_cast<const bf16x4 *>(dst + 4 * hh);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[hh][e] += (float)old[e];
        }
      }
      if constexpr (kWide)
        store8(dst, v[0], v[1]);
      else
        store4(dst, v[0]);
    }
    if constexpr (!kWide) {
      if (c + 1 < nch) {
        stage_rows(sm.tile[0], chunk_t0(c + 1), (c + 1) & 1);
        if (c + 2 < nch) load_rows(chunk_t0(c + 2));
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------ causal output and dV
template <int M>
struct OutSmem {
  bf16 Z[tile_size<scan_wide(M)>()], X[tile_size<scan_wide(M)>()];   // the chunk's rows (see tile_at)
  float D[2][64];               // D~ of the keys, by chunk parity
  float E[2][64];               // forward: a query's stabiliser or factor (see below)
  bf16x8 QA[4][M / 32][64];     // features of the z rows: lane = z, k = features
  bf16x8 KF[4][M / 32][64];     // features of the x rows: lane = x, k = features
  bf16x8 RB[4][M / 32][64];     // a^T without the chunk: lane = value column, k = features
  bf16x8 RE[M / 32][4];         // its last column, one fragment per lane group
  bf16x8 UF[4][2][64];          // (w u)^T: lane = value column, k = z rows
  bf16x8 UE[2][4];              // u~'s last column, one fragment per lane group
  f32x4 red[scan_wide(M) ? 4 : 1][scan_wide(M) ? 5 : 1][64];   // the second half's partial sums
};

// The product of the x rows' features with the aggregate, plus the chunk's own part:
//   B_x = a^T xf_x + sum over z rows of u~_z (zf_z . xf_x),  u~ = w [u, 1 or u_d],
// with z <= x (FWD: x the queries, z and u the keys and values, chunks in order) or
// z >= x (dV: x the keys, z and u the queries and output gradients, chunks from the
// last).
//   FWD: out_x = B_x[:d] / (B_x[d] + eps) (or the numerator times D_Q sqrt(2/M)), and
//        SAVE: rowv_x, the row's 1 / (D-hat + eps) in units of the unscaled features
//   dV:  dV_x = D~_x B_x[:d]
// Each wave forms its features of both row sets and publishes them and its slice
// of the aggregate (accumulators: rows = features, lanes = value columns) in the
// layouts the products over all features read; then wave (jb, half) takes x block
// jb: the masked zf . xf of one 32-row half, its product with u~, and half of the
// feature steps of a^T xf.
template <typename To, int M, int KN, bool FWD, bool RN, bool SAVE>
__global__ __launch_bounds__(64 * scan_waves(M), scan_wide(M) ? 1 : 2) void k_out_scan(
    const bf16 *__restrict__ X, const bf16 *__restrict__ Z, const bf16 *__restrict__ U,
    const float2 *__restrict__ aux, const bf16x8 *__restrict__ wfr,
    const float *__restrict__ bqg, const float *__restrict__ states, To *__restrict__ out,
    float *__restrict__ rowv, int H, int L, int seg_len, int nseg, float s, float eps, float cM) {
  constexpr int NW = scan_waves(M);
  constexpr int FB = M / 16 / NW;
  constexpr int NS = M / 32;
  constexpr int RPT = 8 / NW;
  constexpr bool kWide = scan_wide(M);
  using P = Mma<bf16>;
  using frag = bf16x8;
  __shared__ OutSmem<M> sm;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int bh = item / nseg;
  const int seg = item - bh * nseg;
  const int h = bh % H;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63;
  const int g = l >> 4;
  const int c16 = l & 15;
  const float s2half = 0.5f * s * s;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  const int r0 = seg * seg_len;
  const int r1 = min(L, r0 + seg_len);
  if (r0 >= r1) return;
  const int nch = (r1 - r0 + 63) / 64;
  const bf16 *Xh = X + (size_t)bh * L * kD;
  const bf16 *Zh = Z + (size_t)bh * L * kD;
  const bf16 *Uh = U + (size_t)bh * L * kD;
  const float2 *auh = FWD ? nullptr : aux + (size_t)bh * L;
  const int jb = w & 3;

  // the next chunk's rows: x and z to be staged, and the u rows this wave
  // transposes (row block w % 4, columns 32 (w / 4 + k) ..)
  struct Regs {
    frag z[RPT], x[RPT], u[RPT];
    float2 a[FWD ? 1 : 4];   // dV: row weights of z rows 16 (w % 4) + 4 g + j
  };
  Regs rg;
  auto load_rows = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int t = t0 + (tid >> 3) + 8 * NW * k;
      const size_t off = (size_t)t * kD + 8 * (tid & 7);
      rg.z[k] = rg.x[k] = rg.u[k] = P::splat(0.f);
      if (t < r1) {
        rg.z[k] = load_frag<bf16>(Zh + off);
        rg.x[k] = load_frag<bf16>(Xh + off);
      }
      const int tu = t0 + 16 * (w & 3) + c16;
      if (tu < r1) rg.u[k] = load_frag<bf16>(Uh + (size_t)tu * kD + 32 * ((w >> 2) + k) + 8 * g);
    }
    if constexpr (!FWD) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = t0 + 16 * (w & 3) + 4 * g + j;
        rg.a[j] = t < r1 ? auh[t] : make_float2(0.f, 0.f);
      }
    }
  };
  auto stage_rows = [&](int t0, int par) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int r = (tid >> 3) + 8 * NW * k;
      store_frag<bf16>(&sm.Z[tile_at<kWide>(r, tid & 7)], rg.z[k]);
      store_frag<bf16>(&sm.X[tile_at<kWide>(r, tid & 7)], rg.x[k]);
      const frag &kr = FWD ? rg.z[k] : rg.x[k];
      float D = 1.f;
      if constexpr (KN == kCos) D = cM * expf(s2half * oct_sum_f32(dot8(kr, kr)));
      if ((tid & 7) == 0) sm.D[par][r] = !FWD || t0 + r < r1 ? D : 0.f;
      if (FWD && KN == kCos && (!RN || eps != 0.f)) {
        // D_Q sqrt(2/M), which the features omit, or the stabiliser divided by it
        const float dq = cM * expf(s2half * oct_sum_f32(dot8(rg.x[k], rg.x[k])));
        if ((tid & 7) == 0) sm.E[par][r] = RN ? eps / dq : dq;
      }
    }
  };
  auto chunk_t0 = [&](int c) { return r0 + 64 * (FWD ? c : nch - 1 - c); };
  load_rows(chunk_t0(0));

  frag wf[FB][2];
  f32x4 bx[FB];
  float bz[FB];
#pragma unroll
  for (int mb = 0; mb < FB; ++mb) {
    const int mbg = w * FB + mb;
    const frag *wp = wfr + ((size_t)h * (M / 16) + mbg) * 2 * 64 + l;
    wf[mb][0] = wp[0];
    wf[mb][1] = wp[64];
    const float *bp = bqg + (size_t)h * M + 16 * mbg;
    bx[mb] = *reinterpret_cast<const f32x4 *>(bp + 4 * g);
    bz[mb] = bp[c16];
  }
  // The aggregate: rows = features 16 (w FB + mb) + 4 g + j, lane = value column perm_col(nb, c16)
  // (block 4: the last column, replicated)
  f32x4 acc[FB][5];
  {
    const float *R = states + ((size_t)bh * nseg + seg) * M * 65;
#pragma unroll
    for (int mb = 0; mb < FB; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float *row = R + (size_t)(16 * (w * FB + mb) + 4 * g + j) * 65;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[mb][nb][j] = row[perm_col(nb, c16)];
        acc[mb][4][j] = row[64];
      }
  }
  stage_rows(chunk_t0(0), 0);
  __syncthreads();

  f32x4 va[5];     // this wave's share of the bracket: value blocks, last column
  // after the barrier that publishes the second half's shares: sum, store
  auto finish = [&](int c) __attribute__((always_inline)) {
    if (kWide && w >= 4) return;
    const int j = chunk_t0(c) + 16 * jb + c16;
    if constexpr (kWide) {
#pragma unroll
      for (int nb = 0; nb < 5; ++nb) va[nb] += sm.red[jb][nb][l];
    }
    if constexpr (FWD) {
      float e = RN ? (KN == kCos ? 0.f : eps) : 1.f;
      if (KN == kCos && (!RN || eps != 0.f)) e = sm.E[c & 1][16 * jb + c16];
      const float inv = RN ? 1.0f / (va[4][0] + e) : e;
      if (j < r1) {
#pragma unroll
        for (int pp = 0; pp < 2; ++pp)
          store8(out + ((size_t)bh * L + j) * kD + 32 * pp + 8 * g, va[2 * pp] * inv,
                 va[2 * pp + 1] * inv);
        if (SAVE && g == 0) rowv[(size_t)bh * L + j] = inv;
      }
      return;
    }
    const float D = sm.D[c & 1][16 * jb + c16];
    if (j < r1) {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp)
        store8(out + ((size_t)bh * L + j) * kD + 32 * pp + 8 * g, va[2 * pp] * D,
               va[2 * pp + 1] * D);
    }
  };

  for (int c = 0; c < nch; ++c) {
    const int t0 = chunk_t0(c);
    // (w u)^T and u~'s last column
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int tb = w & 3;
      const int kh = (w >> 2) + k;
      f32x4 wz, ez;
      if constexpr (FWD) {
        wz = ez = *reinterpret_cast<const f32x4 *>(&sm.D[c & 1][16 * tb + 4 * g]);
      } else {
        wz = f32x4{rg.a[0].x, rg.a[1].x, rg.a[2].x, rg.a[3].x};
        ez = f32x4{rg.a[0].y, rg.a[1].y, rg.a[2].y, rg.a[3].y};
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const f32x4 t = P::mma(rg.u[k], scan_select(half), zero4);
        store_half_frag(&sm.UF[2 * kh + half][tb >> 1][l], tb & 1, t * wz);
      }
      if (kh == 0 && c16 == 0)
        store_half_frag(&sm.UE[tb >> 1][g], tb & 1, ez);
    }
    // the aggregate without the chunk's rows
#pragma unroll
    for (int nb = 0; nb < 5; ++nb) {
      if constexpr (FB == 2) {
        const frag f = P::pack(acc[0][nb], acc[1][nb]);
        if (nb < 4)
          sm.RB[nb][w][l] = f;
        else if (c16 == 0)
          sm.RE[w][g] = f;
      } else {
        if (nb < 4)
          store_half_frag(&sm.RB[nb][w >> 1][l], w & 1, acc[0][nb]);
        else if (c16 == 0)
          store_half_frag(&sm.RE[w >> 1][g], w & 1, acc[0][nb]);
      }
    }
    // features of the x rows, lane = x
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) {
      const frag x0 = load_frag<bf16>(&sm.X[tile_at<kWide>(16 * tb + c16, g)]);
      const frag x1 = load_frag<bf16>(&sm.X[tile_at<kWide>(16 * tb + c16, 4 + g)]);
      f32x4 f[2];
#pragma unroll
      for (int mb = 0; mb < FB; ++mb) {
        f32x4 p = P::mma(wf[mb][0], x0, bx[mb]);
        p = P::mma(wf[mb][1], x1, p);
#pragma unroll
        for (int j = 0; j < 4; ++j) f[mb][j] = feature<KN, P>(p[j], bx[mb][j]);
      }
      if constexpr (FB == 2)
        sm.KF[tb][w][l] = P::pack(f[0], f[1]);
      else
        store_half_frag(&sm.KF[tb][w >> 1][l], w & 1, f[0]);
    }
    // features of the z rows as A operand of the fold (row = feature, k = z rows), and
    // transposed on the matrix cores (exact) with lane = z
    frag zt[FB][2];
#pragma unroll
    for (int zs = 0; zs < 2; ++zs) {
      f32x4 f[FB][2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const frag z0 = load_frag<bf16>(&sm.Z[tile_at<kWide>(32 * zs + 16 * q + c16, g)]);
        const frag z1 = load_frag<bf16>(&sm.Z[tile_at<kWide>(32 * zs + 16 * q + c16, 4 + g)]);
#pragma unroll
        for (int mb = 0; mb < FB; ++mb) {
          f32x4 p = P::mma(z0, wf[mb][0], f32x4{bz[mb], bz[mb], bz[mb], bz[mb]});
          p = P::mma(z1, wf[mb][1], p);
#pragma unroll
          for (int j = 0; j < 4; ++j) f[mb][q][j] = feature<KN, P>(p[j], bz[mb]);
        }
      }
#pragma unroll
      for (int mb = 0; mb < FB; ++mb) zt[mb][zs] = P::pack(f[mb][0], f[mb][1]);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        f32x4 t[2];
#pragma unroll
        for (int mb = 0; mb < FB; ++mb) t[mb] = P::mma(zt[mb][zs], chained_select_frag<bf16>(q), zero4);
        if constexpr (FB == 2)
          sm.QA[2 * zs + q][w][l] = P::pack(t[0], t[1]);
        else
          store_half_frag(&sm.QA[2 * zs + q][w >> 1][l], w & 1, t[0]);
      }
    }
    if (c > 0) finish(c - 1);
    __syncthreads();

    if (c + 1 < nch) load_rows(chunk_t0(c + 1));
    // fold the chunk's z rows into the aggregate
#pragma unroll
    for (int zs = 0; zs < 2; ++zs)
#pragma unroll
      for (int nb = 0; nb < 5; ++nb) {
        const frag u = nb < 4 ? sm.UF[nb][zs][l] : sm.UE[zs][g];
#pragma unroll
        for (int mb = 0; mb < FB; ++mb) acc[mb][nb] = P::mma(zt[mb][zs], u, acc[mb][nb]);
      }
    // x block jb against one half of the z rows (wide) or both
    frag kf[NS];
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) kf[ks] = sm.KF[jb][ks][l];
#pragma unroll
    for (int nb = 0; nb < 5; ++nb) va[nb] = zero4;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int zs = (w >> 2) + k;
      if (FWD ? 2 * zs > jb : 2 * zs + 1 < jb) continue;   // wholly masked
      f32x4 p4[2] = {zero4, zero4};
#pragma unroll
      for (int ks = 0; ks < NS; ++ks)
#pragma unroll
        for (int q = 0; q < 2; ++q) p4[q] = P::mma(sm.QA[2 * zs + q][ks][l], kf[ks], p4[q]);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
        {
          const int z = 16 * (2 * zs + q) + 4 * g + e, x = 16 * jb + c16;
          p4[q][e] = (FWD ? z <= x : z >= x) ? p4[q][e] : 0.f;
        }
      const frag pb = P::pack(p4[0], p4[1]);
      // The intra-chunk weights as two bf16 terms. One rounding of the whole sum over
      // the features is a larger error than k_causal_fs's roundings of its four partial
      // sums, and dV reads the row scales that the output's weights gave: B2 H8 L2048
      // M256, relative 2-norms, output 2.5e-3 against 2.7e-3 with one term
      // (k_causal_fs: 2.6e-3). The extra products take 1.7 us of the output scan of
      // B4 H8 L8192 M256 (66 us when they were added).
      f32x4 lo[2];
      float top = 0.f;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          lo[q][e] = p4[q][e] - (float)pb[4 * q + e];
          top = fmaxf(top, fabsf(p4[q][e]));
        }
      // A weight past bf16's range is +-Inf in the first term; the second is then 0 (the
      // difference would be NaN and make the row's Inf one). Tested for the wave as
      // a whole: with a choice per weight the call of B1 H16 L65536 M256 took 353 us, this
      // way 342.
      if (__any(top >= 0x1.ffp127f)) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (fabsf(p4[q][e]) >= 0x1.ffp127f) lo[q][e] = 0.f;
      }
      const frag pl = P::pack(lo[0], lo[1]);
#pragma unroll
      for (int nb = 0; nb < 5; ++nb) {
        const frag u = nb < 4 ? sm.UF[nb][zs][l] : sm.UE[zs][g];
        va[nb] = P::mma(u, pb, va[nb]);
        va[nb] = P::mma(u, pl, va[nb]);
      }
    }
    // a^T xf (wide: this half's feature steps)
    constexpr int kSteps = kWide ? NS / 2 : NS;
    const int kb = kWide ? (w >> 2) * kSteps : 0;
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
      const frag k1 = kWide ? sm.KF[jb][kb + k][l] : kf[k];
#pragma unroll
      for (int nb = 0; nb < 5; ++nb)
        va[nb] = P::mma(nb < 4 ? sm.RB[nb][kb + k][l] : sm.RE[kb + k][g], k1, va[nb]);
    }
    if constexpr (kWide) {
      if (w >= 4) {
#pragma unroll
        for (int nb = 0; nb < 5; ++nb) sm.red[jb][nb][l] = va[nb];
      }
    }
    if (c + 1 < nch) stage_rows(chunk_t0(c + 1), (c + 1) & 1);
    __syncthreads();
  }
  finish(nch - 1);
}

// ------------------------------------------------------------ launchers
#define FAVOR_SCAN_DISPATCH_M(M_, ...)                               \
  switch (M_) {                                                     \
    case 64: { constexpr int MM = 64; __VA_ARGS__; } break;          \
    case 128: { constexpr int MM = 128; __VA_ARGS__; } break;        \
    case 256: { constexpr int MM = 256; __VA_ARGS__; } break;        \
    default: return hipErrorInvalidValue;                           \
  }

template <int KN, bool RN, bool KEY, bool ACC>
static hipError_t row_scan(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  const float wts = sh.kernel == 1 ? sh.s / sqrtf((float)sh.Mr) : sh.s;
  FAVOR_SCAN_DISPATCH_M(
      sh.M, hipLaunchKernelGGL((k_bwd_row_scan<MM, KN, RN, KEY, ACC>), dim3(a.nseg * sh.BH),
                               dim3(64 * scan_waves(MM)), 0, st, (const bf16 *)a.Q,
                               (const bf16 *)a.K, (const bf16 *)a.V, (const bf16 *)a.dout,
                               (const bf16 *)a.out, a.rsave, (const bf16x8 *)a.wfr, a.bq, a.W,
                               a.state, (bf16 *)(KEY ? a.dK : a.dQ), a.aux, sh.H, sh.L, a.seg_len,
                               a.nseg, sh.s, sh.Mr, feature_norm(sh), wts));
  return hipGetLastError();
}

template <int KN, bool RN>
static hipError_t dq_scan(const Shape &sh, const BwdArgs &a, bool accumulate, hipStream_t st) {
  return accumulate ? row_scan<KN, RN, false, true>(sh, a, st)
                    : row_scan<KN, RN, false, false>(sh, a, st);
}

hipError_t launch_bwd_dq_scan(const Shape &sh, const BwdArgs &a, bool accumulate,
                              hipStream_t st) {
  if (sh.kernel == 1)
    return sh.renorm ? dq_scan<kRelu, true>(sh, a, accumulate, st)
                     : dq_scan<kRelu, false>(sh, a, accumulate, st);
  return sh.renorm ? dq_scan<kCos, true>(sh, a, accumulate, st)
                   : dq_scan<kCos, false>(sh, a, accumulate, st);
}

template <int KN>
static hipError_t dv_scan(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  FAVOR_SCAN_DISPATCH_M(
      sh.M, hipLaunchKernelGGL((k_out_scan<bf16, MM, KN, false, true, false>),
                               dim3(a.nseg * sh.BH), dim3(64 * scan_waves(MM)), 0, st,
                               (const bf16 *)a.K, (const bf16 *)a.Q, (const bf16 *)a.dout,
                               a.aux, (const bf16x8 *)a.wfr, a.bq, a.state,
                               (bf16 *)a.dV, (float *)nullptr, sh.H, sh.L, a.seg_len, a.nseg, sh.s, 0.f,
                               feature_norm(sh)));
  return hipGetLastError();
}

hipError_t launch_bwd_dkv_scan(const Shape &sh, const BwdArgs &a, hipStream_t st) {
  const hipError_t e = sh.kernel == 1 ? dv_scan<kRelu>(sh, a, st) : dv_scan<kCos>(sh, a, st);
  if (e != hipSuccess) return e;
  return sh.kernel == 1 ? row_scan<kRelu, true, true, false>(sh, a, st)
                        : row_scan<kCos, true, true, false>(sh, a, st);
}

// The forward scan from the segments' prefix states.
template <typename To, int KN, bool RN, bool SAVE>
static hipError_t fwd_scan(const Shape &sh, const void *Q, const void *K, const void *V,
                           const void *wfr, const float *bq, const float *prefix, void *o,
                           float *rsave, int seg_len, int nseg, hipStream_t st) {
  FAVOR_SCAN_DISPATCH_M(
      sh.M, hipLaunchKernelGGL((k_out_scan<To, MM, KN, true, RN, SAVE>), dim3(nseg * sh.BH),
                               dim3(64 * scan_waves(MM)), 0, st, (const bf16 *)Q,
                               (const bf16 *)K, (const bf16 *)V,
                               (const float2 *)nullptr, (const bf16x8 *)wfr, bq, prefix, (To *)o,
                               rsave, sh.H, sh.L, seg_len, nseg, sh.s, sh.eps, feature_norm(sh)));
  return hipGetLastError();
}

template <typename To, bool SAVE>
static hipError_t fwd_scan_kind(const Shape &sh, const void *Q, const void *K, const void *V,
                                const void *wfr, const float *bq, const float *prefix, void *o,
                                float *rsave, int seg_len, int nseg, hipStream_t st) {
  if (!sh.renorm) {
    if constexpr (SAVE) return hipErrorInvalidValue;
    else
      return sh.kernel == 1
                 ? fwd_scan<To, kRelu, false, false>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st)
                 : fwd_scan<To, kCos, false, false>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st);
  }
  return sh.kernel == 1
             ? fwd_scan<To, kRelu, true, SAVE>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st)
             : fwd_scan<To, kCos, true, SAVE>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st);
}

hipError_t launch_out_scan(const Shape &sh, Dt out, const void *Q, const void *K, const void *V,
                           const void *wfr, const float *bq, const float *prefix, void *o,
                           float *rsave, int seg_len, int nseg, hipStream_t st) {
  if (rsave)
    return fwd_scan_kind<bf16, true>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st);
  return out == Dt::BF16
             ? fwd_scan_kind<bf16, false>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st)
             : fwd_scan_kind<float, false>(sh, Q, K, V, wfr, bq, prefix, o, rsave, seg_len, nseg, st);
}

}  // namespace favor
