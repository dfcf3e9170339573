// Backward pass of non-causal attention on the bf16 path (d = dv = 64, M = 256): gradients of sum(Y * dY) with
// respect to Q, K, V, theta and omega held fixed (chain rule on Section 2.2's attention equation with K_hat = P S^T).
//
// With V1 = [V 1], T = S^T V1 (the forward state, 256 x 65) and Yhat = P T (numerators and normaliser):
//   G1_i = [dY_i / den_i, -(dY_i . Y_i) / den_i]      (65 numbers per query, stored as rows of 80 bf16)
//   R    = P^T G1                                     (256 x 65, the query-side twin of the state)
//   dV   = (S R)[:, :64]
//   dP   = G1 T^T,  dE1 = P * dP,  dQ = dE1 (d E1 / d q)
//   dS   = V1 R^T,  dE2 = S * dS,  dK = dE2 (d E2 / d k)
// Exponents are in the log2 domain with W~ carrying log2(e) and qk_scale, so d E / d (raw row) = ln2 W~ plus, on
// the key side, the derivative of the row term y^T C2 y (y = qk_scale k): qk_scale^2 (C2 + C2^T) k times the row
// sum of dE2.  On the query side that row sum vanishes identically (Y does not depend on a per-row factor of P).
// The exponent shifts and the placement of the bias on the query side cancel in every product above, so the
// kernels work on the same shifted features as the forward pass.
//
// Kernels (one attention_backward call = forward state and reduction, then):
//   k_bwd_rows<0>    queries: Yhat = P T, normalise, G1 rows -> gh; dP = G1 T^T, dE1, dQ
//   k_bwd_rstate     queries: segment sums of P^T G1                                 -> Rpart (k_fast_total sums them)
//   k_bwd_rows<1>    keys:    dV = S R; dS, dE2, dK
//   k_bwd_whole      many or short sequences: all of the above (and the forward state) for one (b,h) per workgroup, on
//                    loops with a wave's 64 features of every operand in registers
#include "fast_bwd.h"
#include "fast_rows.h"
#include "fast_state.h"

namespace fs {

using namespace fast;

namespace bwd {

// ---------------------------------------------------------------------------------------------------------------
// Loops of k_bwd_whole.  A wave has 64 of the features for all rows of a chunk; the waves' partial tiles are summed through LDS.
// MODE 1 (queries): rows of G1.  MODE 2 (keys): dV = S R.
// ---------------------------------------------------------------------------------------------------------------
// Rows [row_beg, row_end) of one (b,h) against the state image tb (state^T as A operand: row v = 16 vt + c, k <->
// features 64w + 32 mb + 16 (e/4) + 4g + e%4); cs: the key shift of the sequence (MODE 2).  Returns the number of
// rows this wave finished with a zero normaliser (MODE 1).
template <int MODE>
__device__ __forceinline__ int apply_rows_b(const BwdArgs& ba, SmemApply& sm, int bh, const bf16x8 (&tb)[NVT][2], float cs,
                                            int row_beg, int row_end) {
  const FastArgs& a = ba.f;
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
  const int pg = group_of(a.pgroups, b, h, a.H);
  constexpr int side = MODE == 1 ? 0 : 1;
  const TensorDev& X = MODE == 1 ? a.Q : a.K;
  const float wmax = max256(a.wnorm + ((size_t)pg * 2 + side) * M), amax = max256(a.bias + ((size_t)pg * 2) * M);
  const uint16_t* Xb = (const uint16_t*)X.ptr + b * X.sb + h * X.sh;
  const float* th = a.theta + (size_t)group_of(a.groups, b, h, a.H) * (FS_THETA_HEADER_ + (size_t)D + 4 * (size_t)D * D);
  const bool isoC = ((int)th[2]) & 1;

  WSlice wx;
  load_wslice(wx, a.Wbf + ((size_t)pg * 2 + side) * M * D);
  QBias qb;
  load_qbias(qb, a.bias + ((size_t)pg * 2) * M, amax);
  int nzero = 0;                   // (MODE 1) rows this wave finished with a zero normaliser

  // staged rows -> LDS with what is added to their exponents: - row_shift (queries), row term - key shift (keys)
  auto stage = [&](const RowRegs& r, int buf, int row0) {
    float n2[2];
    store_rows_s(r, sm.q[buf], n2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = threadIdx.x + NT * i, row = q >> 3;
      if ((q & 7) == 0) {
        float add;
        if (MODE == 1) add = -row_shift(n2[i], wmax);
        else {
          float rt = -0.5f * kLog2e * a.scale * a.scale * n2[i];
          if (!isoC) rt = row0 + row < row_end ? a.rk[(size_t)bh * a.L + row0 + row] : 0.f;
          add = rt - cs;
        }
        sm.qadd[buf][row] = add;
      }
    }
  };

  RowRegs xr;
  load_rows_g(xr, Xb, X.sl, row_beg, row_end);
  stage(xr, 0, row_beg);
  __syncthreads();
  int buf = 0;
  for (int row0 = row_beg; row0 < row_end; row0 += TC, buf ^= 1) {
    const bool more = row0 + TC < row_end;
    if (more) load_rows_g(xr, Xb, X.sl, row0 + TC, row_end);
    // (MODE 1) this wave's rows of dY are requested before the chunk's feature tiles and used after them
    f32x4 gpre[4] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    if (MODE == 1 && row0 + 16 * w + c < row_end) {
      const long long go = b * ba.dY.sb + h * ba.dY.sh + (long long)(row0 + 16 * w + c) * ba.dY.sl + 4 * g;
      if (ba.dY.dtype == 1) {
#pragma unroll
        for (int vt = 0; vt < 4; ++vt) gpre[vt] = __builtin_convertvector(*(const bf16x4*)((const uint16_t*)ba.dY.ptr + go + 16 * vt), f32x4);
      } else {
#pragma unroll
        for (int vt = 0; vt < 4; ++vt) gpre[vt] = *(const f32x4*)((const float*)ba.dY.ptr + go + 16 * vt);
      }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      bf16x8 p[2];
      feature_tile<MODE == 1>(wx, &qb, sm.q[buf], it, sm.qadd[buf][16 * it + c], p);
      f32x4 y[NVT];
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) {
        y[vt] = mfma(tb[vt][0], p[0], f32x4{0.f, 0.f, 0.f, 0.f});
        y[vt] = mfma(tb[vt][1], p[1], y[vt]);
      }
      exchange_put_bf16(sm, y, it, w, lane);
    }
    __syncthreads();
    {
      f32x4 fs[4] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
      finish_tiles(fs, sm, w, 0, lane);
      finish_tiles(fs, sm, w, 2, lane);
      const int token = row0 + 16 * w + c;
      const bool valid = token < row_end;
      if (MODE == 1) {
        unsigned zt;
        const float inv = finish_norm(fs, sm, w, lane, &zt);      // fs = Y rows now
        nzero += count_zero_tokens(zt, w, row_end - row0);
        f32x4 gv[4];
        float dot = 0.f;
#pragma unroll
        for (int vt = 0; vt < 4; ++vt) {
          gv[vt] = gpre[vt];
#pragma unroll
          for (int r = 0; r < 4; ++r) dot += gv[vt][r] * fs[vt][r];
        }
        dot += __shfl_xor(dot, 16);
        dot += __shfl_xor(dot, 32);
        if (valid) {
          uint16_t* go = ba.gh + ((size_t)bh * ba.Lq + token) * DVP + 4 * g;
#pragma unroll
          for (int vt = 0; vt < 4; ++vt) *(bf16x4*)(go + 16 * vt) = __builtin_convertvector(gv[vt] * inv, bf16x4);
          const f32x4 last = {g == 0 ? -dot * inv : 0.f, 0.f, 0.f, 0.f};
          *(bf16x4*)(go + D) = __builtin_convertvector(last, bf16x4);
        }
      } else if (valid) {
        if (ba.dV.dtype == 1) {
          uint16_t* yp = (uint16_t*)ba.dV.ptr + b * ba.dV.sb + h * ba.dV.sh + (long long)token * ba.dV.sl + 4 * g;
#pragma unroll
          for (int vt = 0; vt < 4; ++vt) *(bf16x4*)(yp + 16 * vt) = __builtin_convertvector(fs[vt], bf16x4);
        } else {
          float* yp = (float*)ba.dV.ptr + b * ba.dV.sb + h * ba.dV.sh + (long long)token * ba.dV.sl + 4 * g;
#pragma unroll
          for (int vt = 0; vt < 4; ++vt) *(f32x4*)(yp + 16 * vt) = fs[vt];
        }
      }
    }
    if (more) stage(xr, buf ^ 1, row0 + TC);
    __syncthreads();
  }
  return nzero;
}

// ---------------------------------------------------------------------------------------------------------------
// Segment sums of P^T G1 (state_rows on the query side: features with their per-row shifts, "values" = rows of G1).
// k_bwd_rstate: rows of a state per slot for the causal kernels, or (IMG) accumulator images for slots of few chunks.  grid
// (rslots, B*H), block 256.
// k_bwd_rstate2: two groups of waves per slot, accumulator images (k_fast_total sums them).  grid (rslots, B*H), block 512.
// ---------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ const FastArgs rstate_args(const BwdArgs& ba) {
  FastArgs a = ba.f;
  a.V = TensorDev{ba.gh, 1, (long long)a.H * ba.Lq * DVP, (long long)ba.Lq * DVP, DVP};
  return a;
}
template <bool IMG>
__global__ void __launch_bounds__(NT, 2) k_bwd_rstate(BwdArgs ba) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int slot = blockIdx.x, bh = blockIdx.y;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
  const int row_beg = slot * ba.rows_per_rslot, row_end = min(ba.Lq, row_beg + ba.rows_per_rslot);
  f32x4 R[4][NVT];
  float dk;
  state_rows<STATE_QUERIES>(rstate_args(ba), *reinterpret_cast<SmemState*>(smem_raw), bh, row_beg, row_end, (row_end - row_beg + TC - 1) / TC, R, dk);
  float* out = ba.Rpart + ((size_t)bh * ba.rslots + slot) * M * DVP;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) {
      if (IMG) {
        *(f32x4*)(out + (size_t)((w * 4 + mt) * NVT + vt) * 256 + 4 * lane) = R[mt][vt];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(size_t)(64 * w + 16 * mt + 4 * g + r) * DVP + 16 * vt + c] = R[mt][vt][r];
      }
    }
  if (threadIdx.x == 0) ba.rcpart[(size_t)bh * ba.rslots + slot] = 0.f;
}
__global__ void __launch_bounds__(2 * NT) k_bwd_rstate2(BwdArgs ba) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int slot = blockIdx.x, bh = blockIdx.y, row_beg = slot * ba.rows_per_rslot;
  state_two_groups<STATE_QUERIES>(rstate_args(ba), smem_raw, bh, row_beg, min(ba.Lq, row_beg + ba.rows_per_rslot), true,
                                  ba.Rpart + ((size_t)bh * ba.rslots + slot) * M * DVP, ba.rcpart + (size_t)bh * ba.rslots + slot);
}

// ---------------------------------------------------------------------------------------------------------------
// Gradient rows.  KEY = 0: dQ from (queries, left rows = G1, state = T).  KEY = 1: dK from (keys, left rows = [V 1],
// state = R).  Per 16-token tile: F (feature tile), dF = state x (left rows)^T in the same accumulator layout
// (rows = features, column = token), dE = F * dF, gradient tile = W~^T (A operand: rows = coordinates, k <->
// features; a row of ones appended: row sum of dE) x dE.  The four waves' partial gradient tiles are summed through
// LDS on the MFMA pipe.  (Another loop of k_bwd_whole.)
// ---------------------------------------------------------------------------------------------------------------
struct SmemGrad {
  __attribute__((aligned(16))) uint16_t q[1][TC][LDR];            // rows of the chunk (one buffer)
  float qadd[TC];
  __attribute__((aligned(16))) uint16_t lam[TC][LDL];             // left rows: G1 (queries) or [V 1 0..] (keys)
  __attribute__((aligned(16))) uint16_t xch[NW][NW][16][LDXB];
  // C2 + C2^T as A operands of the keys' row term when C2 is dense: [16-row tile][k-step][lane] (rows = gradient columns)
  __attribute__((aligned(16))) uint16_t csym[4][KS][64][8];
};

// Rows [row_beg, row_end) of one (b,h); sa: the state as A operand of dF (row f = 64w + 16mt + c, k = 32kk + 8g + e
// <-> column v, zero from 80 on); cs: the key shift of the sequence (KEY).
template <int KEY>
__device__ __forceinline__ void grad_rows(const BwdArgs& ba, SmemGrad& sm, int bh, const bf16x8 (&sa)[4][3], float cs,
                                          int row_beg, int row_end) {
  const FastArgs& a = ba.f;
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
  const int pg = group_of(a.pgroups, b, h, a.H);
  const TensorDev& X = KEY ? a.K : a.Q;
  const TensorDev& G = KEY ? ba.dK : ba.dQ;
  const float wmax = max256(a.wnorm + ((size_t)pg * 2 + KEY) * M), amax = max256(a.bias + ((size_t)pg * 2) * M);
  const uint16_t* Xb = (const uint16_t*)X.ptr + b * X.sb + h * X.sh;
  const uint16_t* Vb = (const uint16_t*)a.V.ptr + b * a.V.sb + h * a.V.sh;
  const uint16_t* Gb = ba.gh + (size_t)bh * ba.Lq * DVP;
  const float* th = a.theta + (size_t)group_of(a.groups, b, h, a.H) * (FS_THETA_HEADER_ + (size_t)D + 4 * (size_t)D * D);
  const bool isoC = ((int)th[2]) & 1;
  const float* C2 = th + FS_THETA_HEADER_ + D + 3 * (size_t)D * D;
  const uint16_t* Wg = a.Wbf + ((size_t)pg * 2 + KEY) * M * D;

  WSlice wx;
  load_wslice(wx, Wg);
  QBias qb;
  load_qbias(qb, a.bias + ((size_t)pg * 2) * M, amax);
  // W~^T as A operand of the gradient tile: row = coordinate 16dt + c, k <-> feature 64w + 32blk + 16(e/4) + 4g + e%4;
  // tile dt = 4 has ones in its row 0 (coordinate "64" = the row sum of dE) and zeros elsewhere
  bf16x8 wt[NVT][2];
#pragma unroll
  for (int dt = 0; dt < NVT; ++dt)
#pragma unroll
    for (int bk = 0; bk < 2; ++bk) {
      u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int f = 64 * w + 32 * bk + 16 * (e >> 2) + 4 * g + (e & 3);
        uint32_t bits;
        if (dt < 4) bits = Wg[(size_t)f * D + 16 * dt + c];
        else bits = c == 0 ? 0x3f80u : 0u;
        v[e >> 1] |= bits << (16 * (e & 1));
      }
      wt[dt][bk] = __builtin_bit_cast(bf16x8, v);
    }

  if (KEY && !isoC) {
    for (int piece = threadIdx.x; piece < 4 * KS * 64; piece += NT) {
      const int l = piece & 63, ks = (piece >> 6) % KS, dt = piece / (64 * KS);
      const int dd = 16 * dt + (l & 15), e0 = 32 * ks + 8 * (l >> 4);
      f32x8 cv;
#pragma unroll
      for (int e = 0; e < 8; ++e) cv[e] = C2[dd * D + e0 + e] + C2[(e0 + e) * D + dd];
      *(bf16x8*)(&sm.csym[dt][ks][l][0]) = __builtin_convertvector(cv, bf16x8);
    }
  }
  // zero padding of the left-rows tile (columns the staging never writes)
  for (int idx = threadIdx.x; idx < TC * (KL - (KEY ? D : DVP)); idx += NT) {
    const int n = KL - (KEY ? D : DVP);
    sm.lam[idx / n][(KEY ? D : DVP) + idx % n] = 0;
  }

  auto load_left = [&](RowRegs3& r, int row0) {
    if (KEY) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int q = threadIdx.x + NT * i, row = q >> 3, pc = q & 7;
        r.p[i] = u32x4{0u, 0u, 0u, 0u};
        if (row0 + row < row_end) r.p[i] = *(const u32x4*)(Vb + (long long)(row0 + row) * a.V.sl + pc * 8);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int q = threadIdx.x + NT * i, row = q / 10, pc = q - 10 * row;
        r.p[i] = u32x4{0u, 0u, 0u, 0u};
        if (q < TC * 10 && row0 + row < row_end) r.p[i] = *(const u32x4*)(Gb + (size_t)(row0 + row) * DVP + pc * 8);
      }
    }
  };
  auto stage = [&](const RowRegs& xr, const RowRegs3& lr, int row0) {
    float n2[2];
    store_rows_s(xr, sm.q[0], n2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = threadIdx.x + NT * i, row = q >> 3;
      if ((q & 7) == 0) {
        float add;
        if (!KEY) add = -row_shift(n2[i], wmax);
        else {
          float rt = -0.5f * kLog2e * a.scale * a.scale * n2[i];
          if (!isoC) rt = row0 + row < row_end ? a.rk[(size_t)bh * a.L + row0 + row] : 0.f;
          add = rt - cs;
        }
        sm.qadd[row] = add;
      }
    }
    if (KEY) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int q = threadIdx.x + NT * i, row = q >> 3, pc = q & 7;
        *(u32x4*)(&sm.lam[row][pc * 8]) = lr.p[i];
      }
      if (threadIdx.x < TC) sm.lam[threadIdx.x][D] = row0 + (int)threadIdx.x < row_end ? 0x3f80u : 0u;   // the ones column
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int q = threadIdx.x + NT * i, row = q / 10, pc = q - 10 * row;
        if (q < TC * 10) *(u32x4*)(&sm.lam[row][pc * 8]) = lr.p[i];
      }
    }
  };

  RowRegs xr;
  RowRegs3 lr;
  load_rows_g(xr, Xb, X.sl, row_beg, row_end);
  load_left(lr, row_beg);
  __syncthreads();                 // the zero padding is in place
  stage(xr, lr, row_beg);
  __syncthreads();
  for (int row0 = row_beg; row0 < row_end; row0 += TC) {
    const bool more = row0 + TC < row_end;
    if (more) {
      load_rows_g(xr, Xb, X.sl, row0 + TC, row_end);
      load_left(lr, row0 + TC);
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      bf16x8 s[2];
      feature_tile<!KEY>(wx, &qb, sm.q[0], it, sm.qadd[16 * it + c], s);
      // dF: rows = features 16mt + 4g + r, column = token c
      f32x4 df[4] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        const bf16x8 lop = *(const bf16x8*)(&sm.lam[16 * it + c][32 * kk + 8 * g]);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) df[mt] = mfma(sa[mt][kk], lop, df[mt]);
      }
      // dE = F * dF, F from its bf16 image (element e of block bk <-> feature tile 2bk + e/4, row e%4)
      bf16x8 eimg[2];
#pragma unroll
      for (int bk = 0; bk < 2; ++bk) {
        const f32x8 fv = __builtin_convertvector(s[bk], f32x8);
        const f32x4 lo = {fv[0] * df[2 * bk][0], fv[1] * df[2 * bk][1], fv[2] * df[2 * bk][2], fv[3] * df[2 * bk][3]};
        const f32x4 hi = {fv[4] * df[2 * bk + 1][0], fv[5] * df[2 * bk + 1][1], fv[6] * df[2 * bk + 1][2], fv[7] * df[2 * bk + 1][3]};
        eimg[bk] = pack8(lo, hi);
      }
      f32x4 gt[NVT];
#pragma unroll
      for (int dt = 0; dt < NVT; ++dt) {
        if (dt < 4 || KEY) {
          gt[dt] = mfma(wt[dt][0], eimg[0], f32x4{0.f, 0.f, 0.f, 0.f});
          gt[dt] = mfma(wt[dt][1], eimg[1], gt[dt]);
        } else {
          gt[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      exchange_put_bf16(sm, gt, it, w, lane);
    }
    __syncthreads();
    {
      f32x4 fs[4] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
      finish_tiles(fs, sm, w, 0, lane);
      finish_tiles(fs, sm, w, 2, lane);
      const int trow = 16 * w + c, token = row0 + trow;
      if (KEY) {
        // derivative of the row term: rowsum(dE2) qk_scale^2 (C2 + C2^T) k   (C2 = -I/2: - qk_scale^2 k)
        const float rs = finish_col64(sm, w, lane) * a.scale * a.scale;
        if (isoC) {
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              fs[dt][r] = kLn2 * fs[dt][r] - rs * bf16_bits_to_f32(sm.q[0][trow][16 * dt + 4 * g + r]);
        } else {
          // dense C2 (ADERF, SADERF): the matrix as A operand (rows = gradient columns), the key rows as B operand
          bf16x8 kop[KS];
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) kop[ks] = *(const bf16x8*)(&sm.q[0][trow][32 * ks + 8 * g]);
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) {
            f32x4 u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) u = mfma(*(const bf16x8*)(&sm.csym[dt][ks][lane][0]), kop[ks], u);
            fs[dt] = kLn2 * fs[dt] + rs * u;
          }
        }
      } else {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) fs[dt] *= kLn2;
      }
      if (token < row_end) {
        if (G.dtype == 1) {
          uint16_t* yp = (uint16_t*)G.ptr + b * G.sb + h * G.sh + (long long)token * G.sl + 4 * g;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) *(bf16x4*)(yp + 16 * dt) = __builtin_convertvector(fs[dt], bf16x4);
        } else {
          float* yp = (float*)G.ptr + b * G.sb + h * G.sh + (long long)token * G.sl + 4 * g;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) *(f32x4*)(yp + 16 * dt) = fs[dt];
        }
      }
    }
    __syncthreads();               // every wave is done with the rows and the exchange buffer
    if (more) stage(xr, lr, row0 + TC);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Rows split over the waves (fast_rows.h): all 256 features of a (b,h) in LDS, every wave takes its own 16 NTT rows
// through everything that a row needs.  Nothing a row's gradient depends on belongs to another row once the two states
// are there, so one pass over a side does what used to be two: features are evaluated once, and neither rows nor
// partial tiles cross the waves.
//   queries: P -> Yhat = P T -> normaliser, G1 row (to memory for R) -> dP = G1 T^T -> dE = P * dP -> dQ = dE W~
//   keys:    S -> dV = S R;  dS = [V 1] R^T -> dE = S * dS -> dK = dE W~ + row term
// The contraction indices of dP run over the columns in the order in which the accumulators of Yhat hold them, those of
// dQ / dK over the features in the order of dE's accumulators: every operand on the row side is a packed accumulator.
// What bounds them: LDS operands, 150 KB per wave and 32 rows (9.5k cycles for a CU's eight waves) beside 8.7k cycles of
// matrix pipe and 5k of other vector work.  B8 H8 L4096 (us): features split, four kernels 47 + 54 + 39 + 54 -> rows split, two kernels 58 + 52; with
// the two-group sums of P^T G1 the call 255 -> 171 us, 1 x 4096 116 -> 71, 256 x 1000 262 -> 174, 8 x 32768 292 -> 178.
// ---------------------------------------------------------------------------------------------------------------
constexpr int NTR = 512;           // threads: eight waves, one workgroup per CU (LDS)

struct __attribute__((aligned(16))) SmemGradOps {
  uint16_t rowop[M / 16][2][64][8];   // state as A operand: row = feature 16 ft + c, k-step ks <-> columns (see grad_images)
  uint16_t wt[M / 32][4][64][8];      // W~^T as A operand: row = coordinate 16 dt + c, k <-> feature 32 fb + 16 (e/4) + 4 g + e%4
  float col64[M];                     // the state's normaliser column
};
struct SmemRows { rows::SmemOps f; SmemGradOps g; };
static_assert(sizeof(SmemRows) <= 160 * 1024, "one workgroup per CU");

// The images of SmemGradOps from those of rows::SmemOps by transposing LDS reads.  Column order of k-step ks:
// PACKED: k = 8 g + e <-> column 32 ks + 16 (e/4) + 4 g + e%4 (packed accumulators), else 32 ks + 8 g + e (rows as they
// lie in memory).  The normaliser column is not worth a third k-step of 32: it enters as initial value.
template <bool PACKED>
__device__ __forceinline__ void grad_images(const rows::SmemOps& f, SmemGradOps& out, int w, int lane) {
  const int g = lane >> 4, c = lane & 15, i = c >> 2, a = c & 3;
  for (int u = w; u < (M / 16) * 2; u += NTR / 64) {
    const int ft = u >> 1, ks = u & 1, fb = ft >> 1, mt = ft & 1;
    const int lo = 32 * ks + (PACKED ? 4 * g : 8 * g) + i, hi = lo + (PACKED ? 16 : 4);   // (four columns never cross a tile of 16)
    const u32x2 vl = lds_read_tr(&f.t[fb][lo >> 4][16 * a + (lo & 15)][4 * mt]);
    const u32x2 vh = lds_read_tr(&f.t[fb][hi >> 4][16 * a + (hi & 15)][4 * mt]);
    *(bf16x8*)(&out.rowop[ft][ks][lane][0]) = join8(vl, vh);
  }
  if (threadIdx.x < M) {
    const int q = threadIdx.x & 31;     // feature 32 fb + 16 mt + 4 g + r: element 4 mt + r of lanes (g, .)
    out.col64[threadIdx.x] = bf16_bits_to_f32(f.t[threadIdx.x >> 5][NVT - 1][16 * ((q >> 2) & 3)][4 * (q >> 4) + (q & 3)]);
  }
  for (int u = w; u < (M / 32) * 4; u += NTR / 64) {
    const int fb = u >> 2, dt = u & 3;
    const int piece = 16 * (2 * (dt & 1) + (a >> 1)) + 4 * g + i;
    const u32x2 vl = lds_read_tr(&f.w[2 * fb][dt >> 1][piece][4 * (a & 1)]);
    const u32x2 vh = lds_read_tr(&f.w[2 * fb + 1][dt >> 1][piece][4 * (a & 1)]);
    *(bf16x8*)(&out.wt[fb][dt][lane][0]) = join8(vl, vh);
  }
}

// dF of the 32 features of block fb: rows = features, lane <-> row 16 t + c.  `last[t]`: what the normaliser column meets
// in the lane's row, 1 on the key side (LAST = false).
template <int NTT, bool LAST>
__device__ __forceinline__ void state_times_rows(f32x4 (&df)[2][NTT], const SmemGradOps& sm, int fb, const bf16x8 (&b)[2][NTT],
                                                 const float* last, int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const f32x4 n = *(const f32x4*)(&sm.col64[32 * fb + 16 * mt + 4 * g]);
    const bf16x8 s0 = *(const bf16x8*)(&sm.rowop[2 * fb + mt][0][lane][0]), s1 = *(const bf16x8*)(&sm.rowop[2 * fb + mt][1][lane][0]);
#pragma unroll
    for (int t = 0; t < NTT; ++t) df[mt][t] = mfma(s0, b[0][t], LAST ? n * last[t] : n);
#pragma unroll
    for (int t = 0; t < NTT; ++t) df[mt][t] = mfma(s1, b[1][t], df[mt][t]);
  }
}

__device__ __forceinline__ f32x4 mul4(f32x4 x, f32x4 y) { return f32x4{x[0] * y[0], x[1] * y[1], x[2] * y[2], x[3] * y[3]}; }

// 16 NTT rows of 64 numbers as accumulators hold them (v[dt][t]: columns 16 dt + 4 g + r of row 16 t + c) -> memory.
template <int NTT>
__device__ __forceinline__ void store_acc_rows(const f32x4 (&v)[4][NTT], const TensorDev& T, long long base, int row0, int nv, int lane) {
  const int g = lane >> 4, c = lane & 15;
  if (T.dtype == 1) {
    const __amdgpu_buffer_rsrc_t r = pc::chunk_rsrc((const uint16_t*)T.ptr + base + (long long)row0 * T.sl, 2 * (int)T.sl, min(nv, 16 * NTT), 2 * D);
#pragma unroll
    for (int t = 0; t < NTT; ++t)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, __builtin_convertvector(v[dt][t], bf16x4)), r,
                                              2 * ((16 * t + c) * (int)T.sl + 16 * dt + 4 * g), 0, 0);
  } else {
    const __amdgpu_buffer_rsrc_t r = pc::chunk_rsrc((const float*)T.ptr + base + (long long)row0 * T.sl, 4 * (int)T.sl, min(nv, 16 * NTT), 4 * D);
#pragma unroll
    for (int t = 0; t < NTT; ++t)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[dt][t]), r, 4 * ((16 * t + c) * (int)T.sl + 16 * dt + 4 * g), 0, 0);
  }
}
// The other way, as fp32 (rows from nv on are zero).
template <int NTT>
__device__ __forceinline__ void load_acc_rows(f32x4 (&v)[4][NTT], const TensorDev& T, long long base, int row0, int nv, int lane) {
  const int g = lane >> 4, c = lane & 15;
  if (T.dtype == 1) {
    const __amdgpu_buffer_rsrc_t r = pc::chunk_rsrc((const uint16_t*)T.ptr + base + (long long)row0 * T.sl, 2 * (int)T.sl, min(nv, 16 * NTT), 2 * D);
#pragma unroll
    for (int t = 0; t < NTT; ++t)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const u32x2 p = __builtin_amdgcn_raw_buffer_load_b64(r, 2 * ((16 * t + c) * (int)T.sl + 16 * dt + 4 * g), 0, 0);
        v[dt][t] = f32x4{__uint_as_float(p[0] << 16), __uint_as_float(p[0] & 0xffff0000u), __uint_as_float(p[1] << 16),
                         __uint_as_float(p[1] & 0xffff0000u)};
      }
  } else {
    const __amdgpu_buffer_rsrc_t r = pc::chunk_rsrc((const float*)T.ptr + base + (long long)row0 * T.sl, 4 * (int)T.sl, min(nv, 16 * NTT), 4 * D);
#pragma unroll
    for (int t = 0; t < NTT; ++t)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        v[dt][t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, 4 * ((16 * t + c) * (int)T.sl + 16 * dt + 4 * g), 0, 0));
  }
}

// Query rows [row_beg, row_end): G1 rows and dQ.  Returns the number of rows this wave finished with a zero normaliser.
template <int NTT>
__device__ __forceinline__ int query_rows(const BwdArgs& ba, const SmemRows& sm, float wmax, int bh, int row_beg, int row_end) {
  const FastArgs& a = ba.f;
  const int b = bh / a.H, h = bh % a.H;
  const int lane0 = threadIdx.x & 63, g = lane0 >> 4, c = lane0 & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* Qb = (const uint16_t*)a.Q.ptr + b * a.Q.sb + h * a.Q.sh;
  constexpr int RT = 16 * NTT, STEP = RT * (NTR / 64);
  int nzero = 0, row0 = row_beg + RT * w;
  bf16x8 x[NTT][KS];
  rows::load_row_ops(x, Qb + (long long)row0 * a.Q.sl, a.Q.sl, row_end - row0, lane0);
  for (; row0 < row_end; row0 += STEP) {
    const int nv = row_end - row0;
    // (an opaque copy of the lane number: the images do not depend on the row, and operands read ahead of the loop spill)
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    f32x4 dy[4][NTT];
    load_acc_rows(dy, ba.dY, b * ba.dY.sb + h * ba.dY.sh, row0, nv, lane);
    bf16x8 p[M / 32][NTT], gop[2][NTT];
    float glast[NTT];
    {
      f32x4 y[NVT][NTT];
      float add[NTT];
      // (always shifted: the kernel that sums P^T G1 evaluates the features again and has to meet this scale)
#pragma unroll
      for (int t = 0; t < NTT; ++t) add[t] = -row_shift(__shfl(tile_row_norms(x[t][0], x[t][1], lane), 16 * (c >> 2) + c), wmax);
      rows::contract_rows<NTT, true, true>(y, sm.f, x, add, lane, p);
      // G1 = [dY / den, -(dY . Y) / den]
      const __amdgpu_buffer_rsrc_t rg = pc::chunk_rsrc(ba.gh + ((size_t)bh * ba.Lq + row0) * DVP, 2 * DVP, min(nv, RT), 2 * DVP);
#pragma unroll
      for (int t = 0; t < NTT; ++t) {
        const float den = y[NVT - 1][t][0];
        const float inv = den > 0.f ? __builtin_amdgcn_rcpf(den) : 0.f;
        nzero += count_zero_tokens((unsigned)__ballot(!(den > 0.f)) & 0xffffu, t, nv);
        float dot = 0.f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) dot += dy[dt][t][r] * (y[dt][t][r] * inv);
        dot += __shfl_xor(dot, 16);
        dot += __shfl_xor(dot, 32);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) dy[dt][t] *= inv;
        // (column 64 as the sum behind R will read it)
        const uint32_t last = f32_to_bf16_bits(-dot * inv);
        glast[t] = bf16_bits_to_f32((uint16_t)last);
        gop[0][t] = pack8(dy[0][t], dy[1][t]);
        gop[1][t] = pack8(dy[2][t], dy[3][t]);
        const u32x4 g0 = __builtin_bit_cast(u32x4, gop[0][t]), g1 = __builtin_bit_cast(u32x4, gop[1][t]);
        const int off = 2 * ((16 * t + c) * DVP + 4 * g);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{g0[0], g0[1]}, rg, off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{g0[2], g0[3]}, rg, off + 32, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{g1[0], g1[1]}, rg, off + 64, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{g1[2], g1[3]}, rg, off + 96, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{g == 0 ? last : 0u, 0u}, rg, off + 128, 0, 0);
      }
    }
    // the next rows travel during the second half
    const int next = row0 + STEP;
    rows::load_row_ops(x, Qb + (long long)next * a.Q.sl, a.Q.sl, row_end - next, lane);
    f32x4 gr[4][NTT], df[2][NTT];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int t = 0; t < NTT; ++t) gr[dt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    state_times_rows<NTT, true>(df, sm.g, 0, gop, glast, lane);
#pragma unroll
    for (int fb = 0; fb < M / 32; ++fb) {
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 e[NTT];
#pragma unroll
      for (int t = 0; t < NTT; ++t) {
        const u32x4 v = __builtin_bit_cast(u32x4, p[fb][t]);
        const f32x4 p0 = {__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xffff0000u), __uint_as_float(v[1] << 16), __uint_as_float(v[1] & 0xffff0000u)};
        const f32x4 p1 = {__uint_as_float(v[2] << 16), __uint_as_float(v[2] & 0xffff0000u), __uint_as_float(v[3] << 16), __uint_as_float(v[3] & 0xffff0000u)};
        e[t] = pack8(mul4(p0, df[0][t]), mul4(p1, df[1][t]));
      }
      if (fb + 1 < M / 32) {
        state_times_rows<NTT, true>(df, sm.g, fb + 1, gop, glast, lane);
#pragma unroll
        for (int i = 0; i < 4 * NTT; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 wv = *(const bf16x8*)(&sm.g.wt[fb][dt][lane][0]);
#pragma unroll
        for (int t = 0; t < NTT; ++t) gr[dt][t] = mfma(wv, e[t], gr[dt][t]);
      }
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int t = 0; t < NTT; ++t) gr[dt][t] *= kLn2;
    store_acc_rows(gr, ba.dQ, b * ba.dQ.sb + h * ba.dQ.sh, row0, nv, lane);
  }
  return nzero;
}

// Key rows [row_beg, row_end): dV and dK; cs: the key shift of the sequence.
template <int NTT>
__device__ __forceinline__ void key_rows(const BwdArgs& ba, const SmemRows& sm, const float* th, float cs, int bh, int row_beg, int row_end) {
  const FastArgs& a = ba.f;
  const int b = bh / a.H, h = bh % a.H;
  const int lane0 = threadIdx.x & 63, c = lane0 & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* Kb = (const uint16_t*)a.K.ptr + b * a.K.sb + h * a.K.sh;
  const uint16_t* Vb = (const uint16_t*)a.V.ptr + b * a.V.sb + h * a.V.sh;
  const bool isoC = ((int)th[2]) & 1;
  constexpr int RT = 16 * NTT, STEP = RT * (NTR / 64);
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
  int row0 = row_beg + RT * w;
  bf16x8 x[NTT][KS], v[2][NTT];
  auto load = [&](int r0) {
    rows::load_row_ops(x, Kb + (long long)r0 * a.K.sl, a.K.sl, row_end - r0, lane0);
    bf16x8 vr[NTT][KS];
    rows::load_row_ops(vr, Vb + (long long)r0 * a.V.sl, a.V.sl, row_end - r0, lane0);
#pragma unroll
    for (int t = 0; t < NTT; ++t) { v[0][t] = vr[t][0]; v[1][t] = vr[t][1]; }
  };
  load(row0);
  for (; row0 < row_end; row0 += STEP) {
    const int nv = row_end - row0;
    // (an opaque copy of the lane number: the images do not depend on the row, and operands read ahead of the loop spill)
    int lane = lane0;
    asm volatile("" : "+v"(lane));
    // row term - key shift of the lane's rows
    f32x4 add[NTT];
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      float rt;
      if (isoC) rt = -0.5f * kLog2e * a.scale * a.scale * __shfl(tile_row_norms(x[t][0], x[t][1], lane), 16 * (c >> 2) + c);
      else rt = 16 * t + c < nv ? a.rk[(size_t)bh * a.L + row0 + 16 * t + c] : 0.f;
      add[t] = f32x4{rt - cs, rt - cs, rt - cs, rt - cs};
    }
    f32x4 y[4][NTT], gr[4][NTT], rsum[NTT], acc[2][NTT], df[2][NTT];
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      rsum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) y[dt][t] = gr[dt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    rows::project<NTT, false>(acc, sm.f, 0, x, add, lane);
#pragma unroll
    for (int fb = 0; fb < M / 32; ++fb) {
      __builtin_amdgcn_sched_barrier(0);
      // exponentials of the block beside dF of the block
      state_times_rows<NTT, false>(df, sm.g, fb, v, nullptr, lane);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int t = 0; t < NTT; ++t) acc[mt][t] = exp2v(acc[mt][t]);
      bf16x8 p[NTT];
#pragma unroll
      for (int t = 0; t < NTT; ++t) p[t] = pack8(acc[0][t], acc[1][t]);
#pragma unroll
      for (int i = 0; i < 4 * NTT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      // dE beside dV
#pragma unroll
      for (int vt = 0; vt < 4; ++vt) {
        const bf16x8 s = *(const bf16x8*)(&sm.f.t[fb][vt][lane][0]);
#pragma unroll
        for (int t = 0; t < NTT; ++t) y[vt][t] = mfma(s, p[t], y[vt][t]);
      }
      bf16x8 e[NTT];
#pragma unroll
      for (int t = 0; t < NTT; ++t) e[t] = pack8(mul4(acc[0][t], df[0][t]), mul4(acc[1][t], df[1][t]));
#pragma unroll
      for (int i = 0; i < 4 * NTT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (fb + 1 < M / 32) rows::project<NTT, false>(acc, sm.f, fb + 1, x, add, lane);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 wv = *(const bf16x8*)(&sm.g.wt[fb][dt][lane][0]);
#pragma unroll
        for (int t = 0; t < NTT; ++t) gr[dt][t] = mfma(wv, e[t], gr[dt][t]);
      }
#pragma unroll
      for (int t = 0; t < NTT; ++t) rsum[t] = mfma(ones, e[t], rsum[t]);
    }
    store_acc_rows(y, ba.dV, b * ba.dV.sb + h * ba.dV.sh, row0, nv, lane);
    // derivative of the row term: rowsum(dE) qk_scale^2 (C2 + C2^T) k   (C2 = -I/2: - qk_scale^2 k)
    if (isoC) {
      f32x4 k[4][NTT];
      load_acc_rows(k, a.K, b * a.K.sb + h * a.K.sh, row0, nv, lane);
#pragma unroll
      for (int t = 0; t < NTT; ++t) {
        const float rs = rsum[t][0] * a.scale * a.scale;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) gr[dt][t] = kLn2 * gr[dt][t] - rs * k[dt][t];
      }
    } else {
      // dense C2 (ADERF, SADERF): the matrix as A operand (rows = gradient columns), the key rows as B operand
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        f32x4 u[NTT];
#pragma unroll
        for (int t = 0; t < NTT; ++t) u[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 cv = *(const bf16x8*)(&sm.f.t[KS * dt + ks][NVT - 1][lane][0]);
#pragma unroll
          for (int t = 0; t < NTT; ++t) u[t] = mfma(cv, x[t][ks], u[t]);
        }
#pragma unroll
        for (int t = 0; t < NTT; ++t) gr[dt][t] = kLn2 * gr[dt][t] + rsum[t][0] * a.scale * a.scale * u[t];
      }
    }
    load(row0 + STEP);
    store_acc_rows(gr, ba.dK, b * ba.dK.sb + h * ba.dK.sh, row0, nv, lane);
  }
}

// C2 + C2^T as A operand of the keys' row term, k-step ks of rows 16 dt + c, in the place of the state image's last column
// tile of block 2 dt + ks, which the key side does not need (dV has 64 columns, and column 64 is in rowop).
__device__ __forceinline__ void put_csym(rows::SmemOps& f, const float* C2) {
  const int piece = threadIdx.x, l = piece & 63, ks = (piece >> 6) % KS, dt = piece / (64 * KS);
  const int dd = 16 * dt + (l & 15), e0 = 32 * ks + 8 * (l >> 4);
  f32x8 cv;
#pragma unroll
  for (int e = 0; e < 8; ++e) cv[e] = C2[dd * D + e0 + e] + C2[(e0 + e) * D + dd];
  *(bf16x8*)(&f.t[KS * dt + ks][NVT - 1][l][0]) = __builtin_convertvector(cv, bf16x8);
}
static_assert(4 * KS * 64 == NTR && 4 * KS == M / 32, "one piece per thread, one block of the state image per k-step");

// SIDE 0: queries against T, SIDE 1: keys against R (both as k_fast_total leaves them).  grid (nblk * B*H), block 512.
template <int SIDE, int NTT>
__global__ void __launch_bounds__(NTR) k_bwd_rows(BwdArgs ba, int rows_per_blk, int nblk) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SmemRows& sm = *reinterpret_cast<SmemRows*>(smem_raw);
  const FastArgs& a = ba.f;
  const int id = rows::xcd_contiguous(blockIdx.x, gridDim.x), bh = id / nblk, blk = id - bh * nblk;
  const int b = bh / a.H, h = bh % a.H, pg = group_of(a.pgroups, b, h, a.H);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  rows::load_t_image<NTR>(sm.f, SIDE ? ba.Rpart + (size_t)bh * ba.rslots * M * DVP : a.Tpart + (size_t)bh * a.nslot * M * DVP);
  rows::load_w_image<NTR>(sm.f, a.Wbf + ((size_t)pg * 2 + SIDE) * M * D, a.bias + ((size_t)pg * 2) * M, max256(a.bias + ((size_t)pg * 2) * M));
  const float wmax = max256(a.wnorm + ((size_t)pg * 2 + SIDE) * M);
  rows::dma_wait<0>();
  __syncthreads();
  grad_images<SIDE == 0>(sm.f, sm.g, w, lane);
  __syncthreads();
  const int row_beg = blk * rows_per_blk, row_end = min(SIDE ? ba.Lk : ba.Lq, row_beg + rows_per_blk);
  if (SIDE == 0) {
    const int nzero = query_rows<NTT>(ba, sm, wmax, bh, row_beg, row_end);
    report_zero_rows(a.flushed, nzero, lane);
  } else {
    const float* th = a.theta + (size_t)group_of(a.groups, b, h, a.H) * (FS_THETA_HEADER_ + (size_t)D + 4 * (size_t)D * D);
    if (!(((int)th[2]) & 1)) {
      put_csym(sm.f, th + FS_THETA_HEADER_ + D + 3 * (size_t)D * D);
      __syncthreads();
    }
    key_rows<NTT>(ba, sm, th, a.cstar[bh], bh, row_beg, row_end);
  }
}

// R of a whole sequence for k_bwd_whole: the simpler loop of the two (no interleaving, values transposed in LDS) has the
// fewer registers, and that kernel has none to spare (512 sequences of 1024: 368 us against 417 with state_rows).
__device__ __forceinline__ void rstate_rows(const BwdArgs& ba, Smem& sm, int bh, int row_beg, int row_end, f32x4 (&R)[4][NVT]) {
  const FastArgs& a = ba.f;
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = lane & 15;
  const int pg = group_of(a.pgroups, b, h, a.H);
  const float wmax = max256(a.wnorm + ((size_t)pg * 2) * M), amax = max256(a.bias + ((size_t)pg * 2) * M);
  const uint16_t* Qb = (const uint16_t*)a.Q.ptr + b * a.Q.sb + h * a.Q.sh;
  const uint16_t* Gb = ba.gh + (size_t)bh * ba.Lq * DVP;

  WSlice wq;
  load_wslice(wq, a.Wbf + ((size_t)pg * 2) * M * D);
  float bcol[4];         // 2 (bias - largest bias) of feature 64w + 16 mt + c
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) bcol[mt] = 2.f * (a.bias[((size_t)pg * 2) * M + 64 * w + 16 * mt + c] - amax);
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) R[mt][vt] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto stage = [&](const RowRegs& qr, const RowRegs3& gr, int buf) {
    float n2[2];
    store_rows_s(qr, sm.k[buf], n2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = threadIdx.x + NT * i;
      if ((q & 7) == 0) sm.kadd[buf][q >> 3] = -row_shift(n2[i], wmax);
    }
    store_g80_s(gr, sm.vt[buf]);
  };

  RowRegs qr;
  RowRegs3 gr;
  load_rows_g(qr, Qb, a.Q.sl, row_beg, row_end);
  load_g80_g(gr, Gb, row_beg, row_end);
  stage(qr, gr, 0);
  __syncthreads();

  int buf = 0;
  for (int row0 = row_beg; row0 < row_end; row0 += TC, buf ^= 1) {
    const bool more = row0 + TC < row_end;
    if (more) {
      load_rows_g(qr, Qb, a.Q.sl, row0 + TC, row_end);
      load_g80_g(gr, Gb, row0 + TC, row_end);
    }
#pragma unroll
    for (int jp = 0; jp < 2; ++jp) {
      bf16x8 st[4];
      feature_pair_major<true>(wq, bcol, sm.k[buf], sm.kadd[buf], jp, 0.f, st);
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) {
        const bf16x8 vop = load_vop(sm.vt[buf], jp, vt);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) R[mt][vt] = mfma(st[mt], vop, R[mt][vt]);
      }
    }
    if (more) stage(qr, gr, buf ^ 1);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------------------------
// The whole backward pass of one (b,h) in one workgroup (non-causal calls with many or short sequences): the states T
// and R never leave the workgroup.  In the separate kernels each of them goes to memory once per slot, through a
// reduction, and back, 80 kB a time, while a sequence of 128 tokens is 150 kB of rows altogether.  Phases, each a loop
// over all rows of the sequence:
//   keys:    T = S^T [V 1]                (state_rows)
//   queries: G1 rows -> gh                (apply_rows_b<1>, T as operand image)
//   queries: dQ                           (grad_rows<0>; T's image turned into the row operand through LDS)
//   queries: R = P^T G1                   (rstate_rows; gh read back: written by this workgroup, behind a barrier)
//   keys:    dV = S R                     (apply_rows_b<2>)
//   keys:    dK                           (grad_rows<1>)
// T is dead before R is built.  grid (B*H), block 256, two per CU.
// ---------------------------------------------------------------------------------------------------------------
union SmemBwdWhole {
  SmemState s;
  SmemApply q;
  Smem r;
  SmemGrad g;
  uint16_t tr[NW][64][LDL];        // a wave's state slice as rows of 96 columns (transposition of the operand image)
};

// Operand image of a state slice (apply kernels: tb[vt][mb] element e <-> feature 32 mb + 16 (e/4) + 4g + e%4, column
// 16 vt + c) -> rows operand of the gradient kernels (sa[mt][kk] element e <-> feature 16 mt + c, column 32 kk + 8g + e;
// columns 80 .. 95 zero), through the wave's own LDS rows.  Barriers on both sides: the region overlays the buffers
// of the phases before and after.
__device__ __forceinline__ void image_to_rows(const bf16x8 (&tb)[NVT][2], uint16_t (*tr)[LDL], bf16x8 (&sa)[4][3]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  __syncthreads();
#pragma unroll
  for (int vt = 0; vt < NVT; ++vt)
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const u32x4 bits = __builtin_bit_cast(u32x4, tb[vt][mb]);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        tr[32 * mb + 16 * (e >> 2) + 4 * g + (e & 3)][16 * vt + c] = (uint16_t)(bits[e >> 1] >> (16 * (e & 1)));
    }
  *(u32x4*)(&tr[lane][DVP]) = u32x4{0u, 0u, 0u, 0u};
  *(u32x4*)(&tr[lane][DVP + 8]) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) sa[mt][kk] = *(const bf16x8*)(&tr[16 * mt + c][32 * kk + 8 * g]);
  __syncthreads();
}

__device__ __forceinline__ void pack_state(const f32x4 (&T)[4][NVT], bf16x8 (&tb)[NVT][2]) {
#pragma unroll
  for (int vt = 0; vt < NVT; ++vt)
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) tb[vt][mb] = pack8(T[2 * mb][vt], T[2 * mb + 1][vt]);
}

__global__ void __launch_bounds__(NT, 2) k_bwd_whole(BwdArgs ba) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SmemBwdWhole& sm = *reinterpret_cast<SmemBwdWhole*>(smem_raw);
  const FastArgs& a = ba.f;
  const int bh = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  bf16x8 tb[NVT][2];
  float cs;
  {
    f32x4 T[4][NVT];
    state_rows(a, sm.s, bh, 0, ba.Lk, (ba.Lk + TC - 1) / TC, T, cs);
    pack_state(T, tb);
  }
  const int nzero = apply_rows_b<1>(ba, sm.q, bh, tb, cs, 0, ba.Lq);
  report_zero_rows(a.flushed, nzero, lane);
  {
    bf16x8 sa[4][3];
    image_to_rows(tb, sm.tr[w], sa);
    grad_rows<0>(ba, sm.g, bh, sa, cs, 0, ba.Lq);
  }
  {
    f32x4 R[4][NVT];
    rstate_rows(ba, sm.r, bh, 0, ba.Lq, R);
    pack_state(R, tb);
  }
  apply_rows_b<2>(ba, sm.q, bh, tb, cs, 0, ba.Lk);
  {
    bf16x8 sa[4][3];
    image_to_rows(tb, sm.tr[w], sa);
    grad_rows<1>(ba, sm.g, bh, sa, cs, 0, ba.Lk);
  }
}

#define FS_LAUNCH_CHECK_() do { if (hipGetLastError() != hipSuccess) return 5; } while (0)
int launch_bwd_rstate(const BwdArgs& ba, int BH, hipStream_t st) {
  hipLaunchKernelGGL(k_bwd_rstate<false>, dim3(ba.rslots, BH), dim3(NT), sizeof(SmemState), st, ba);
  FS_LAUNCH_CHECK_();
  return 0;
}

}  // namespace bwd

using namespace bwd;

#define FS_LAUNCH_CHECK() do { if (hipGetLastError() != hipSuccess) return 5; } while (0)

size_t fast_bwd_lds_bytes() { return std::max(sizeof(SmemBwdWhole), sizeof(SmemRows)); }

// One non-causal backward call with a workgroup per sequence (after the constants; no state pass before it).
int launch_fast_backward_whole(const FastLaunch& f, const FastArgs& a, const TensorDev& dY, const TensorDev& dQ,
                               const TensorDev& dK, const TensorDev& dV, uint16_t* gh, hipStream_t st) {
  static_assert(sizeof(SmemBwdWhole) <= 80 * 1024, "k_bwd_whole: two workgroups per CU");
  BwdArgs ba;
  ba.f = a;
  ba.dY = dY; ba.dQ = dQ; ba.dK = dK; ba.dV = dV;
  ba.gh = gh; ba.Rpart = nullptr; ba.rcpart = nullptr;
  ba.Lq = f.Lq; ba.Lk = f.Lk; ba.rslots = 0; ba.rows_per_rslot = 0;
  if (hipFuncSetAttribute((const void*)k_bwd_whole, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmemBwdWhole)) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  hipLaunchKernelGGL(k_bwd_whole, dim3(f.B * f.H), dim3(NT), sizeof(SmemBwdWhole), st, ba);
  FS_LAUNCH_CHECK();
  return 0;
}

// One non-causal backward call after the forward state pass (f.Tpart slot 0 = total state, f.cstar = key shifts).
int launch_fast_backward(const FastLaunch& f, const FastArgs& a, const TensorDev& dY, const TensorDev& dQ,
                         const TensorDev& dK, const TensorDev& dV, uint16_t* gh, float* Rpart, float* rcpart,
                         int rslots, hipStream_t st) {
  BwdArgs ba;
  ba.f = a;
  ba.dY = dY; ba.dQ = dQ; ba.dK = dK; ba.dV = dV;
  ba.gh = gh; ba.Rpart = Rpart; ba.rcpart = rcpart;
  ba.Lq = f.Lq; ba.Lk = f.Lk;
  const int BH = f.B * f.H;
  {       // the slots of R: cut like the forward states, within the planned ones
    const int chunks = (f.Lq + TC - 1) / TC, want = rows::parts_per_sequence(BH, (chunks + 1) / 2, std::min(chunks, rslots), 2.f);
    ba.rows_per_rslot = (chunks + want - 1) / want * TC;
    ba.rslots = (f.Lq + ba.rows_per_rslot - 1) / ba.rows_per_rslot;
  }
  // row tiles of 16 per wave: two where that leaves every wave of the chip a step; one workgroup per CU, whole steps each
  auto launch = [&](int side, int L) {
    const bool two = (long long)BH * ((L + 15) / 16) >= 2 * 2048;
    auto kernel = side ? (two ? k_bwd_rows<1, 2> : k_bwd_rows<1, 1>) : (two ? k_bwd_rows<0, 2> : k_bwd_rows<0, 1>);
    const int step = (two ? 32 : 16) * (NTR / 64) / 2;
    const int want = rows::parts_per_sequence(BH, (L + 2 * step - 1) / (2 * step), (L + step - 1) / step, 1.f);
    const int rows_per_blk = (((L + want - 1) / want) + step - 1) / step * step, nblk = (L + rows_per_blk - 1) / rows_per_blk;
    if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmemRows)) != hipSuccess) {
      (void)hipGetLastError();
      return 2;
    }
    hipLaunchKernelGGL(kernel, dim3(nblk * BH), dim3(NTR), sizeof(SmemRows), st, ba, rows_per_blk, nblk);
    return hipGetLastError() == hipSuccess ? 0 : 5;
  };
  if (int rc = launch(0, f.Lq)) return rc;
  if (hipFuncSetAttribute((const void*)k_bwd_rstate2, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kState2Lds) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  // (time of a call with two groups over one: 1.02 at three chunks a slot, 1.00 at four)
  if (ba.rows_per_rslot > 4 * TC) hipLaunchKernelGGL(k_bwd_rstate2, dim3(ba.rslots, BH), dim3(2 * NT), kState2Lds, st, ba);
  else hipLaunchKernelGGL(k_bwd_rstate<true>, dim3(ba.rslots, BH), dim3(NT), sizeof(SmemState), st, ba);
  FS_LAUNCH_CHECK();
  launch_fast_total(Rpart, rcpart, nullptr, ba.rslots, ba.rslots, BH, nullptr, st);
  FS_LAUNCH_CHECK();
  if (int rc = launch(1, f.Lk)) return rc;
  return 0;
}

}  // namespace fs
