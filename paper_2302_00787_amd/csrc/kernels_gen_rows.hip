// General-shape kernels on fp32 matrix instructions (v_mfma_f32_16x16x4_f32) without data movement between the stages:
// any d <= 128, any M, f32 or bf16 storage.  (The kernels that still stage every operand in LDS: kernels_generic.hip.)
//
// Lane l = (g, c) = (l / 16, l % 16) supplies A[i = c][k = g] and B[k = g][j = c] and owns D[i = 4 g + r][j = c] in register
// r.  The order of the contraction index is free as long as both operands agree, and with k = g of step r standing for
// index 4 g + r an accumulator register IS an operand: features (rows = tokens, columns = features) feed the state update
// as they come from exp2, and so on.  Rows of 16 q + 4 g .. + 3 of a tensor are one 16-byte load per lane and four steps.
// The matrix pipe (32 cycles an instruction, 2048 flops) is busy 52 % of the SIMD time in k_gen_kmax and 38 % in k_gen_state at d = 128,
// M = 512: the rest is waiting for rows (half of a state wave's cycles: every wave fetches rows and values for itself) and the
// exponentials.
#include <type_traits>

#include "gen_widths.h"
#include "kernels.h"
#include "split3.h"

namespace fs {
namespace {

using namespace gen;

// Nothing in a kernel depends on the sizes within a width (a uniform branch around a load is a wait for it: state of B2 H4
// L4096 d64 M256 68 us with, 37 without): what lies past a row or a value row is multiplied by zero.

// BF: storage of a tensor.
template <int BF>
__device__ __forceinline__ float load1(const TensorDev& t, long long idx) {
  return BF ? bf16_bits_to_f32(((const uint16_t*)t.ptr)[idx]) : ((const float*)t.ptr)[idx];
}

// Numbers 16 q + 4 g .. + 3 of a row of d at element `at`, as they lie in memory.  Rows start at multiples of 16 bytes, so that a
// row of a multiple of four numbers is read four at a time and never past its end; groups past the end repeat the last.
template <int BF, int Q> struct RawRow { typename std::conditional<BF, u32x2, u32x4>::type v[Q]; };
// D4: d is a multiple of four.
template <int D4, int BF, int Q>
__device__ __forceinline__ void fetch_row(RawRow<BF, Q>& x, const TensorDev& t, long long at, int d, int g) {
  typedef typename std::conditional<BF, u32x2, u32x4>::type Raw;
  typedef typename std::conditional<BF, uint16_t, uint32_t>::type Elem;
  const Elem* p = (const Elem*)t.ptr + at;
  if constexpr (D4) {
#pragma unroll
    for (int q = 0; q < Q; ++q) x.v[q] = *(const Raw*)(p + min(16 * q + 4 * g, d - 4));
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t e[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int col = 16 * q + 4 * g + s;
        const uint32_t v = p[min(col, d - 1)];
        e[s] = col < d ? v : 0u;
      }
      if constexpr (BF) x.v[q] = u32x2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
      else x.v[q] = u32x4{e[0], e[1], e[2], e[3]};
    }
  }
}
// scale[q]: what the numbers of group q are multiplied by, zero past the row (row_scales).
template <int Q>
__device__ __forceinline__ void row_scales(float (&sc)[Q], int d, float scale, int g) {
#pragma unroll
  for (int q = 0; q < Q; ++q) sc[q] = 16 * q + 4 * g < d ? scale : 0.f;
}
template <int BF, int Q>
__device__ __forceinline__ f32x4 row_group(const RawRow<BF, Q>& x, int q, float sc) {
  if constexpr (BF) {
    const u32x2 p = x.v[q];
    return f32x4{__uint_as_float(p[0] << 16), __uint_as_float(p[0] & 0xffff0000u), __uint_as_float(p[1] << 16), __uint_as_float(p[1] & 0xffff0000u)} * sc;
  } else {
    return __builtin_bit_cast(f32x4, x.v[q]) * sc;
  }
}

// Registers and rows of sixteen lanes exchanged: register j of row g <- register g of row j.  Of numbers 16 q + 4 g + r that makes
// 16 q + 4 r + g: the order in which the kernels on LDS tiles (kernels_generic.hip) run through a row.
__device__ __forceinline__ f32x4 lane_rows_transposed(f32x4 v) {
  const u32x4 u = __builtin_bit_cast(u32x4, v);
  const auto a = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false), b = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
  const auto p = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), q = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return __builtin_bit_cast(f32x4, u32x4{p[0], p[1], q[0], q[1]});
}

// ---------------------------------------------------------------------------------------------------
// Key-side maximum of the exponent per (b, h), max_{j,m} E2[j,m]: one partial maximum per workgroup, part[bh][block], or
// where there is no room for them an atomic maximum into kmax[bh] (ordered-uint image; atomics of many workgroups on one
// address queue up in memory, 15 ns each: 38 us of a 188 us call with one per wave); and the row terms of the keys (rk). A
// workgroup takes four (wide rows: two) tiles of 16 tokens, which every wave holds as operands.  Row terms: of an isotropic
// set a tile per wave; of a dense one every wave takes every fourth group of sixteen coordinates of all the tiles through C, as
// groups of four numbers, and the waves' parts are summed in LDS (each tile's terms by one wave, C in single words: causal f32
// B8 H8 L300 d128 M200 378 us for the call, now 258).  Then every fourth tile of 16 features.  grid (tokens, B*H), block 256.
// ---------------------------------------------------------------------------------------------------
template <int Q> constexpr int KMAX_T = Q >= 6 ? 2 : 4;      // token tiles per workgroup
// SP: the projection on bf16 pieces (split3.h), W~ from the images of the kernels behind (bf16 B1 H16 L4096 d128 M512 92 -> 66 us, f32
// B2 H4 L4096 d64 M256 17.2 -> 14.7).
template <int Q, int XB, int D4, int SP>
__global__ void __launch_bounds__(256, 2) k_gen_kmax(GenSide ks, int Lk, int H, int M, int d, uint32_t* kmax_u, float* part, GenSplit split) {
  constexpr int TT = KMAX_T<Q>;
  __shared__ __align__(16) float rpart[4][16 * TT];
  __shared__ float wmax[4];
  const int bh = blockIdx.y, b = bh / H, h = bh % H, row0 = blockIdx.x * 16 * TT;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pg = group_of(ks.pgroups, b, h, H);
  const TensorDev W{ks.W + ((size_t)pg * 2 + 1) * M * d, 0, 0, 0, 0};
  const float* bias = ks.bias + ((size_t)pg * 2 + 1) * M;
  const float* th = ks.theta + (size_t)group_of(ks.groups, b, h, H) * ks.theta_stride;
  const long long xbase = b * ks.X.sb + h * ks.X.sh;
  float sc[Q], one[Q];
  row_scales(sc, d, ks.scale, g);
  row_scales(one, d, 1.f, g);
  // everything the kernel starts from is requested at once
  RawRow<XB, Q> raw[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) fetch_row<D4>(raw[t], ks.X, xbase + (long long)min(row0 + 16 * t + c, Lk - 1) * ks.X.sl, d, g);
  const int nft = (M + 15) / 16;
  RawRow<0, Q> wn;
  if (!SP) fetch_row<D4>(wn, W, (long long)min(16 * w + c, M - 1) * d, d, g);
  float bn = bias[min(16 * w + c, M - 1)];
  f32x4 x[TT][Q];
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int q = 0; q < Q; ++q) x[t][q] = row_group(raw[t], q, sc[q]);
  // row terms x C x + alpha |x|^2 of all the tokens, by way of LDS into accumulator order.  Isotropic: a tile per wave.
  // Dense: every fourth group of sixteen coordinates per wave, (C x)[a] for a = 16 q + 4 g + r of token c times x[a],
  // which the lane holds
  f32x4 rt[TT];
  if (((int)th[2]) & 1) {
    const int tw = w & (TT - 1), row = row0 + 16 * tw + c;
    float p = 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t)
      if (t == tw)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) p += x[t][q][r] * x[t][q][r];
    p *= ks.alpha - 0.5f;
    p += __shfl_xor(p, 16);
    p += __shfl_xor(p, 32);
    if (g == 0) {
      rpart[0][16 * tw + c] = p;       // (two waves for a tile, where there are two tiles, agree)
      if (row < Lk) ks.rk[(size_t)bh * Lk + row] = kLog2e * p;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TT; ++t) rt[t] = *(const f32x4*)(&rpart[0][16 * t + 4 * g]);
  } else {
    const TensorDev Cm{th + ks.c_offset, 0, 0, 0, 0};
    float p[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) p[t] = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if ((q & 3) != w) continue;
      f32x4 cx[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) cx[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      RawRow<0, Q> cr;
      fetch_row<D4>(cr, Cm, (long long)min(16 * q + c, d - 1) * d, d, g);
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const f32x4 ck = row_group(cr, k, one[k]);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int t = 0; t < TT; ++t) cx[t] = mfma4(ck[s], x[t][k][s], cx[t]);
      }
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[t] += x[t][q][r] * (cx[t][r] + ks.alpha * x[t][q][r]);
    }
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      p[t] += __shfl_xor(p[t], 16);
      p[t] += __shfl_xor(p[t], 32);
      if (g == 0) rpart[w][16 * t + c] = p[t];
    }
    __syncthreads();
    const int tid = threadIdx.x;
    if (tid < 16 * TT && row0 + tid < Lk)
      ks.rk[(size_t)bh * Lk + row0 + tid] = kLog2e * ((rpart[0][tid] + rpart[1][tid]) + (rpart[2][tid] + rpart[3][tid]));
#pragma unroll
    for (int t = 0; t < TT; ++t)
      rt[t] = (*(const f32x4*)(&rpart[0][16 * t + 4 * g]) + *(const f32x4*)(&rpart[1][16 * t + 4 * g])) +
              (*(const f32x4*)(&rpart[2][16 * t + 4 * g]) + *(const f32x4*)(&rpart[3][16 * t + 4 * g]));
  }
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 16 * t + 4 * g + r;
      rt[t][r] = row < Lk ? kLog2e * rt[t][r] : -INFINITY;
    }
  float m = -INFINITY;
  if constexpr (SP) {
    constexpr int KS = (Q + 1) / 2;
    typedef typename std::conditional<XB, bf16x8, Split3>::type XOp;
    XOp xo[TT][KS];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const long long at = xbase + (long long)min(row0 + 16 * t + c, Lk - 1) * ks.X.sl;
#pragma unroll
      for (int k = 0; k < KS; ++k) {         // (past the row W~ is zero)
        const int c0 = min(32 * k + 8 * g, d - 4), c1 = min(32 * k + 8 * g + 4, d - 4);
        if constexpr (XB) {
          const u32x2 lo = *(const u32x2*)((const uint16_t*)ks.X.ptr + at + c0), hi = *(const u32x2*)((const uint16_t*)ks.X.ptr + at + c1);
          xo[t][k] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
        } else {
          xo[t][k] = split3(*(const f32x4*)((const float*)ks.X.ptr + at + c0), *(const f32x4*)((const float*)ks.X.ptr + at + c1));
        }
      }
    }
    const uint16_t* img = split.img + ((size_t)pg * 2 + 1) * split.tiles * split.steps * 3 * 512 + 8 * lane;
    auto image = [&](Split3 (&o)[KS], int ft) {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const uint16_t* p = img + ((size_t)ft * split.steps + k) * 3 * 512;
        o[k] = {*(const bf16x8*)p, *(const bf16x8*)(p + 512), *(const bf16x8*)(p + 1024)};
      }
    };
    Split3 wn[KS];
    image(wn, min(w, nft - 1));
    for (int ft = w; ft < nft; ft += 4) {
      f32x4 acc[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      Split3 wr[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) wr[k] = wn[k];
      const float bf = 16 * ft + c < M ? bn : -INFINITY;
      const int fn = min(ft + 4, nft - 1);   // the next tile's operands travel meanwhile
      image(wn, fn);
      bn = bias[min(16 * fn + c, M - 1)];
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          if constexpr (XB) {
            acc[t] = mfma_bf16(xo[t][k], wr[k].l, acc[t]);
            acc[t] = mfma_bf16(xo[t][k], wr[k].m, acc[t]);
            acc[t] = mfma_bf16(xo[t][k], wr[k].h, acc[t]);
          } else {
            acc[t] = mfma3_t(xo[t][k], wr[k], acc[t]);
          }
        }
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, acc[t][r] + bf + rt[t][r]);
    }
  } else {
    for (int ft = w; ft < nft; ft += 4) {
      f32x4 acc[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      f32x4 wr[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) wr[q] = row_group(wn, q, one[q]);
      const float bf = 16 * ft + c < M ? bn : -INFINITY;
      const int fn = min(16 * (ft + 4) + c, M - 1);       // the next tile's row travels meanwhile
      fetch_row<D4>(wn, W, (long long)fn * d, d, g);
      bn = bias[fn];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int t = 0; t < TT; ++t) acc[t] = mfma4(x[t][q][s], wr[q][s], acc[t]);
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, acc[t][r] + bf + rt[t][r]);
    }
  }
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) m = fmaxf(m, __shfl_xor(m, s));
  if (lane == 0) wmax[w] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    if (part != nullptr) part[(size_t)bh * gridDim.x + blockIdx.x] = m;
    else atomicMax(&kmax_u[bh], float_to_ordered(m));
  }
}

// ---------------------------------------------------------------------------------------------------
// Partial states (Section 2.1, S^T C): Tpart[bh][seg][m][v] = sum_{j in seg} exp2(E2[j,m] - kmax) * V1[j,v].  With row_shift !=
// nullptr the query side of the backward pass: features of side 0 with the per-row shifts of the forward pass (no row term),
// "values" = rows of the output gradient.  The gradients' kernels evaluate the features of both sides again, and what they and
// this one round differently does not cancel in them against the normalisers: where they go through LDS tiles (TILES), the
// projection runs through a row in their order, four lane swaps per four numbers (without: dV and dK of the non-causal
// backward pass 1.1 times as far off on average, up to 1.6).  A wave holds 16 FT features (state_tiles): their rows of W~ and their state stay in
// registers, tokens pass by sixteen at a time straight from memory; no LDS, no barrier.  f32 B2 H4 L4096 d64 M256: 60 -> 37
// us (18 at the matrix rate), bf16 B1 H16 L4096 d128 M512: 425 -> 310 (118).  grid (nseg, ceil(M / (16 FT
// waves)), B*H), block 64 waves.
// ---------------------------------------------------------------------------------------------------
template <int Q, int XB, int VB, int D4, int TILES, int FT>
__global__ void __launch_bounds__(256, 2) k_gen_state(GenSide ks, TensorDev V, int Lk, int H, int M, int d, int nv, int append_ones,
                                                      int ldt, int rows_per_seg, int nseg, uint32_t* kmax_u, const float* part,
                                                      int npart, const float* row_shift, float* Tpart) {
  constexpr int VT = VT_OF<Q>;
  const int seg = blockIdx.x, bh = blockIdx.z, b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int f0 = 16 * FT * (blockIdx.y * (blockDim.x >> 6) + w);
  if (f0 >= M) return;
  const int pg = group_of(ks.pgroups, b, h, H), side = row_shift == nullptr ? 1 : 0;
  const TensorDev W{ks.W + ((size_t)pg * 2 + side) * M * d, 0, 0, 0, 0};
  const float* bias = ks.bias + ((size_t)pg * 2 + side) * M;
  float shift = 0.f;
  if (row_shift == nullptr) {
    if (part != nullptr) {
      shift = -INFINITY;
      for (int i = lane; i < npart; i += 64) shift = fmaxf(shift, part[(size_t)bh * npart + i]);
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) shift = fmaxf(shift, __shfl_xor(shift, s));
      if (seg == 0 && f0 == 0 && lane == 0) kmax_u[bh] = float_to_ordered(shift);      // for the kernels behind this one
    } else {
      shift = ordered_to_float(kmax_u[bh]);
    }
  }
  const int row_beg = seg * rows_per_seg, row_end = min(Lk, row_beg + rows_per_seg);
  const long long xbase = b * ks.X.sb + h * ks.X.sh, vbase = b * V.sb + h * V.sh;
  const float* rterm = row_shift == nullptr ? ks.rk + (size_t)bh * Lk : row_shift + (size_t)bh * Lk;
  const float rsign = row_shift == nullptr ? 1.f : -1.f;
  typedef typename std::conditional<VB, uint16_t, uint32_t>::type VElem;

  float sc[Q];
  row_scales(sc, d, ks.scale, g);
  int off[VT];                       // the columns of values the lane reads
#pragma unroll
  for (int vt = 0; vt < VT; ++vt) off[vt] = min(16 * vt + c, nv - 1);
  const int ones_col = append_ones ? nv : -1;
  RawRow<XB, Q> xn;
  fetch_row<D4>(xn, ks.X, xbase + (long long)min(row_beg + c, row_end - 1) * ks.X.sl, d, g);
  f32x4 wr[FT][Q], T[FT][VT];
  float bf[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int f = f0 + 16 * ft + c;
    RawRow<0, Q> raw;
    fetch_row<D4>(raw, W, (long long)min(f, M - 1) * d, d, g);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      wr[ft][q] = row_group(raw, q, 16 * q + 4 * g < d ? 1.f : 0.f);
      if (TILES) wr[ft][q] = lane_rows_transposed(wr[ft][q]);
    }
    bf[ft] = f < M ? bias[f] : -INFINITY;
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) T[ft][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int row0 = row_beg; row0 < row_end; row0 += 16) {
    // values of tokens 4 g + r, column 16 vt + c, and the tokens' row terms: used after the projections
    VElem vraw[VT][4];
    float rt[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rc = min(row0 + 4 * g + r, row_end - 1);
      rt[r] = rterm[rc];
      const VElem* p = (const VElem*)V.ptr + vbase + (long long)rc * V.sl;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) vraw[vt][r] = p[off[vt]];
    }
    f32x4 acc[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) acc[ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      f32x4 x = row_group(xn, q, sc[q]);
      if (TILES) x = lane_rows_transposed(x);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) acc[ft] = mfma4(x[s], wr[ft][q][s], acc[ft]);
    }
    fetch_row<D4>(xn, ks.X, xbase + (long long)min(row0 + 16 + c, row_end - 1) * ks.X.sl, d, g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = row0 + 4 * g + r < row_end;
      rt[r] = ok ? rsign * rt[r] : -INFINITY;
      // (in this order: row term less shift first, as far as 64-bit sums tell, leaves 1.04 times the error in non-causal
      // attention over the range of d and M, up to 1.3 times at d = 8)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) acc[ft][r] = fast_exp2(((acc[ft][r] + bf[ft]) + rt[r]) - shift);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = row0 + 4 * g + r < row_end;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        float v = VB ? bf16_bits_to_f32((uint16_t)vraw[vt][r]) : __uint_as_float((uint32_t)vraw[vt][r]);
        v = 16 * vt + c < nv ? v : (16 * vt + c == ones_col ? 1.f : 0.f);
        v = ok ? v : 0.f;
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) T[ft][vt] = mfma4(acc[ft][r], v, T[ft][vt]);
      }
    }
  }
  float* out = Tpart + (((size_t)bh * nseg + seg) * M) * ldt;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int vt = 0; vt < VT; ++vt)
      if (16 * vt < ldt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = f0 + 16 * ft + 4 * g + r;
          if (m < M) out[(size_t)m * ldt + 16 * vt + c] = T[ft][vt][r];
        }
      }
}

#define FS_LAUNCH_CHECK() do { if (hipGetLastError() != hipSuccess) return 5; } while (0)

}  // namespace

// Rows of a workgroup of k_gen_kmax, and its partial maxima where they fit.  (The room is that of one side's projection matrices:
// with room for every call some workspaces would pass the fixed size of the scratch array that serves calls without one.)
static int kmax_rows(int d) {
  return by_width(d, 0, [](auto q) { return 16 * KMAX_T<q()>; });
}
static float* kmax_part(const GenSide& ks, int Lk, int BH, int d) {
  const int n = (Lk + kmax_rows(d) - 1) / kmax_rows(d);
  return ks.kpart != nullptr && (size_t)BH * n <= ks.kcap ? ks.kpart : nullptr;
}

const float* gen_kmax_part(const GenSide& ks, int Lk, int BH, int d, int* npart) {
  *npart = (Lk + kmax_rows(d) - 1) / kmax_rows(d);
  return kmax_part(ks, Lk, BH, d);
}

int launch_gen_kmax(const GenSide& ks, int Lk, int BH, int H, int M, int d, uint32_t* kmax_u, hipStream_t st, const GenSplit& split) {
  return by_width(d, 0, [&](auto width) -> int {
    constexpr int Q = width(), TR = 16 * KMAX_T<Q>;
    auto kernel = d % 4 ? (ks.X.dtype ? k_gen_kmax<Q, 1, 0, 0> : k_gen_kmax<Q, 0, 0, 0>) : (ks.X.dtype ? k_gen_kmax<Q, 1, 1, 0> : k_gen_kmax<Q, 0, 1, 0>);
    if constexpr (Q > 1)         // (the kernels behind begin beyond rows of 16 numbers)
      if (split.img != nullptr) {
        if (ks.X.dtype) kernel = k_gen_kmax<Q, 1, 1, 1>;
        else if constexpr (Q < 6) kernel = k_gen_kmax<Q, 0, 1, 1>;
      }
    hipLaunchKernelGGL(kernel, dim3((Lk + TR - 1) / TR, BH), dim3(256), 0, st, ks, Lk, H, M, d, kmax_u, kmax_part(ks, Lk, BH, d), split);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

// Tiles of 16 features per wave of k_gen_state: few where the chip's 1024 SIMDs want waves or the last wave's tiles would be padding,
// more where rows and values, which every wave fetches for itself, are what it waits for.  us per call with 1 / 2 / 4 of them:
//   few waves       causal bf16 1 x 415 d 48 M 32  64.1 / 69.2 / 76.9;  f32 8 x 1472 d 64 M 256 backward  266.8 / 273.8 / 269.3 (736 waves of 4)
//   M <= 64         causal f32 1024 x 512 d 48 M 64  574 / 610 / 605;  bf16 1024 x 128 d 8 M 16  44.1 / 47.3 / 52.0
//   M <= 128        f32 4 x 16384 d 64 M 128  148 / 149 / 156;  causal f32 64 x 8192 d 16 M 128  404 / 395 / 403
//   M larger        causal f32 128 x 2048 d 64 M 512  1811 / 1809 / 1672;  causal f32 8 x 4096 d 64 M 256  152 / 153 / 147
//   wide rows       (four tiles do not fit)  f32 128 x 1024 d 128 M 256  1267 / 1064;  bf16 75 x 320 (segments of 96)  262 / 288
//   the same in the order of the LDS tiles (f32: two spill 53 registers, not 26)  f32 128 x 1024 d 128 M 256 backward
//                   2630 / 2893;  bf16 2600 / 2548
static int state_tiles(int Q, bool tiles, int M, int BH, int nseg, int rows_per_seg, bool bf16) {
  auto waves = [&](int ft) { return (long long)nseg * BH * ((M + 16 * ft - 1) / (16 * ft)); };
  if (Q == 8 && tiles && !bf16) return 1;
  if (Q >= 6) return waves(2) >= 1600 && (!bf16 || rows_per_seg >= 128) ? 2 : 1;
  if (M > 128 && waves(4) >= 800) return 4;
  return M > 64 && waves(2) >= 1600 ? 2 : 1;
}

int launch_gen_state(const GenSide& ks, const TensorDev& V, int Lk, int BH, int H, int M, int d, int nv, int append_ones, int ldt,
                     int rows_per_seg, int nseg, uint32_t* kmax_u, const float* row_shift, bool tiles, float* Tpart, hipStream_t st) {
  return by_width(d, ldt, [&](auto width) -> int {
    constexpr int Q = width();
    auto launch = [&](auto nft) -> int {
      constexpr int FT = nft();
      const int groups = (M + 16 * FT - 1) / (16 * FT), waves = groups < 4 ? groups : 4;
      auto pick = [&](auto d4, auto tl) {
        constexpr int D4 = d4(), TL = tl();
        return !ks.X.dtype ? k_gen_state<Q, 0, 0, D4, TL, FT> : V.dtype ? k_gen_state<Q, 1, 1, D4, TL, FT> : k_gen_state<Q, 1, 0, D4, TL, FT>;
      };
      const std::integral_constant<int, 0> no;
      const std::integral_constant<int, 1> yes;
      auto kernel = d % 4 ? (tiles ? pick(no, yes) : pick(no, no)) : (tiles ? pick(yes, yes) : pick(yes, no));
      hipLaunchKernelGGL(kernel, dim3(nseg, (groups + waves - 1) / waves, BH), dim3(64 * waves), 0, st, ks, V, Lk, H, M, d,
                         nv, append_ones, ldt, rows_per_seg, nseg, kmax_u, kmax_part(ks, Lk, BH, d), (Lk + kmax_rows(d) - 1) / kmax_rows(d),
                         row_shift, Tpart);
      FS_LAUNCH_CHECK();
      return 0;
    };
    const int ft = state_tiles(Q, tiles, M, BH, nseg, rows_per_seg, ks.X.dtype != 0);
    if (ft == 1) return launch(std::integral_constant<int, 1>());
    if constexpr (Q < 6)
      if (ft == 4) return launch(std::integral_constant<int, 4>());
    return launch(std::integral_constant<int, 2>());
  });
}

}  // namespace fs
