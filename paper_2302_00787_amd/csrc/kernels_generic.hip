// General-shape FAVOR# kernels: fp32 arithmetic on fp32 MFMA tiles (v_mfma_f32_16x16x4_f32), any d <= 128,
// any M, any sequence length, f32 or bf16 storage.  They serve the fp32 workloads and every shape the
// bf16 fast path does not cover; key maxima and states are in kernels_gen_rows.hip, the causal kernels of most shapes with d
// and dv multiples of four and M <= 512 in kernels_gen_walk.hip (its gen_walk_attention and gen_walk_backward say which).  All exponents are kept in the log2 domain: the projection matrices and
// biases arrive pre-multiplied by log2(e), so a feature is exp2(E2 - shift).
//
// Tile shape everywhere: 32 rows (tokens) x 32 features per step, 256 threads = 4 waves.
// MFMA 16x16x4 f32 operand layout used below: lane l supplies A[l%16][l/16] and B[l/16][l%16];
// accumulator register r of lane l is D[4*(l/16) + r][l%16].
#include <type_traits>

#include "fs_common.h"
#include "kernels.h"
#include "split3.h"

namespace fs {

constexpr int TR = 32;     // rows per tile
constexpr int MB = 32;     // features per block
constexpr int NT = 256;    // threads per workgroup (causal kernels: NTC)
// The causal kernels have eight waves, two per SIMD: with 164 to 256 registers (d > 32) one workgroup fills a CU, and at
// d = 128 it needs most of its LDS as well (they serve what the walks of kernels_gen_walk.hip do not).  Four waves work on the query side while the other four work on the key
// side, both projection blocks in LDS (two barriers fewer per block).  Against four waves: causal attention B2 H4 L4096
// d64 M256 f32 388 -> 320 us, causal backward pass B1 H16 L4096 d128 M512 5.63 -> 4.64 ms.
constexpr int NTC = 512;

// Every kernel comes in three widths W: rows of at most 32 W columns and values of at most 32 NV (W = 1: 64, 2: 96,
// 4: 144).  Registers of a tile and accumulators are counted for the width: with those of W = 4 for every d, two or three
// waves of k_gen_apply and k_gen_bwd_side fitted a SIMD, now four or five at d <= 32 and three or four at
// d <= 64.  f32, 2048 sequences of 128, d 8, M 32, when this was done: attention 152 -> 106 us, backward pass 425 -> 258.
template <int W> constexpr int NV = W == 4 ? 5 : W + 1;
template <int W, int WAVES> constexpr int ACC_V = (4 * NV<W> + WAVES - 1) / WAVES;   // 16 x 16 tiles of 32 rows of values, per wave
template <int W, int WAVES> constexpr int ACC_D = (4 * W + WAVES - 1) / WAVES;       // of 32 rows of a side

// This side's C matrix, or nullptr when the parameter set says C = -I/2 (flag bit 0 of the theta header).
__device__ __forceinline__ const float* side_cmat(const GenSide& s, int b, int h, int H) {
  const float* th = s.theta + (size_t)group_of(s.groups, b, h, H) * s.theta_stride;
  return (((int)th[2]) & 1) ? nullptr : th + s.c_offset;
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// acc += sum over k < n (a multiple of 4) of A[.][k] B[k][.]: ap and bp point at this lane's k = lane / 16 elements,
// sa and sb are the distances of consecutive k.  Eight steps' operands are read from LDS together: read one step at a
// time, each matrix instruction waits for an LDS latency of its own.
__device__ __forceinline__ f32x4 mfma_chain(const float* ap, int sa, const float* bp, int sb, int n, f32x4 acc) {
  int k = 0;
  for (; k + 32 <= n; k += 32) {
    float a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a[i] = ap[(k + 4 * i) * sa];
      b[i] = bp[(k + 4 * i) * sb];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = mfma4(a[i], b[i], acc);
  }
  for (; k < n; k += 4) acc = mfma4(ap[k * sa], bp[k * sb], acc);
  return acc;
}

// A tile of 32 rows and up to 32 NI columns travelling global -> registers -> LDS: thread t carries rows t/32 + (TH/32) j,
// columns t%32 + 32i.  All loads of a tile are in flight together, and between fetch and put a kernel may compute.  A
// loop that stores each element to LDS as it arrives is a chain of 16 - 18 memory latencies per tile, with one
// workgroup per CU (LDS) to hide them; together with mfma_chain and the state update from the LDS copy this took
// causal attention B2 H4 L4096 d64 M256 f32 from 704 to 405 us and the causal backward pass B1 H16 L4096 d128 M512
// from 15.2 to 5.9 ms (388 us and 5.6 ms once k_prep was faster too), bit for bit the same.  Addresses outside the tile are clamped into it, so that no load is
// conditional; the put writes zeros there.  The registers hold the raw bits (f32, or bf16 zero-extended).
template <int NI, int TH> struct Tile { uint32_t v[TR * 32 / TH][NI]; };
template <int NI, int TH>
__device__ __forceinline__ void tile_fetch(Tile<NI, TH>& t, const void* ptr, int dtype, long long base, long long stride,
                                           int live, int ncols) {
  int tid = threadIdx.x;
  // (causal kernels: offsets are computed at each fetch; hoisted out of the loops they take more than 100 registers)
  if constexpr (TH == NTC) asm volatile("" : "+v"(tid));
  const int r0 = tid >> 5, c0 = tid & 31;
  if (dtype == 0) {
    const uint32_t* p = (const uint32_t*)ptr + base;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (32 * i < ncols) {
#pragma unroll
        for (int j = 0; j < TR * 32 / TH; ++j) t.v[j][i] = p[(long long)min(r0 + (TH / 32) * j, live - 1) * stride + min(c0 + 32 * i, ncols - 1)];
      }
  } else {
    const uint16_t* p = (const uint16_t*)ptr + base;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (32 * i < ncols) {
#pragma unroll
        for (int j = 0; j < TR * 32 / TH; ++j) t.v[j][i] = p[(long long)min(r0 + (TH / 32) * j, live - 1) * stride + min(c0 + 32 * i, ncols - 1)];
      }
  }
}
// dst[r][c] = scale * tile for r < live, c < ncols, `fill` at column ncols of the live rows, 0 elsewhere up to ncols_pad.
template <int NI, int TH>
__device__ __forceinline__ void tile_put(const Tile<NI, TH>& t, int dtype, float* dst, int ld, int live, int ncols,
                                         int ncols_pad, float scale, float fill) {
  const int r0 = threadIdx.x >> 5, c0 = threadIdx.x & 31, shift = dtype == 0 ? 0 : 16;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = c0 + 32 * i;
    if (c < ncols_pad) {
#pragma unroll
      for (int j = 0; j < TR * 32 / TH; ++j) {
        const int r = r0 + (TH / 32) * j;
        float v = 0.f;
        if (r < live) v = c < ncols ? scale * __uint_as_float(t.v[j][i] << shift) : (c == ncols ? fill : 0.f);
        dst[r * ld + c] = v;
      }
    }
  }
}

// Rows of a side, and of values with the column of ones that is the normaliser.
template <int W, int TH> using RowTile = Tile<W, TH>;
template <int W, int TH> using ValTile = Tile<NV<W>, TH>;
static_assert(TR == 32 && MB == 32, "32 threads carry a row of a tile");
template <int N, int TH>
__device__ __forceinline__ void rows_fetch(Tile<N, TH>& x, const TensorDev& t, long long base, int row0, int nrows, int ncols) {
  tile_fetch(x, t.ptr, t.dtype, base + (long long)row0 * t.sl, t.sl, nrows - row0, ncols);
}
template <int N, int TH>
__device__ __forceinline__ void rows_put(const Tile<N, TH>& x, const TensorDev& t, float* dst, int ld, int row0, int nrows,
                                         int ncols, int ncols_pad, float scale) {
  tile_put(x, t.dtype, dst, ld, nrows - row0, ncols, ncols_pad, scale, 0.f);
}
template <int N, int TH>
__device__ __forceinline__ void values_fetch(Tile<N, TH>& x, const TensorDev& t, long long base, int row0, int nrows, int ncols) {
  tile_fetch(x, t.ptr, t.dtype, base + (long long)row0 * t.sl, t.sl, nrows - row0, ncols);
}
template <int N, int TH>
__device__ __forceinline__ void values_put(const Tile<N, TH>& x, const TensorDev& t, float* dst, int ld, int row0, int nrows,
                                           int ncols, int ncols_pad, int append_ones) {
  tile_put(x, t.dtype, dst, ld, nrows - row0, ncols, ncols_pad, 1.f, append_ones ? 1.f : 0.f);
}

// dst[r][c] = scale * T[row0 + r][c] for r < 32; zero outside [0, nrows) x [0, ncols); columns up to ncols_pad written.
template <int W, int TH = NT>
__device__ __forceinline__ void load_rows(float* dst, int ld, const TensorDev& t, long long base, int row0, int nrows,
                                          int ncols, int ncols_pad, float scale) {
  RowTile<W, TH> x;
  rows_fetch(x, t, base, row0, nrows, ncols);
  rows_put(x, t, dst, ld, row0, nrows, ncols, ncols_pad, scale);
}

// Value tile with an optional column of ones at index ncols (the normaliser column of attention).
template <int W, int TH = NT>
__device__ __forceinline__ void load_values(float* dst, int ld, const TensorDev& t, long long base, int row0, int nrows,
                                            int ncols, int ncols_pad, int append_ones) {
  ValTile<W, TH> x;
  values_fetch(x, t, base, row0, nrows, ncols);
  values_put(x, t, dst, ld, row0, nrows, ncols, ncols_pad, append_ones);
}

// Ws[f][c] = W[m0 + f][c] (zero rows past M), bias_s[f] = bias[m0 + f], in two halves.
template <int W, int TH> struct WRegs { RowTile<W, TH> w; float b; };
template <int N, int TH>
__device__ __forceinline__ void wblock_fetch(WRegs<N, TH>& r, const float* W, const float* bias, int m0, int M, int d) {
  tile_fetch(r.w, W, 0, (long long)m0 * d, d, M - m0, d);
  r.b = bias[min(m0 + (int)(threadIdx.x & (MB - 1)), M - 1)];
}
template <int N, int TH>
__device__ __forceinline__ void wblock_put(const WRegs<N, TH>& r, float* Ws, float* bias_s, int ld, int m0, int M, int d, int dpad) {
  tile_put(r.w, 0, Ws, ld, M - m0, d, dpad, 1.f, 0.f);
  if (threadIdx.x < MB) bias_s[threadIdx.x] = m0 + (int)threadIdx.x < M ? r.b : 0.f;
}
template <int WD>
__device__ __forceinline__ void load_wblock(float* Ws, float* bias_s, int ld, const float* W, const float* bias, int m0,
                                            int M, int d, int dpad) {
  WRegs<WD, NT> r;
  wblock_fetch(r, W, bias, m0, M, d);
  wblock_put(r, Ws, bias_s, ld, m0, M, d, dpad);
}

// The block of a state that belongs to features m0 .. m0 + 31 (rows of ldt floats; zero rows past M).
template <int N, int TH>
__device__ __forceinline__ void sblock_fetch(Tile<N, TH>& t, const float* T, int m0, int M, int ldt) {
  tile_fetch(t, T, 0, (long long)m0 * ldt, ldt, M - m0, ldt);
}
template <int N, int TH>
__device__ __forceinline__ void sblock_put(const Tile<N, TH>& t, float* Ts, int ld, int m0, int M, int ldt) {
  tile_put(t, 0, Ts, ld, M - m0, ldt, ldt, 1.f, 0.f);
}

// ((C + C^T) x)[c] for a dense C (four partial sums and several loads in flight: a plain loop is a chain of cache
// latencies).
__device__ __forceinline__ float sym_row_dot(const float* Cmat, int d, int c, const float* x) {
  const float* crow = Cmat + (size_t)c * d;
  const float* ccol = Cmat + c;
  float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
  int a = 0;
#pragma unroll 2
  for (; a + 4 <= d; a += 4) {
    t0 += (crow[a] + ccol[(size_t)a * d]) * x[a];
    t1 += (crow[a + 1] + ccol[(size_t)(a + 1) * d]) * x[a + 1];
    t2 += (crow[a + 2] + ccol[(size_t)(a + 2) * d]) * x[a + 2];
    t3 += (crow[a + 3] + ccol[(size_t)(a + 3) * d]) * x[a + 3];
  }
  for (; a < d; ++a) t0 += (crow[a] + ccol[(size_t)a * d]) * x[a];
  return (t0 + t1) + (t2 + t3);
}

// rterm[r] = log2e * (x_r^T C x_r + alpha |x_r|^2); Cmat == nullptr means C = -I/2.
__device__ void row_terms(float* rterm, const float* Xs, int ld, int d, const float* Cmat, float alpha) {
  if (threadIdx.x >= 8 * TR) return;         // eight threads a row
  const int r = threadIdx.x >> 3, part = threadIdx.x & 7;
  const float* x = Xs + r * ld;
  float acc = 0.f;
  if (Cmat == nullptr) {
    for (int a = part; a < d; a += 8) acc += x[a] * x[a];
    acc *= (alpha - 0.5f);
  } else {
    // (eight loads of the row of C in flight and four partial sums: the loop is a chain of cache latencies otherwise)
    for (int a = part; a < d; a += 8) {
      const float* crow = Cmat + (size_t)a * d;
      float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
      int b = 0;
#pragma unroll 2
      for (; b + 4 <= d; b += 4) {
        t0 += crow[b] * x[b];
        t1 += crow[b + 1] * x[b + 1];
        t2 += crow[b + 2] * x[b + 2];
        t3 += crow[b + 3] * x[b + 3];
      }
      for (; b < d; ++b) t0 += crow[b] * x[b];
      acc += x[a] * ((t0 + t1) + (t2 + t3) + alpha * x[a]);
    }
  }
  acc += __shfl_xor(acc, 1);
  acc += __shfl_xor(acc, 2);
  acc += __shfl_xor(acc, 4);
  if (part == 0) rterm[r] = kLog2e * acc;
}

// Row terms of the 32-row tile at row0 of (b,h), as k_gen_kmax left them.  Rows of padding get -inf, so that their features
// are exactly zero: with 0 the exponent of a feature is its bias less the sequence's key shift, which overflows where all
// keys are long.
__device__ __forceinline__ void row_terms_of(float* rterm, const GenSide& sd, int bh, int L, int row0, int row_end) {
  if (threadIdx.x < TR) rterm[threadIdx.x] = row0 + (int)threadIdx.x < row_end ? sd.rk[(size_t)bh * L + row0 + threadIdx.x] : -INFINITY;
}

// Wave w (of four) computes the 16x16 tile (row tile w>>1, feature tile w&1) of Xs * Ws^T.
__device__ __forceinline__ f32x4 proj_tile(const float* Xs, const float* Ws, int ld, int dpad) {
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
  const float* ap = Xs + ((w >> 1) * 16 + (lane & 15)) * ld + (lane >> 4);
  const float* bp = Ws + ((w & 1) * 16 + (lane & 15)) * ld + (lane >> 4);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  acc = mfma_chain(ap, 1, bp, 1, dpad, acc);
  return acc;
}

// Max of e[0..3] over the 16 lanes that share lane>>4, combined into LDS (ordered-uint image) per row.
__device__ __forceinline__ void rowmax_update(uint32_t* rowmax_u, const float e[4]) {
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float v = e[r];
    v = fmaxf(v, __shfl_xor(v, 1));
    v = fmaxf(v, __shfl_xor(v, 2));
    v = fmaxf(v, __shfl_xor(v, 4));
    v = fmaxf(v, __shfl_xor(v, 8));
    if ((lane & 15) == 0) atomicMax(&rowmax_u[(w >> 1) * 16 + 4 * (lane >> 4) + r], float_to_ordered(v));
  }
}

// One pass over all feature blocks computing, per row, max_m (W_m . x + bias_m) (+ rterm is added by the caller).
template <int WD>
__device__ void rowmax_pass(uint32_t* rowmax_u, const float* Xs, float* Ws, float* bias_s, int ld, const float* W,
                            const float* bias, int M, int d, int dpad) {
  if (threadIdx.x < TR) rowmax_u[threadIdx.x] = 0u;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  WRegs<WD, NT> wr;
  wblock_fetch(wr, W, bias, 0, M, d);
  for (int m0 = 0; m0 < M; m0 += MB) {
    __syncthreads();
    wblock_put(wr, Ws, bias_s, ld, m0, M, d, dpad);
    __syncthreads();
    if (m0 + MB < M) wblock_fetch(wr, W, bias, m0 + MB, M, d);
    const f32x4 acc = proj_tile(Xs, Ws, ld, dpad);
    const int f = (w & 1) * 16 + (lane & 15);
    float e[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) e[r] = (m0 + f < M) ? acc[r] + bias_s[f] : -INFINITY;
    rowmax_update(rowmax_u, e);
  }
  __syncthreads();
}

// The same with eight waves: two feature blocks per step, four waves each.
template <int WD>
__device__ void rowmax_pass2(uint32_t* rowmax_u, const float* Xs, float* Ws, float* Ws2, float* bias_s, float* bias2_s,
                             int ld, const float* W, const float* bias, int M, int d, int dpad) {
  if (threadIdx.x < TR) rowmax_u[threadIdx.x] = 0u;
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3, half = threadIdx.x >> 8;
  WRegs<WD, NTC> wa, wb;
  wblock_fetch(wa, W, bias, 0, M, d);
  if (MB < M) wblock_fetch(wb, W, bias, MB, M, d);
  for (int m0 = 0; m0 < M; m0 += 2 * MB) {
    __syncthreads();
    wblock_put(wa, Ws, bias_s, ld, m0, M, d, dpad);
    if (m0 + MB < M) wblock_put(wb, Ws2, bias2_s, ld, m0 + MB, M, d, dpad);
    __syncthreads();
    if (m0 + 2 * MB < M) wblock_fetch(wa, W, bias, m0 + 2 * MB, M, d);
    if (m0 + 3 * MB < M) wblock_fetch(wb, W, bias, m0 + 3 * MB, M, d);
    const int mb = m0 + half * MB;
    if (mb < M) {
      const f32x4 acc = proj_tile(Xs, half ? Ws2 : Ws, ld, dpad);
      const int f = (w & 1) * 16 + (lane & 15);
      float e[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) e[r] = (mb + f < M) ? acc[r] + (half ? bias2_s : bias_s)[f] : -INFINITY;
      rowmax_update(rowmax_u, e);
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------------
// Projection constants (Section 4, evaluation recipe): W~[m,:] = log2e * omega_m^T B, bias_m = log2e *
// (omega_m^T A omega_m + log D - 1/2 log M).  grid (ceil(M/4), 2 sides, pgroups), block 128: thread c carries column c
// of four features, so that a row of B is read once for the four, eight rows at a time in flight (one feature per
// workgroup and one load at a time: 231 us for 16 heads of d 128, M 512 and 24 us for 4 of d 64, M 256; now 28 and 8).  Four and not
// more: with few features the launch would leave most of the chip idle.  Further layers of the grid's second axis: value_maxima.
// ---------------------------------------------------------------------------------------------------
constexpr int PREP_F = 4;

// The largest finite number of rows row0 .. row0 + rows - 1 of a tensor, 4 cols numbers each, by 128 threads.
__device__ __forceinline__ float largest_of(const TensorDev& t, long long base, int row0, int rows, int cols, float* red) {
  float m = 0.f;
  for (int e0 = threadIdx.x; e0 < rows * cols; e0 += 8 * 128) {
    f32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = min(e0 + 128 * i, rows * cols - 1), row = e / cols;
      const long long at = base + (long long)(row0 + row) * t.sl + 4 * (e - row * cols);
      if (t.dtype) {
        const u32x2 p = *(const u32x2*)((const uint16_t*)t.ptr + at);
        v[i] = f32x4{__uint_as_float(p[0] << 16), __uint_as_float(p[0] & 0xffff0000u), __uint_as_float(p[1] << 16), __uint_as_float(p[1] & 0xffff0000u)};
      } else {
        v[i] = *(const f32x4*)((const float*)t.ptr + at);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) m = fmaxf(m, fabsf(v[i][j]) < INFINITY ? fabsf(v[i][j]) : 0.f);
  }
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) m = fmaxf(m, __shfl_xor(m, s));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmaxf(red[0], red[1]);
  __syncthreads();
  return m;
}
// Partial maxima of values and gradient, on the compute units that the constants leave idle (causal f32 B2 H4 L4096 d64 M256: 0.8 us,
// in k_gen_kmax, whose rows they are, 1.7).
__device__ __forceinline__ void value_maxima(const GenSplit& sp, int H, int first, int step, float* red) {
  const int parts = (sp.L + VMAX_ROWS - 1) / VMAX_ROWS, cols = sp.nv / 4;
  for (int p = first; p < sp.BH * parts; p += step) {
    const int bh = p / parts, b = bh / H, h = bh % H, row0 = (p - bh * parts) * VMAX_ROWS, rows = min(VMAX_ROWS, sp.L - row0);
    const float v = largest_of(sp.V, b * sp.V.sb + h * sp.V.sh, row0, rows, cols, red);
    const float g = sp.dmax != nullptr ? largest_of(sp.dY, b * sp.dY.sb + h * sp.dY.sh, row0, rows, cols, red) : 0.f;
    if (threadIdx.x == 0) {
      sp.vmax[p] = v;
      if (sp.dmax != nullptr) sp.dmax[p] = g;
    }
  }
}
__global__ void __launch_bounds__(128) k_prep(const float* theta, int groups, const float* Omega, int omega_groups, int pgroups,
                       int B, int H, int M, int d, float* W, float* bias, uint32_t* clear, int nclear, GenSplit split) {
  __shared__ float om[PREP_F][128];
  if (blockIdx.y >= 2) {
    value_maxima(split, H, ((blockIdx.y - 2) * gridDim.z + blockIdx.z) * gridDim.x + blockIdx.x, (gridDim.y - 2) * gridDim.z * gridDim.x, om[0]);
    return;
  }
  const int m0 = blockIdx.x * PREP_F, side = blockIdx.y, pg = blockIdx.z, nf = min(PREP_F, M - m0);
  int b = 0, h = 0;
  if (pgroups == H && pgroups != 1) h = pg;
  else if (pgroups != 1) { b = pg / H; h = pg % H; }
  const size_t tf = FS_THETA_HEADER_ + (size_t)d + 4 * (size_t)d * d;
  const float* th = theta + (size_t)group_of(groups, b, h, H) * tf;
  const float* omg = Omega + ((size_t)group_of(omega_groups, b, h, H) * M + m0) * d;
  const float* Bm = th + FS_THETA_HEADER_ + d + (side ? (size_t)d * d : 0);
  const size_t o = (((size_t)pg * 2 + side) * M + m0);
  const int c = threadIdx.x;
  // the call's counter and key maxima start at zero (a launch of its own costs 4 us)
  for (int i = ((blockIdx.z * 2 + blockIdx.y) * gridDim.x + blockIdx.x) * 128 + c; i < nclear; i += gridDim.x * 2 * gridDim.z * 128) clear[i] = 0u;
#pragma unroll
  for (int f = 0; f < PREP_F; ++f) om[f][c] = (f < nf && c < d) ? omg[(size_t)f * d + c] : 0.f;
  __syncthreads();
  float acc[PREP_F];
#pragma unroll
  for (int f = 0; f < PREP_F; ++f) acc[f] = 0.f;
  if (c < d) {
    int l = 0;
    for (; l + 8 <= d; l += 8) {
      float bv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) bv[i] = Bm[(l + i) * d + c];
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int f = 0; f < PREP_F; ++f) acc[f] += om[f][l + i] * bv[i];
    }
    for (; l < d; ++l) {
      const float bv = Bm[l * d + c];
#pragma unroll
      for (int f = 0; f < PREP_F; ++f) acc[f] += om[f][l] * bv;
    }
#pragma unroll
    for (int f = 0; f < PREP_F; ++f)
      if (f < nf) {
        const float v = acc[f] * kLog2e;
        W[(o + f) * d + c] = v;
      }
  }
  if (split.img != nullptr && c < 32 * split.steps) {      // (zero past the features and past the row)
    const size_t base = ((size_t)pg * 2 + side) * split.tiles * split.steps * 3 * 512;
#pragma unroll
    for (int f = 0; f < PREP_F; ++f) {
      const int m = m0 + f, tile = m >> 4, i = m & 15;
      const float v = acc[f] * kLog2e * split.scale;
      split3_store(split.img + base + ((size_t)tile * split.steps + (c >> 5)) * 3 * 512 + ((c & 31) / 8 * 16 + i) * 8 + (c & 7), 512, v);
      if (split.img_t != nullptr)
        split3_store(split.img_t + base + ((size_t)(tile >> 1) * 2 * split.steps + (c >> 4)) * 3 * 512 + (i / 4 * 16 + (c & 15)) * 8 +
                         4 * (tile & 1) + (i & 3), 512, v);
    }
  }
  if (c < nf) {
    const float* A = th + FS_THETA_HEADER_;
    float q = 0.f;
#pragma unroll 8
    for (int l = 0; l < d; ++l) q += A[l] * om[c][l] * om[c][l];
    bias[o + c] = kLog2e * (q + th[0] - 0.5f * logf((float)M));
  }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------------------------------
// Materialised features (Section 2.1, rows of P or S).  grid (ceil(n/32)), dynamic LDS.
// ---------------------------------------------------------------------------------------------------
template <int WD>
__global__ void __launch_bounds__(NT) k_gen_features(TensorDev X, int n, int d, float scale, float alpha,
                                                     const float* W, const float* bias, const float* theta,
                                                     long long c_offset, int M, float* out, float* row_logscale) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1;
  float* Xs = smem;
  float* Ws = Xs + TR * ld;
  float* bias_s = Ws + MB * ld;
  float* rterm = bias_s + MB;
  uint32_t* rowmax_u = (uint32_t*)(rterm + TR);
  const int row0 = blockIdx.x * TR;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const float* Cmat = (((int)theta[2]) & 1) ? nullptr : theta + c_offset;

  load_rows<WD>(Xs, ld, X, 0, row0, n, d, dpad, scale);
  __syncthreads();
  row_terms(rterm, Xs, ld, d, Cmat, alpha);
  __syncthreads();
  if (row_logscale != nullptr) {
    rowmax_pass<WD>(rowmax_u, Xs, Ws, bias_s, ld, W, bias, M, d, dpad);
    if (threadIdx.x < TR && row0 + threadIdx.x < n)
      row_logscale[row0 + threadIdx.x] = (ordered_to_float(rowmax_u[threadIdx.x]) + rterm[threadIdx.x]) * kLn2;
  }
  for (int m0 = 0; m0 < M; m0 += MB) {
    __syncthreads();
    load_wblock<WD>(Ws, bias_s, ld, W, bias, m0, M, d, dpad);
    __syncthreads();
    const f32x4 acc = proj_tile(Xs, Ws, ld, dpad);
    const int f = (w & 1) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (w >> 1) * 16 + 4 * (lane >> 4) + r;
      float e = acc[r] + bias_s[f];
      e = (row_logscale != nullptr) ? e - ordered_to_float(rowmax_u[row]) : e + rterm[row];
      if (row0 + row < n && m0 + f < M) out[(size_t)(row0 + row) * M + m0 + f] = fast_exp2(e);
    }
  }
}

// Sum over the segments, result in segment 0's slot.  block (64, 4): 64 consecutive elements, four interleaved groups of
// segments that are added up through LDS.
__global__ void __launch_bounds__(256) k_gen_reduce(float* Tpart, int nseg, size_t per_state, size_t total) {
  __shared__ float part[4][64];
  const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
  const int grp = threadIdx.y;
  const bool live = i < total;
  const size_t bh = live ? i / per_state : 0, e = live ? i - bh * per_state : 0;
  float* p = Tpart + bh * nseg * per_state + e;
  float run = 0.f;
  if (live)
    for (int s = grp; s < nseg; s += 4) run += p[(size_t)s * per_state];
  part[grp][threadIdx.x] = run;
  __syncthreads();
  if (live && grp == 0) p[0] = (part[0][threadIdx.x] + part[1][threadIdx.x]) + (part[2][threadIdx.x] + part[3][threadIdx.x]);
}

// Exclusive prefix (step = 1) or suffix (step = -1) over the segments, in place; four numbers per thread (a state's rows are
// multiples of 16 numbers).  Bound by memory as soon as the loads are in flight: eight segments' are requested before the first
// store (one at a time, a number per thread, the walk over the segments is a chain of latencies: f32 B2 H4
// L4096 d64 M256 13.3 -> 8.2 us, bf16 B1 H16 L4096 d128 M512 72 -> 46 us, 142 MB).
// n4, total4: 16-byte pieces of a state and of all sequences' states.
__global__ void __launch_bounds__(64) k_gen_scan(float* Tpart, int nseg, size_t n4, size_t total4, int step) {
  const size_t i = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (i >= total4) return;
  const size_t bh = i / n4, e = i - bh * n4;
  f32x4* p = (f32x4*)Tpart + bh * nseg * n4 + e + (step < 0 ? (size_t)(nseg - 1) * n4 : 0);
  const ptrdiff_t stride = step * (ptrdiff_t)n4;
  constexpr int BATCH = 8;
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < nseg; s += BATCH) {
    f32x4 v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) v[j] = p[min(s + j, nseg - 1) * stride];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      if (s + j < nseg) p[(s + j) * stride] = run;
      run += v[j];
    }
  }
}

// Normalise (attention) or rescale (operator) an accumulated 32 x ldt tile held in LDS and store it.  Attention
// rows whose normaliser is not positive are written as zeros and, with a counter, counted (once per row).
template <int TH = NT>
__device__ void store_result(const float* Os, int ldo, const TensorDev& Y, long long ybase, int row0, int nrows,
                             int nv, int matvec, const float* row_log2scale, unsigned* flushed = nullptr) {
  for (int idx = threadIdx.x; idx < TR * nv; idx += TH) {
    const int r = idx / nv, c = idx - r * nv;
    if (row0 + r >= nrows) continue;
    float v = Os[r * ldo + c];
    if (matvec) v *= fast_exp2(row_log2scale[r]);
    else {
      const float den = Os[r * ldo + nv];
      v = den > 0.f ? v / den : 0.f;
      if (flushed != nullptr && c == 0 && !(den > 0.f)) atomicAdd(flushed, 1u);
    }
    store_elem(Y, ybase + (long long)(row0 + r) * Y.sl + c, v);
  }
}

// ---------------------------------------------------------------------------------------------------
// Query side of the non-causal contraction (Section 2.1, P (S^T C); Section 2.2 for the row normalisation).
// grid (ceil(Lq/32), B*H).  T: [bh][M][ldt] with stride state_stride between (b,h).
// ---------------------------------------------------------------------------------------------------
template <int WD>
__global__ void __launch_bounds__(NT) k_gen_apply(GenSide qs, int Lq, int H, int M, int d, int nv, int ldt,
                                                  const float* T, size_t state_stride, const uint32_t* kmax_u,
                                                  int matvec, TensorDev Y, float* den_out, float* shift_out,
                                                  unsigned* flushed) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1, ldts = ldt + 1, lds = MB + 1;
  float* Xs = smem;
  float* Ws = Xs + TR * ld;
  float* Ts = Ws + MB * ld;          // also reused as the output tile (32 x ldts)
  float* Ps = Ts + MB * ldts;
  float* bias_s = Ps + TR * lds;
  float* rterm = bias_s + MB;
  float* rscale = rterm + TR;
  uint32_t* rowmax_u = (uint32_t*)(rscale + TR);
  const int bh = blockIdx.y, b = bh / H, h = bh % H, row0 = blockIdx.x * TR;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int pg = group_of(qs.pgroups, b, h, H);
  const float* W = qs.W + ((size_t)pg * 2) * M * d;
  const float* bias = qs.bias + ((size_t)pg * 2) * M;
  const float* Cmat = side_cmat(qs, b, h, H);
  const float* Tb = T + (size_t)bh * state_stride;
  const int nvt = ldt / 16, ntiles = 2 * nvt;

  load_rows<WD>(Xs, ld, qs.X, b * qs.X.sb + h * qs.X.sh, row0, Lq, d, dpad, qs.scale);
  __syncthreads();
  // (the query row terms matter in operator mode only: in attention they cancel in the normalisation)
  if (matvec) row_terms(rterm, Xs, ld, d, Cmat, qs.alpha);
  else if (threadIdx.x < TR) rterm[threadIdx.x] = 0.f;
  rowmax_pass<WD>(rowmax_u, Xs, Ws, bias_s, ld, W, bias, M, d, dpad);
  // operator mode multiplies the shifts back: exp2(rowmax + rterm + kmax)
  if (threadIdx.x < TR)
    rscale[threadIdx.x] = ordered_to_float(rowmax_u[threadIdx.x]) + rterm[threadIdx.x] + ordered_to_float(kmax_u[bh]);

  f32x4 acc[ACC_V<WD, 4>];
#pragma unroll
  for (int t = 0; t < ACC_V<WD, 4>; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the projection block and the state block of the next step are fetched while the current step computes
  WRegs<WD, NT> wr;
  ValTile<WD, NT> tr;
  wblock_fetch(wr, W, bias, 0, M, d);
  sblock_fetch(tr, Tb, 0, M, ldt);
  for (int m0 = 0; m0 < M; m0 += MB) {
    __syncthreads();
    wblock_put(wr, Ws, bias_s, ld, m0, M, d, dpad);
    sblock_put(tr, Ts, ldts, m0, M, ldt);
    __syncthreads();
    if (m0 + MB < M) {
      wblock_fetch(wr, W, bias, m0 + MB, M, d);
      sblock_fetch(tr, Tb, m0 + MB, M, ldt);
    }
    const f32x4 e = proj_tile(Xs, Ws, ld, dpad);
    const int f = (w & 1) * 16 + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (w >> 1) * 16 + 4 * (lane >> 4) + r;
      Ps[row * lds + f] = (m0 + f < M) ? fast_exp2(e[r] + bias_s[f] - ordered_to_float(rowmax_u[row])) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 4>; ++tl) {
      const int t = w + 4 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
        const float* ap = Ps + (rt * 16 + (lane & 15)) * lds + (lane >> 4);    // A[i][k=m] = Ps[i][m]
        const float* bp = Ts + (lane >> 4) * ldts + vt * 16 + (lane & 15);     // B[k=m][n=v] = Ts[m][v]
        acc[tl] = mfma_chain(ap, 1, bp, ldts, MB, acc[tl]);
      }
    }
  }
  __syncthreads();
  float* Os = Ts;
#pragma unroll
  for (int tl = 0; tl < ACC_V<WD, 4>; ++tl) {
    const int t = w + 4 * tl;
    if (t < ntiles) {
      const int rt = t & 1, vt = t >> 1;
#pragma unroll
      for (int r = 0; r < 4; ++r) Os[(rt * 16 + 4 * (lane >> 4) + r) * ldts + vt * 16 + (lane & 15)] = acc[tl][r];
    }
  }
  __syncthreads();
  store_result(Os, ldts, Y, b * Y.sb + h * Y.sh, row0, Lq, nv, matvec, rscale, flushed);
  // for the backward pass: the (shifted) denominators and the shifts themselves, so that it rebuilds the same features
  if (den_out != nullptr && threadIdx.x < TR && row0 + threadIdx.x < Lq) {
    den_out[(size_t)bh * Lq + row0 + threadIdx.x] = Os[threadIdx.x * ldts + nv];
    shift_out[(size_t)bh * Lq + row0 + threadIdx.x] = ordered_to_float(rowmax_u[threadIdx.x]);
  }
}

// ---------------------------------------------------------------------------------------------------
// Causal contraction over one segment of one sequence, 32 rows per step, running state in global memory
// (initialised with the exclusive prefix of the segment states).  For each step:
//   Y_c = (tril(P_c S_c^T) [V_c 1] + P_c T_prev) normalised by its last column;  T += S_c^T [V_c 1].
// grid (nseg, B*H).
// ---------------------------------------------------------------------------------------------------
// (WD = 1: 129 registers by the compiler's own choice, one too many for two workgroups per CU; held to 128 without spills,
// 2048 sequences of 128 at d 8 248 -> 175 us.  The backward kernels would spill 41 and 62 and get slower.)
template <int WD>
__global__ void __launch_bounds__(NTC, WD == 1 ? 4 : 2) k_gen_causal(GenSide qs, GenSide ks, TensorDev V, int L, int H, int M, int d,
                                                   int nv, int ldt, int rows_per_seg, int nseg,
                                                   const uint32_t* kmax_u, float* Tstate, TensorDev Y, float* den_out,
                                                   float* shift_out, unsigned* flushed) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1, ldv = ldt + 1, lds = MB + 1;
  float* Qs = smem;
  float* Ks = Qs + TR * ld;
  float* Ws = Ks + TR * ld;
  float* Ws2 = Ws + MB * ld;          // Ws, bias_s: query side, Ws2, bias2_s: key side
  float* Vs = Ws2 + MB * ld;
  float* Ts = Vs + TR * ldv;          // state block, later the output tile
  float* Ps = Ts + MB * ldv;
  float* Ss = Ps + TR * lds;
  float* As = Ss + TR * lds;
  float* bias_s = As + TR * lds;
  float* bias2_s = bias_s + MB;
  float* rterm = bias2_s + MB;
  uint32_t* rowmax_u = (uint32_t*)(rterm + TR);
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, w4 = w & 3, half = w >> 2;
  const int pgq = group_of(qs.pgroups, b, h, H);
  const float* W1 = qs.W + ((size_t)pgq * 2) * M * d;
  const float* bias1 = qs.bias + ((size_t)pgq * 2) * M;
  const float* W2 = ks.W + ((size_t)pgq * 2 + 1) * M * d;
  const float* bias2 = ks.bias + ((size_t)pgq * 2 + 1) * M;
  const float c = ordered_to_float(kmax_u[bh]);
  float* Tg = Tstate + ((size_t)bh * nseg + seg) * M * ldt;
  const int nvt = ldt / 16, ntiles = 2 * nvt;
  const long long qbase = b * qs.X.sb + h * qs.X.sh, kbase = b * ks.X.sb + h * ks.X.sh;

  const int row_end = min(L, (seg + 1) * rows_per_seg);
  for (int row0 = seg * rows_per_seg; row0 < row_end; row0 += TR) {
    __syncthreads();
    load_rows<WD, NTC>(Qs, ld, qs.X, qbase, row0, row_end, d, dpad, qs.scale);
    load_rows<WD, NTC>(Ks, ld, ks.X, kbase, row0, row_end, d, dpad, ks.scale);
    load_values<WD, NTC>(Vs, ldv, V, b * V.sb + h * V.sh, row0, row_end, nv, ldt, 1);
    __syncthreads();
    row_terms_of(rterm, ks, bh, L, row0, row_end);
    rowmax_pass2<WD>(rowmax_u, Qs, Ws, Ws2, bias_s, bias2_s, ld, W1, bias1, M, d, dpad);

    f32x4 acc[ACC_V<WD, 8>];
#pragma unroll
    for (int t = 0; t < ACC_V<WD, 8>; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};          // scores tile (query tile w>>1, key tile w&1)
    // the three blocks of the next step are fetched while the current one computes (rows of the state that this step
    // writes are not among them)
    WRegs<WD, NTC> wa, wb;
    ValTile<WD, NTC> tr;
    wblock_fetch(wa, W1, bias1, 0, M, d);
    sblock_fetch(tr, Tg, 0, M, ldt);
    wblock_fetch(wb, W2, bias2, 0, M, d);
    for (int m0 = 0; m0 < M; m0 += MB) {
      const int f = (w4 & 1) * 16 + (lane & 15);
      __syncthreads();
      wblock_put(wa, Ws, bias_s, ld, m0, M, d, dpad);
      wblock_put(wb, Ws2, bias2_s, ld, m0, M, d, dpad);
      sblock_put(tr, Ts, ldv, m0, M, ldt);
      __syncthreads();
      if (m0 + MB < M) {
        wblock_fetch(wa, W1, bias1, m0 + MB, M, d);
        wblock_fetch(wb, W2, bias2, m0 + MB, M, d);
        sblock_fetch(tr, Tg, m0 + MB, M, ldt);
      }
      if (half == 0) {
        const f32x4 e = proj_tile(Qs, Ws, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          Ps[row * lds + f] = (m0 + f < M) ? fast_exp2(e[r] + bias_s[f] - ordered_to_float(rowmax_u[row])) : 0.f;
        }
      }
      else {
        const f32x4 e = proj_tile(Ks, Ws2, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          Ss[row * lds + f] = (m0 + f < M) ? fast_exp2(e[r] + bias2_s[f] + rterm[row] - c) : 0.f;
        }
      }
      __syncthreads();
      if (half == 1) {   // scores: A[i][k=m] = Ps[i][m], B[k=m][n=j] = Ss[j][m]
        const float* ap = Ps + ((w4 >> 1) * 16 + (lane & 15)) * lds + (lane >> 4);
        const float* bp = Ss + ((w4 & 1) * 16 + (lane & 15)) * lds + (lane >> 4);
        sc = mfma_chain(ap, 1, bp, 1, MB, sc);
      }
#pragma unroll
      for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
        const int t = w + 8 * tl;
        if (t < ntiles) {
          const int rt = t & 1, vt = t >> 1;
          {   // inter-chunk term with the state before this step
            const float* ap = Ps + (rt * 16 + (lane & 15)) * lds + (lane >> 4);
            const float* bp = Ts + (lane >> 4) * ldv + vt * 16 + (lane & 15);
            acc[tl] = mfma_chain(ap, 1, bp, ldv, MB, acc[tl]);
          }
          {   // state update for feature tile rt: T[m][v] += sum_j Ss[j][m] Vs[j][v]
            f32x4 up = {0.f, 0.f, 0.f, 0.f};
            const float* ap = Ss + (lane >> 4) * lds + rt * 16 + (lane & 15);
            const float* bp = Vs + (lane >> 4) * ldv + vt * 16 + (lane & 15);
            up = mfma_chain(ap, lds, bp, ldv, TR, up);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int mb = rt * 16 + 4 * (lane >> 4) + r;
              if (m0 + mb < M) Tg[(size_t)(m0 + mb) * ldt + vt * 16 + (lane & 15)] = Ts[mb * ldv + vt * 16 + (lane & 15)] + up[r];
            }
          }
        }
      }
    }
    // causal mask inside the step (key j <= query i), then the intra-chunk product
    if (half == 1)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = (w4 >> 1) * 16 + 4 * (lane >> 4) + r, j = (w4 & 1) * 16 + (lane & 15);
      As[i * lds + j] = (j <= i) ? sc[r] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
        const float* ap = As + (rt * 16 + (lane & 15)) * lds + (lane >> 4);
        const float* bp = Vs + (lane >> 4) * ldv + vt * 16 + (lane & 15);
        acc[tl] = mfma_chain(ap, 1, bp, ldv, TR, acc[tl]);
      }
    }
    __syncthreads();
    float* Os = Ts;
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) Os[(rt * 16 + 4 * (lane >> 4) + r) * ldv + vt * 16 + (lane & 15)] = acc[tl][r];
      }
    }
    __syncthreads();
    store_result<NTC>(Os, ldv, Y, b * Y.sb + h * Y.sh, row0, row_end, nv, 0, nullptr, flushed);
    if (den_out != nullptr && threadIdx.x < TR && row0 + threadIdx.x < row_end) {   // for the backward pass
      den_out[(size_t)bh * L + row0 + threadIdx.x] = Os[threadIdx.x * ldv + nv];
      shift_out[(size_t)bh * L + row0 + threadIdx.x] = ordered_to_float(rowmax_u[threadIdx.x]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Statistics scan for the fits: per (b,h) and row chunk, sum x and sum x x^T of the scaled rows (fp32 MFMA,
// fp32 partials), then a second kernel adds the partials of all (b,h) of a group in fp64.
// grid (nchunks, B*H, 2 tensors).  part: [2][B*H][nchunks][d*d + d].
// ---------------------------------------------------------------------------------------------------
template <int WD>
__global__ void __launch_bounds__(NT) k_stats_partial(TensorDev X, TensorDev Yt, int Lx, int Ly, int H, int d,
                                                      float scale, int rows_per_chunk, int nchunks, float* part) {
  extern __shared__ float smem[];
  const int dpad = (d + 15) & ~15, ld = dpad + 1;
  float* Xs = smem;
  const int which = blockIdx.z, bh = blockIdx.y, b = bh / H, h = bh % H, chunk = blockIdx.x;
  const TensorDev& T = which ? Yt : X;
  const int L = which ? Ly : Lx;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nt = dpad / 16, ntiles = nt * nt;      // <= 4 WD^2 tiles
  f32x4 acc[WD * WD];
#pragma unroll
  for (int t = 0; t < WD * WD; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float colsum = 0.f;
  const int row_end = min(L, (chunk + 1) * rows_per_chunk);
  for (int row0 = chunk * rows_per_chunk; row0 < row_end; row0 += TR) {
    __syncthreads();
    load_rows<WD>(Xs, ld, T, b * T.sb + h * T.sh, row0, row_end, d, dpad, scale);
    __syncthreads();
    if (threadIdx.x < d)
      for (int r = 0; r < TR; ++r) colsum += Xs[r * ld + threadIdx.x];
#pragma unroll
    for (int tl = 0; tl < WD * WD; ++tl) {
      const int t = w + 4 * tl;
      if (t < ntiles) {
        const int at = t / nt, bt = t - at * nt;
        const float* ap = Xs + (lane >> 4) * ld + at * 16 + (lane & 15);      // A[i=a][k=row] = Xs[row][a]
        const float* bp = Xs + (lane >> 4) * ld + bt * 16 + (lane & 15);
        for (int k = 0; k < TR; k += 4) acc[tl] = mfma4(ap[k * ld], bp[k * ld], acc[tl]);
      }
    }
  }
  float* out = part + (((size_t)which * gridDim.y + bh) * nchunks + chunk) * ((size_t)d * d + d);
#pragma unroll
  for (int tl = 0; tl < WD * WD; ++tl) {
    const int t = w + 4 * tl;
    if (t < ntiles) {
      const int at = t / nt, bt = t - at * nt;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = at * 16 + 4 * (lane >> 4) + r, bb = bt * 16 + (lane & 15);
        if (a < d && bb < d) out[(size_t)a * d + bb] = acc[tl][r];
      }
    }
  }
  if (threadIdx.x < d) out[(size_t)d * d + threadIdx.x] = colsum;
}

// stats: [groups][2][d*d + d] doubles: mean x x^T then mean x, for X (0) and Y (1).
__global__ void k_stats_final(const float* part, int B, int H, int nchunks, int d, int groups, int Lx, int Ly,
                              double* stats) {
  const size_t per = (size_t)d * d + d;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)groups * 2 * per) return;
  const int g = (int)(i / (2 * per));
  const int which = (int)((i / per) & 1);
  const size_t e = i % per;
  // the parts of the group's sequences: pairs (b, h) from `first` on, `step` apart
  const int first = groups == 1 ? 0 : g, step = groups == 1 ? 1 : H, count = groups == 1 ? B * H : (groups == H ? B : 1);
  const float* p = part + ((size_t)which * B * H + first) * nchunks * per + e;
  const long long rows = (long long)count * (which ? Ly : Lx);
  // Sixteen parts' loads are in flight together: a thread is one chain of memory latencies, which is what this kernel takes,
  // with the scalar work between the requests beside it: a clamp, a select and a 64-bit product per part took longer than the
  // loads.  So the pointer only advances, parts that lie next to each other (one group, or one per sequence) by constants, and
  // the last, shorter pass alone is clamped.  us, four chunks of one sequence at a time -> sixteen with a product each -> this:
  // 8 heads of 8 sequences, d = 64: 11.3 -> 8.7 -> 5.9; d = 128: 15.4 -> 16.6 -> 13.1; one group, d = 128: 50.5 -> 53.3 -> 19.5;
  // one sequence of 20000, d = 128: 28.0 -> 34.5 -> 13.4; eight of 1000, d = 8: 8.2 -> 4.4 -> 3.4.
  const int total = count * nchunks;
  double s4[4] = {0.0, 0.0, 0.0, 0.0};
  const size_t skip = count == 1 ? 0 : (size_t)(step - 1) * nchunks * per;  // between two of the group's sequences
  int done = 0, c = 0;
  for (; done + 16 <= total; done += 16) {
    float v[16];
    if (skip == 0) {
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = p[u * per];
      p += 16 * per;
    } else {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        v[u] = *p;
        const bool wrap = ++c == nchunks;
        p += wrap ? per + skip : per;
        c = wrap ? 0 : c;
      }
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) s4[u & 3] += (double)v[u];
  }
  if (done < total) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      v[u] = *p;
      const bool wrap = ++c == nchunks;
      p += done + u + 1 < total ? (wrap ? per + skip : per) : 0;
      c = wrap ? 0 : c;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) s4[u & 3] += done + u < total ? (double)v[u] : 0.0;
  }
  const double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
  stats[i] = s / (double)rows;
}

// ---------------------------------------------------------------------------------------------------
// Backward pass of non-causal attention (chain rule on Section 2.2's attention equation with K_hat = P S^T;
// theta and omega are constants).  With V1 = [V 1], T = S^T V1, Yhat = P T:
//   G1_i = [dY_i / den_i, -(dY_i . Y_i) / den_i],  dP = G1 T^T,  R = P^T G1,  dV1 = S R,  dS = V1 R^T,
//   dE = F * dF  (F = P or S),   dx = dE W + rowsum(dE) (C + C^T) x,   d(input) = qk_scale dx.
// The exponent shifts of the forward pass (one per query row, one per sequence for the keys) cancel in every
// product above, so the kernels work on the shifted quantities throughout.
// ---------------------------------------------------------------------------------------------------

// In place: row i of `buf` ([bh][L][ldt], holding Y_i in its first nv columns) becomes G1_i (zero padded).
// Sixteen lanes per row (consecutive columns: coalesced), 16 rows per workgroup of 256 threads.
// SPLIT (behind k_split_walk): dY is divided by 2^exps, normalisers have a factor 2^24, which is taken out here, and the largest |G1| of the
// workgroup's rows is left in `largest`; grid (ceil(L / GMAX_ROWS), B H).  Else grid ceil(rows / 16).
template <bool SPLIT>
__global__ void __launch_bounds__(256) k_bwd_ghat(TensorDev dY, float* buf, const float* den, const int* exps, float* largest, int L, int H, int nv,
                                                  int ldt, size_t rows) {
  const size_t i = (size_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int l = threadIdx.x & 15;
  const bool live = i < rows;
  const size_t ii = (live ? i : 0) + (SPLIT ? (size_t)blockIdx.y * L : 0);
  const int bh = (int)(ii / L), row = (int)(ii - (size_t)bh * L), b = bh / H, h = bh % H;
  float* g = buf + ii * ldt;
  const float dn = den[ii];
  const int e = SPLIT ? -exps[bh] : 0, late = SPLIT && dn < 1.f ? 24 : 0;
  const float inv = dn > 0.f ? ldexpf(1.f / dn, SPLIT ? 24 - late : 0) : 0.f;      // (neither it nor its product with dY vanishes)
  const long long base = b * dY.sb + h * dY.sh + (long long)row * dY.sl;
  const auto dy = [&](int c) { return SPLIT ? ldexpf(load_elem(dY, base + c), e) : load_elem(dY, base + c); };
  float dot = 0.f;
  for (int c = l; c < nv; c += 16) dot += dy(c) * g[c];
  dot += __shfl_xor(dot, 1);
  dot += __shfl_xor(dot, 2);
  dot += __shfl_xor(dot, 4);
  dot += __shfl_xor(dot, 8);
  if (!SPLIT && !live) return;
  float most = 0.f;
  if (live)
    for (int c = l; c < ldt; c += 16) {
      float v = c < nv ? dy(c) * inv : (c == nv ? -dot * inv : 0.f);
      if (SPLIT) {
        v = ldexpf(v, late);
        if (fabsf(v) < INFINITY) most = fmaxf(most, fabsf(v));
      }
      g[c] = v;
    }
  if constexpr (SPLIT) {
    __shared__ float red[4];
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) most = fmaxf(most, __shfl_xor(most, s));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = most;
    __syncthreads();
    if (threadIdx.x == 0) largest[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  }
}

// One side of the backward pass for a tile of 32 rows.  F = this side's features (query side: per-row shifts from
// the forward pass, no row term; key side: the sequence's key shift and the row term), A = the rows' "left" factor
// (query side: G1; key side: V1), St = the state it is contracted with (query side: T; key side: R).
//   out1 = F St          (key side only: its first nv columns are dV)
//   dF   = A St^T,  dE = F * dF,  grad = scale (dE W / log2e + rowsum(dE) (C + C^T) x)
// grid (ceil(L/32), B*H).
template <int WD>
__global__ void __launch_bounds__(NT) k_gen_bwd_side(GenSide sd, int side, TensorDev A, int a_cols, int append_ones, int L,
                                                     int H, int M, int d, int nv, int ldt, const float* St,
                                                     size_t state_stride, const uint32_t* kmax_u, const float* row_shift,
                                                     TensorDev out1, int want_out1, TensorDev grad) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1, ldts = ldt + 1, lds = MB + 1;
  float* Xs = smem;
  float* Ws = Xs + TR * ld;          // also the gradient tile (32 x ld) at the end
  float* As = Ws + MB * ld;
  float* Sts = As + TR * ldts;       // also the out1 tile (32 x ldts) at the end
  float* Fs = Sts + MB * ldts;
  float* dEs = Fs + TR * lds;
  float* bias_s = dEs + TR * lds;
  float* rterm = bias_s + MB;        // what is added to the exponent per row (row term - shift)
  float* rsum = rterm + TR;
  const int bh = blockIdx.y, b = bh / H, h = bh % H, row0 = blockIdx.x * TR;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int pg = group_of(sd.pgroups, b, h, H);
  const float* W = sd.W + ((size_t)pg * 2 + side) * M * d;
  const float* bias = sd.bias + ((size_t)pg * 2 + side) * M;
  const float* Cmat = side_cmat(sd, b, h, H);
  const float* Sb = St + (size_t)bh * state_stride;
  const int nvt = ldt / 16, ntiles = 2 * nvt, nct = dpad / 16 + ((dpad & 15) ? 1 : 0), ngt = 2 * nct;

  load_rows<WD>(Xs, ld, sd.X, b * sd.X.sb + h * sd.X.sh, row0, L, d, dpad, sd.scale);
  load_values<WD>(As, ldts, A, b * A.sb + h * A.sh, row0, L, a_cols, ldt, append_ones);
  __syncthreads();
  if (side == 1) {
    row_terms_of(rterm, sd, bh, L, row0, L);
    __syncthreads();
    if (threadIdx.x < TR) rterm[threadIdx.x] -= ordered_to_float(kmax_u[bh]);
  } else if (threadIdx.x < TR) {
    rterm[threadIdx.x] = row0 + threadIdx.x < L ? -row_shift[(size_t)bh * L + row0 + threadIdx.x] : 0.f;
  }

  f32x4 acc_o[ACC_V<WD, 4>], acc_g[ACC_D<WD, 4>];
#pragma unroll
  for (int t = 0; t < ACC_V<WD, 4>; ++t) acc_o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < ACC_D<WD, 4>; ++t) acc_g[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rs_part = 0.f;               // thread (row = tid / 8, part = tid % 8): its share of rowsum(dE)

  WRegs<WD, NT> wr;                          // the next step's blocks, fetched while the current one computes
  ValTile<WD, NT> tr;
  wblock_fetch(wr, W, bias, 0, M, d);
  sblock_fetch(tr, Sb, 0, M, ldt);
  for (int m0 = 0; m0 < M; m0 += MB) {
    __syncthreads();
    wblock_put(wr, Ws, bias_s, ld, m0, M, d, dpad);
    sblock_put(tr, Sts, ldts, m0, M, ldt);
    __syncthreads();
    if (m0 + MB < M) {
      wblock_fetch(wr, W, bias, m0 + MB, M, d);
      sblock_fetch(tr, Sb, m0 + MB, M, ldt);
    }
    const f32x4 e = proj_tile(Xs, Ws, ld, dpad);
    const int f = (w & 1) * 16 + (lane & 15);
    float fv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (w >> 1) * 16 + 4 * (lane >> 4) + r;
      fv[r] = (m0 + f < M && row0 + row < L) ? fast_exp2(e[r] + bias_s[f] + rterm[row]) : 0.f;
      Fs[row * lds + f] = fv[r];
    }
    // dF tile of this wave (rows (w>>1)*16.., features (w&1)*16..): A[i][k=v] = As[i][v], B[k=v][n=m] = Sts[m][v]
    {
      const float* ap = As + ((w >> 1) * 16 + (lane & 15)) * ldts + (lane >> 4);
      const float* bp = Sts + ((w & 1) * 16 + (lane & 15)) * ldts + (lane >> 4);
      f32x4 df = {0.f, 0.f, 0.f, 0.f};
      df = mfma_chain(ap, 1, bp, 1, ldt, df);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = (w >> 1) * 16 + 4 * (lane >> 4) + r;
        dEs[row * lds + f] = fv[r] * df[r];
      }
    }
    __syncthreads();
    if (want_out1) {
#pragma unroll
      for (int tl = 0; tl < ACC_V<WD, 4>; ++tl) {
        const int t = w + 4 * tl;
        if (t < ntiles) {
          const int rt = t & 1, vt = t >> 1;
          const float* ap = Fs + (rt * 16 + (lane & 15)) * lds + (lane >> 4);     // A[i][k=m] = Fs[i][m]
          const float* bp = Sts + (lane >> 4) * ldts + vt * 16 + (lane & 15);     // B[k=m][n=v] = Sts[m][v]
          acc_o[tl] = mfma_chain(ap, 1, bp, ldts, MB, acc_o[tl]);
        }
      }
    }
#pragma unroll
    for (int tl = 0; tl < ACC_D<WD, 4>; ++tl) {
      const int t = w + 4 * tl;
      if (t < ngt) {
        const int rt = t & 1, ct = t >> 1;
        const float* ap = dEs + (rt * 16 + (lane & 15)) * lds + (lane >> 4);      // A[i][k=m] = dEs[i][m]
        const float* bp = Ws + (lane >> 4) * ld + min(ct * 16 + (lane & 15), dpad - 1);   // B[k=m][n=c] = Ws[m][c]; columns past dpad are dropped below
        acc_g[tl] = mfma_chain(ap, 1, bp, ld, MB, acc_g[tl]);
      }
    }
    {
      const int row = threadIdx.x >> 3, part = threadIdx.x & 7;
#pragma unroll
      for (int q = 0; q < 4; ++q) rs_part += dEs[row * lds + part * 4 + q];
    }
  }
  __syncthreads();
  // tiles back to LDS
  float* Gs = Ws;
  float* Os = Sts;
#pragma unroll
  for (int tl = 0; tl < ACC_D<WD, 4>; ++tl) {
    const int t = w + 4 * tl;
    if (t < ngt) {
      const int rt = t & 1, ct = t >> 1, col = ct * 16 + (lane & 15);
      if (col < dpad) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Gs[(rt * 16 + 4 * (lane >> 4) + r) * ld + col] = acc_g[tl][r];
      }
    }
  }
  if (want_out1) {
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 4>; ++tl) {
      const int t = w + 4 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) Os[(rt * 16 + 4 * (lane >> 4) + r) * ldts + vt * 16 + (lane & 15)] = acc_o[tl][r];
      }
    }
  }
  rs_part += __shfl_xor(rs_part, 1);
  rs_part += __shfl_xor(rs_part, 2);
  rs_part += __shfl_xor(rs_part, 4);
  if ((threadIdx.x & 7) == 0) rsum[threadIdx.x >> 3] = rs_part;
  __syncthreads();
  // grad[i][c] = scale (Gs[i][c] / log2e + rsum_i ((C + C^T) x_i)[c]);  C = -I/2: (C + C^T) x = -x
  for (int idx = threadIdx.x; idx < TR * d; idx += NT) {
    const int r = idx / d, c = idx - r * d;
    if (row0 + r >= L) continue;
    float cx;
    if (Cmat == nullptr) cx = -Xs[r * ld + c];
    else {
      cx = sym_row_dot(Cmat, d, c, Xs + r * ld);
    }
    const float v = sd.scale * (Gs[r * ld + c] * kLn2 + rsum[r] * (cx + 2.f * sd.alpha * Xs[r * ld + c]));
    store_elem(grad, b * grad.sb + h * grad.sh + (long long)(row0 + r) * grad.sl + c, v);
  }
  if (want_out1) {
    for (int idx = threadIdx.x; idx < TR * nv; idx += NT) {
      const int r = idx / nv, c = idx - r * nv;
      if (row0 + r < L) store_elem(out1, b * out1.sb + h * out1.sh + (long long)(row0 + r) * out1.sl + c, Os[r * ldts + c]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Backward pass of causal attention.  With T_i the prefix state (keys j <= i) and R_j the suffix sum
// sum_{i >= j} P_i^T G1_i, per chunk c of 32 rows (A = tril(G1_c V1_c^T), B = tril(P_c S_c^T)):
//   dP_c  = G1_c T_{c-1}^T + A S_c                 dV1_c = S_c R_{c+1} + B^T G1_c
//   dS_c  = V1_c R_{c+1}^T + A^T P_c               and dE = F * dF, dx = dE W + rowsum(dE) (C + C^T) x as above.
// The query kernel walks a segment forwards with the running prefix state (initialised with the exclusive prefix
// of the segment states), the key kernel walks it backwards with the running suffix sum (initialised with the
// exclusive suffix of the segments' P^T G1).  G1, the denominators and the query shifts come from a forward pass.
// grid (nseg, B*H) both.
// ---------------------------------------------------------------------------------------------------
struct BwdCausalSmem {
  float *Qs, *Ks, *Ws, *Ws2, *Vs, *Gs, *Ts, *Ps, *Ss, *dEs, *As, *Bs, *bias_s, *bias2_s, *rterm, *qsh, *rsum;
};
__device__ __forceinline__ BwdCausalSmem bwd_causal_carve(float* smem, int ld, int ldv, int lds) {
  BwdCausalSmem m;
  m.Qs = smem;
  m.Ks = m.Qs + TR * ld;
  m.Ws = m.Ks + TR * ld;
  m.Ws2 = m.Ws + MB * ld;              // Ws, bias_s: query side, Ws2, bias2_s: key side
  m.Vs = m.Ws2 + MB * ld;
  m.Gs = m.Vs + TR * ldv;
  m.Ts = m.Gs + TR * ldv;
  m.Ps = m.Ts + MB * ldv;
  m.Ss = m.Ps + TR * lds;
  m.dEs = m.Ss + TR * lds;
  m.As = m.dEs + TR * lds;
  m.Bs = m.As + TR * lds;
  m.bias_s = m.Bs + TR * lds;
  m.bias2_s = m.bias_s + MB;
  m.rterm = m.bias2_s + MB;
  m.qsh = m.rterm + TR;
  m.rsum = m.qsh + TR;
  return m;
}

// As[i][j] = (j <= i) ? G1_i . V1_j : 0 for the chunk's 32 x 32 (query, key) pairs; wave w owns tile (w>>1, w&1).
__device__ __forceinline__ void bwd_causal_amat(float* As, const float* Gs, const float* Vs, int ldv, int lds, int ldt) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (w >= 4) return;
  const float* ap = Gs + ((w >> 1) * 16 + (lane & 15)) * ldv + (lane >> 4);   // A[i][k=v] = Gs[i][v]
  const float* bp = Vs + ((w & 1) * 16 + (lane & 15)) * ldv + (lane >> 4);    // B[k=v][n=j] = Vs[j][v]
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  a = mfma_chain(ap, 1, bp, 1, ldt, a);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = (w >> 1) * 16 + 4 * (lane >> 4) + r, j = (w & 1) * 16 + (lane & 15);
    As[i * lds + j] = (j <= i) ? a[r] : 0.f;
  }
}

// grad rows of a 32-row tile from the accumulated dE W tile (Gsrc, stride ld), the row sums and x.
__device__ __forceinline__ void bwd_store_grad(const TensorDev& grad, long long base, int row0, int row_end, int d, int ld,
                                               const float* Gsrc, const float* rsum, const float* Xs, const float* Cmat,
                                               float scale, float alpha) {
  for (int idx = threadIdx.x; idx < TR * d; idx += NTC) {
    const int r = idx / d, c = idx - r * d;
    if (row0 + r >= row_end) continue;
    float cx;
    if (Cmat == nullptr) cx = -Xs[r * ld + c];
    else {
      cx = sym_row_dot(Cmat, d, c, Xs + r * ld);
    }
    const float v = scale * (Gsrc[r * ld + c] * kLn2 + rsum[r] * (cx + 2.f * alpha * Xs[r * ld + c]));
    store_elem(grad, base + (long long)(row0 + r) * grad.sl + c, v);
  }
}

template <int WD>
__global__ void __launch_bounds__(NTC) k_gen_bwd_causal_q(GenSide qs, GenSide ks, TensorDev V, const float* ghat, int L,
                                                         int H, int M, int d, int nv, int ldt, int rows_per_seg, int nseg,
                                                         const uint32_t* kmax_u, const float* row_shift, float* Tstate,
                                                         TensorDev dQ) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1, ldv = ldt + 1, lds = MB + 1;
  const BwdCausalSmem m = bwd_causal_carve(smem, ld, ldv, lds);
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, w4 = w & 3, half = w >> 2;
  const int pg = group_of(qs.pgroups, b, h, H);
  const float* W1 = qs.W + ((size_t)pg * 2) * M * d;
  const float* bias1 = qs.bias + ((size_t)pg * 2) * M;
  const float* W2 = ks.W + ((size_t)pg * 2 + 1) * M * d;
  const float* bias2 = ks.bias + ((size_t)pg * 2 + 1) * M;
  const float* Cmat1 = side_cmat(qs, b, h, H);
  const float c = ordered_to_float(kmax_u[bh]);
  float* Tg = Tstate + ((size_t)bh * nseg + seg) * M * ldt;
  const TensorDev G{ghat, 0, (long long)H * L * ldt, (long long)L * ldt, (long long)ldt};
  const int nvt = ldt / 16, ntiles = 2 * nvt, nct = (dpad + 15) / 16, ngt = 2 * nct;
  const long long qbase = b * qs.X.sb + h * qs.X.sh, kbase = b * ks.X.sb + h * ks.X.sh;

  const int row_end = min(L, (seg + 1) * rows_per_seg);
  for (int row0 = seg * rows_per_seg; row0 < row_end; row0 += TR) {
    __syncthreads();
    load_rows<WD, NTC>(m.Qs, ld, qs.X, qbase, row0, row_end, d, dpad, qs.scale);
    load_rows<WD, NTC>(m.Ks, ld, ks.X, kbase, row0, row_end, d, dpad, ks.scale);
    load_values<WD, NTC>(m.Vs, ldv, V, b * V.sb + h * V.sh, row0, row_end, nv, ldt, 1);
    load_values<WD, NTC>(m.Gs, ldv, G, b * G.sb + h * G.sh, row0, row_end, ldt, ldt, 0);
    if (threadIdx.x < TR) m.qsh[threadIdx.x] = row0 + threadIdx.x < row_end ? -row_shift[(size_t)bh * L + row0 + threadIdx.x] : 0.f;
    __syncthreads();
    row_terms_of(m.rterm, ks, bh, L, row0, row_end);
    bwd_causal_amat(m.As, m.Gs, m.Vs, ldv, lds, ldt);

    f32x4 acc_g[ACC_D<WD, 8>];
#pragma unroll
    for (int t = 0; t < ACC_D<WD, 8>; ++t) acc_g[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float rs_part = 0.f;
    // the three blocks of the next step are fetched while the current one computes (rows of the state that this step
    // writes are not among them)
    WRegs<WD, NTC> wa, wb;
    ValTile<WD, NTC> tr;
    wblock_fetch(wa, W2, bias2, 0, M, d);
    sblock_fetch(tr, Tg, 0, M, ldt);
    wblock_fetch(wb, W1, bias1, 0, M, d);
    for (int m0 = 0; m0 < M; m0 += MB) {
      const int f = (w4 & 1) * 16 + (lane & 15);
      __syncthreads();
      wblock_put(wa, m.Ws2, m.bias2_s, ld, m0, M, d, dpad);
      wblock_put(wb, m.Ws, m.bias_s, ld, m0, M, d, dpad);
      sblock_put(tr, m.Ts, ldv, m0, M, ldt);
      __syncthreads();
      if (m0 + MB < M) {
        wblock_fetch(wa, W2, bias2, m0 + MB, M, d);
        wblock_fetch(wb, W1, bias1, m0 + MB, M, d);
        sblock_fetch(tr, Tg, m0 + MB, M, ldt);
      }
      // waves 0 - 3: features and dP tile (rows (w4>>1)*16.., features (w4&1)*16..) = G1 T_prev^T + A S of the queries;
      // waves 4 - 7: features of the keys
      float fv[4];
      f32x4 df = {0.f, 0.f, 0.f, 0.f};
      if (half == 0) {
        const f32x4 e = proj_tile(m.Qs, m.Ws, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          fv[r] = (m0 + f < M && row0 + row < row_end) ? fast_exp2(e[r] + m.bias_s[f] + m.qsh[row]) : 0.f;
        }
        const float* ap = m.Gs + ((w4 >> 1) * 16 + (lane & 15)) * ldv + (lane >> 4);   // A[i][k=v] = Gs[i][v]
        const float* bp = m.Ts + ((w4 & 1) * 16 + (lane & 15)) * ldv + (lane >> 4);    // B[k=v][n=m] = Ts[m][v]
        df = mfma_chain(ap, 1, bp, 1, ldt, df);
      } else {
        const f32x4 e = proj_tile(m.Ks, m.Ws2, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          m.Ss[row * lds + f] = (m0 + f < M && row0 + row < row_end) ? fast_exp2(e[r] + m.bias2_s[f] + m.rterm[row] - c) : 0.f;
        }
      }
      __syncthreads();
      if (half == 0) {
        const float* ap = m.As + ((w4 >> 1) * 16 + (lane & 15)) * lds + (lane >> 4);   // A[i][k=j] = As[i][j]
        const float* bp = m.Ss + (lane >> 4) * lds + (w4 & 1) * 16 + (lane & 15);      // B[k=j][n=m] = Ss[j][m]
        df = mfma_chain(ap, 1, bp, lds, TR, df);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          m.dEs[row * lds + f] = fv[r] * df[r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int tl = 0; tl < ACC_D<WD, 8>; ++tl) {
        const int t = w + 8 * tl;
        if (t < ngt) {
          const int rt = t & 1, ct = t >> 1;
          const float* ap = m.dEs + (rt * 16 + (lane & 15)) * lds + (lane >> 4);        // A[i][k=m] = dEs[i][m]
          const float* bp = m.Ws + (lane >> 4) * ld + min(ct * 16 + (lane & 15), dpad - 1);   // (columns past dpad are dropped below)
          acc_g[tl] = mfma_chain(ap, 1, bp, ld, MB, acc_g[tl]);
        }
      }
      if (half == 0) {
        const int row = threadIdx.x >> 3, part = threadIdx.x & 7;
#pragma unroll
        for (int q = 0; q < 4; ++q) rs_part += m.dEs[row * lds + part * 4 + q];
      }
      // the state takes this chunk's keys (after its last use above): T[m][v] += sum_j Ss[j][m] Vs[j][v]
#pragma unroll
      for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
        const int t = w + 8 * tl;
        if (t < ntiles) {
          const int rt = t & 1, vt = t >> 1;
          f32x4 up = {0.f, 0.f, 0.f, 0.f};
          const float* ap = m.Ss + (lane >> 4) * lds + rt * 16 + (lane & 15);
          const float* bp = m.Vs + (lane >> 4) * ldv + vt * 16 + (lane & 15);
          up = mfma_chain(ap, lds, bp, ldv, TR, up);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int mb = rt * 16 + 4 * (lane >> 4) + r;
            if (m0 + mb < M) Tg[(size_t)(m0 + mb) * ldt + vt * 16 + (lane & 15)] = m.Ts[mb * ldv + vt * 16 + (lane & 15)] + up[r];
          }
        }
      }
    }
    __syncthreads();
    float* Gd = m.Ws;
#pragma unroll
    for (int tl = 0; tl < ACC_D<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ngt) {
        const int rt = t & 1, ct = t >> 1, col = ct * 16 + (lane & 15);
        if (col < dpad) {
#pragma unroll
          for (int r = 0; r < 4; ++r) Gd[(rt * 16 + 4 * (lane >> 4) + r) * ld + col] = acc_g[tl][r];
        }
      }
    }
    rs_part += __shfl_xor(rs_part, 1);
    rs_part += __shfl_xor(rs_part, 2);
    rs_part += __shfl_xor(rs_part, 4);
    if (half == 0 && (threadIdx.x & 7) == 0) m.rsum[threadIdx.x >> 3] = rs_part;
    __syncthreads();
    bwd_store_grad(dQ, b * dQ.sb + h * dQ.sh, row0, row_end, d, ld, Gd, m.rsum, m.Qs, Cmat1, qs.scale, 0.f);
  }
}

template <int WD>
__global__ void __launch_bounds__(NTC) k_gen_bwd_causal_k(GenSide qs, GenSide ks, TensorDev V, const float* ghat, int L,
                                                         int H, int M, int d, int nv, int ldt, int rows_per_seg, int nseg,
                                                         const uint32_t* kmax_u, const float* row_shift, float* Rstate,
                                                         TensorDev dK, TensorDev dV) {
  extern __shared__ float smem[];
  const int dpad = (d + 3) & ~3, ld = dpad + 1, ldv = ldt + 1, lds = MB + 1;
  const BwdCausalSmem m = bwd_causal_carve(smem, ld, ldv, lds);
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / H, h = bh % H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, w4 = w & 3, half = w >> 2;
  const int pg = group_of(qs.pgroups, b, h, H);
  const float* W1 = qs.W + ((size_t)pg * 2) * M * d;
  const float* bias1 = qs.bias + ((size_t)pg * 2) * M;
  const float* W2 = ks.W + ((size_t)pg * 2 + 1) * M * d;
  const float* bias2 = ks.bias + ((size_t)pg * 2 + 1) * M;
  const float* Cmat2 = side_cmat(ks, b, h, H);
  const float c = ordered_to_float(kmax_u[bh]);
  float* Rg = Rstate + ((size_t)bh * nseg + seg) * M * ldt;
  const TensorDev G{ghat, 0, (long long)H * L * ldt, (long long)L * ldt, (long long)ldt};
  const int nvt = ldt / 16, ntiles = 2 * nvt, nct = (dpad + 15) / 16, ngt = 2 * nct;
  const long long qbase = b * qs.X.sb + h * qs.X.sh, kbase = b * ks.X.sb + h * ks.X.sh;

  const int row_beg = seg * rows_per_seg, row_end = min(L, (seg + 1) * rows_per_seg);
  const int nchunk = (row_end - row_beg + TR - 1) / TR;
  for (int ch = nchunk - 1; ch >= 0; --ch) {
    const int row0 = row_beg + ch * TR;
    __syncthreads();
    load_rows<WD, NTC>(m.Qs, ld, qs.X, qbase, row0, row_end, d, dpad, qs.scale);
    load_rows<WD, NTC>(m.Ks, ld, ks.X, kbase, row0, row_end, d, dpad, ks.scale);
    load_values<WD, NTC>(m.Vs, ldv, V, b * V.sb + h * V.sh, row0, row_end, nv, ldt, 1);
    load_values<WD, NTC>(m.Gs, ldv, G, b * G.sb + h * G.sh, row0, row_end, ldt, ldt, 0);
    if (threadIdx.x < TR) m.qsh[threadIdx.x] = row0 + threadIdx.x < row_end ? -row_shift[(size_t)bh * L + row0 + threadIdx.x] : 0.f;
    __syncthreads();
    row_terms_of(m.rterm, ks, bh, L, row0, row_end);
    bwd_causal_amat(m.As, m.Gs, m.Vs, ldv, lds, ldt);

    f32x4 acc_o[ACC_V<WD, 8>], acc_g[ACC_D<WD, 8>];
#pragma unroll
    for (int t = 0; t < ACC_V<WD, 8>; ++t) acc_o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < ACC_D<WD, 8>; ++t) acc_g[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sc = {0.f, 0.f, 0.f, 0.f};      // scores tile (query tile w>>1, key tile w&1)
    float rs_part = 0.f;
    // the three blocks of the next step are fetched while the current one computes (rows of the state that this step
    // writes are not among them)
    WRegs<WD, NTC> wa, wb;
    ValTile<WD, NTC> tr;
    wblock_fetch(wa, W1, bias1, 0, M, d);
    sblock_fetch(tr, Rg, 0, M, ldt);
    wblock_fetch(wb, W2, bias2, 0, M, d);
    for (int m0 = 0; m0 < M; m0 += MB) {
      const int f = (w4 & 1) * 16 + (lane & 15);
      __syncthreads();
      wblock_put(wa, m.Ws, m.bias_s, ld, m0, M, d, dpad);
      wblock_put(wb, m.Ws2, m.bias2_s, ld, m0, M, d, dpad);
      sblock_put(tr, m.Ts, ldv, m0, M, ldt);
      __syncthreads();
      if (m0 + MB < M) {
        wblock_fetch(wa, W1, bias1, m0 + MB, M, d);
        wblock_fetch(wb, W2, bias2, m0 + MB, M, d);
        sblock_fetch(tr, Rg, m0 + MB, M, ldt);
      }
      // waves 0 - 3: features of the queries, then scores; waves 4 - 7: features and dS tile (keys (w4>>1)*16..,
      // features (w4&1)*16..) = V1 R_next^T + A^T P of the keys
      float fv[4];
      f32x4 ds = {0.f, 0.f, 0.f, 0.f};
      if (half == 0) {
        const f32x4 e = proj_tile(m.Qs, m.Ws, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          m.Ps[row * lds + f] = (m0 + f < M && row0 + row < row_end) ? fast_exp2(e[r] + m.bias_s[f] + m.qsh[row]) : 0.f;
        }
      } else {
        const f32x4 e = proj_tile(m.Ks, m.Ws2, ld, dpad);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          fv[r] = (m0 + f < M && row0 + row < row_end) ? fast_exp2(e[r] + m.bias2_s[f] + m.rterm[row] - c) : 0.f;
          m.Ss[row * lds + f] = fv[r];
        }
        const float* ap = m.Vs + ((w4 >> 1) * 16 + (lane & 15)) * ldv + (lane >> 4);   // A[j][k=v] = Vs[j][v]
        const float* bp = m.Ts + ((w4 & 1) * 16 + (lane & 15)) * ldv + (lane >> 4);    // B[k=v][n=m] = Rs[m][v]
        ds = mfma_chain(ap, 1, bp, 1, ldt, ds);
      }
      __syncthreads();
      if (half == 0) {   // scores: A[i][k=m] = Ps[i][m], B[k=m][n=j] = Ss[j][m]
        const float* ap = m.Ps + ((w4 >> 1) * 16 + (lane & 15)) * lds + (lane >> 4);
        const float* bp = m.Ss + ((w4 & 1) * 16 + (lane & 15)) * lds + (lane >> 4);
        sc = mfma_chain(ap, 1, bp, 1, MB, sc);
      } else {
        const float* ap = m.As + (lane >> 4) * lds + (w4 >> 1) * 16 + (lane & 15);     // A[j][k=i] = As[i][j]
        const float* bp = m.Ps + (lane >> 4) * lds + (w4 & 1) * 16 + (lane & 15);      // B[k=i][n=m] = Ps[i][m]
        ds = mfma_chain(ap, lds, bp, lds, TR, ds);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (w4 >> 1) * 16 + 4 * (lane >> 4) + r;
          m.dEs[row * lds + f] = fv[r] * ds[r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
        const int t = w + 8 * tl;
        if (t < ntiles) {
          const int rt = t & 1, vt = t >> 1;
          {   // dV1 += S R_next: A[j][k=m] = Ss[j][m], B[k=m][n=v] = Rs[m][v]
            const float* ap = m.Ss + (rt * 16 + (lane & 15)) * lds + (lane >> 4);
            const float* bp = m.Ts + (lane >> 4) * ldv + vt * 16 + (lane & 15);
            acc_o[tl] = mfma_chain(ap, 1, bp, ldv, MB, acc_o[tl]);
          }
          {   // the suffix sum takes this chunk's queries (after its last use): R[m][v] += sum_i Ps[i][m] Gs[i][v]
            f32x4 up = {0.f, 0.f, 0.f, 0.f};
            const float* ap = m.Ps + (lane >> 4) * lds + rt * 16 + (lane & 15);
            const float* bp = m.Gs + (lane >> 4) * ldv + vt * 16 + (lane & 15);
            up = mfma_chain(ap, lds, bp, ldv, TR, up);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int mb = rt * 16 + 4 * (lane >> 4) + r;
              if (m0 + mb < M) Rg[(size_t)(m0 + mb) * ldt + vt * 16 + (lane & 15)] = m.Ts[mb * ldv + vt * 16 + (lane & 15)] + up[r];
            }
          }
        }
      }
#pragma unroll
      for (int tl = 0; tl < ACC_D<WD, 8>; ++tl) {
        const int t = w + 8 * tl;
        if (t < ngt) {
          const int rt = t & 1, ct = t >> 1;
          const float* ap = m.dEs + (rt * 16 + (lane & 15)) * lds + (lane >> 4);
          const float* bp = m.Ws2 + (lane >> 4) * ld + min(ct * 16 + (lane & 15), dpad - 1);   // (columns past dpad are dropped below)
          acc_g[tl] = mfma_chain(ap, 1, bp, ld, MB, acc_g[tl]);
        }
      }
      if (half == 0) {
        const int row = threadIdx.x >> 3, part = threadIdx.x & 7;
#pragma unroll
        for (int q = 0; q < 4; ++q) rs_part += m.dEs[row * lds + part * 4 + q];
      }
    }
    // B = tril(P S^T); dV1 += B^T G1: A[j][k=i] = Bs[i][j], B[k=i][n=v] = Gs[i][v]
    if (half == 0)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = (w4 >> 1) * 16 + 4 * (lane >> 4) + r, j = (w4 & 1) * 16 + (lane & 15);
      m.Bs[i * lds + j] = (j <= i) ? sc[r] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
        const float* ap = m.Bs + (lane >> 4) * lds + rt * 16 + (lane & 15);
        const float* bp = m.Gs + (lane >> 4) * ldv + vt * 16 + (lane & 15);
        acc_o[tl] = mfma_chain(ap, lds, bp, ldv, TR, acc_o[tl]);
      }
    }
    __syncthreads();
    float* Gd = m.Ws;
    float* Os = m.Ts;
#pragma unroll
    for (int tl = 0; tl < ACC_D<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ngt) {
        const int rt = t & 1, ct = t >> 1, col = ct * 16 + (lane & 15);
        if (col < dpad) {
#pragma unroll
          for (int r = 0; r < 4; ++r) Gd[(rt * 16 + 4 * (lane >> 4) + r) * ld + col] = acc_g[tl][r];
        }
      }
    }
#pragma unroll
    for (int tl = 0; tl < ACC_V<WD, 8>; ++tl) {
      const int t = w + 8 * tl;
      if (t < ntiles) {
        const int rt = t & 1, vt = t >> 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) Os[(rt * 16 + 4 * (lane >> 4) + r) * ldv + vt * 16 + (lane & 15)] = acc_o[tl][r];
      }
    }
    rs_part += __shfl_xor(rs_part, 1);
    rs_part += __shfl_xor(rs_part, 2);
    rs_part += __shfl_xor(rs_part, 4);
    if (half == 0 && (threadIdx.x & 7) == 0) m.rsum[threadIdx.x >> 3] = rs_part;
    __syncthreads();
    bwd_store_grad(dK, b * dK.sb + h * dK.sh, row0, row_end, d, ld, Gd, m.rsum, m.Ks, Cmat2, ks.scale, 0.f);
    for (int idx = threadIdx.x; idx < TR * nv; idx += NTC) {
      const int r = idx / nv, cc = idx - r * nv;
      if (row0 + r < row_end) store_elem(dV, b * dV.sb + h * dV.sh + (long long)(row0 + r) * dV.sl + cc, Os[r * ldv + cc]);
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------------------
static size_t lds_floats_basic(int d) { const int ld = ((d + 3) & ~3) + 1; return (size_t)(TR + MB) * ld + MB + 2 * TR + TR; }

size_t gen_lds_features(int d) { return lds_floats_basic(d) * 4; }
size_t gen_lds_apply(int d, int ldt) {
  const int ld = ((d + 3) & ~3) + 1;
  return ((size_t)(TR + MB) * ld + (size_t)MB * (ldt + 1) + (size_t)TR * (MB + 1) + MB + 3 * TR) * 4;
}
size_t gen_lds_causal(int d, int ldt) {
  const int ld = ((d + 3) & ~3) + 1;
  return ((size_t)2 * (TR + MB) * ld + (size_t)(TR + MB) * (ldt + 1) + (size_t)3 * TR * (MB + 1) + 2 * MB + 2 * TR) * 4;
}
size_t gen_lds_stats(int d) { return (size_t)TR * (((d + 15) & ~15) + 1) * 4; }

#define FS_LAUNCH_CHECK() do { if (hipGetLastError() != hipSuccess) return 5; } while (0)

static int set_lds(const void* fn, size_t bytes) {
  if (bytes > 48 * 1024) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) {
      (void)hipGetLastError();
      return 2;
    }
  }
  return 0;
}

// The kernels' width for rows of d and values of ldt columns: the narrowest that holds both.
template <class F>
static int by_width(int d, int ldt, F launch) {
  if (d <= 32 && ldt <= 64) return launch(std::integral_constant<int, 1>());
  if (d <= 64 && ldt <= 96) return launch(std::integral_constant<int, 2>());
  return launch(std::integral_constant<int, 4>());
}

int launch_prep(const float* theta, int groups, const float* Omega, int omega_groups, int pgroups, int B, int H,
                int M, int d, float* W, float* bias, uint32_t* clear, int nclear, hipStream_t st, const GenSplit& split) {
  const int features = split.img != nullptr ? 16 * split.tiles : M;
  const int nx = (features + PREP_F - 1) / PREP_F;
  const long long parts = split.img != nullptr ? (long long)split.BH * ((split.L + VMAX_ROWS - 1) / VMAX_ROWS) : 0;
  const long long layers = (parts + (long long)nx * pgroups - 1) / ((long long)nx * pgroups);      // (of the grid, for value_maxima)
  hipLaunchKernelGGL(k_prep, dim3(nx, 2 + (unsigned)(layers < 1024 ? layers : 1024), pgroups), dim3(128), 0, st, theta, groups, Omega, omega_groups, pgroups, B, H,
                     M, d, W, bias, clear, nclear, split);
  FS_LAUNCH_CHECK();
  return 0;
}

int launch_fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t st) {
  if (n == 0) return 0;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
  FS_LAUNCH_CHECK();
  return 0;
}

int launch_gen_features(const TensorDev& X, int n, int d, float scale, float alpha, const float* W, const float* bias,
                        const float* theta, long long c_offset, int M, float* out, float* row_logscale,
                        hipStream_t st) {
  return by_width(d, 0, [&](auto width) -> int {
    constexpr int WD = width();
    const size_t lds = gen_lds_features(d);
    if (int rc = set_lds((const void*)k_gen_features<WD>, lds)) return rc;
    hipLaunchKernelGGL((k_gen_features<WD>), dim3((n + TR - 1) / TR), dim3(NT), lds, st, X, n, d, scale, alpha, W, bias, theta,
                       c_offset, M, out, row_logscale);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

int launch_gen_reduce(float* Tpart, int BH, int nseg, size_t per_state, int prefix, hipStream_t st) {
  const size_t total = (size_t)BH * per_state;
  if (prefix == 0) {
    hipLaunchKernelGGL(k_gen_reduce, dim3((unsigned)((total + 63) / 64)), dim3(64, 4), 0, st, Tpart, nseg, per_state, total);
  } else {
    hipLaunchKernelGGL(k_gen_scan, dim3((unsigned)((total / 4 + 63) / 64)), dim3(64), 0, st, Tpart, nseg, per_state / 4, total / 4,
                       prefix == 2 ? -1 : 1);
  }
  FS_LAUNCH_CHECK();
  return 0;
}

int launch_gen_apply(const GenSide& qs, int Lq, int BH, int H, int M, int d, int nv, int ldt, const float* T,
                     size_t state_stride, const uint32_t* kmax_u, int matvec, const TensorDev& Y, float* den_out,
                     float* shift_out, hipStream_t st, unsigned* flushed) {
  return by_width(d, ldt, [&](auto width) -> int {
    constexpr int WD = width();
    const size_t lds = gen_lds_apply(d, ldt);
    if (int rc = set_lds((const void*)k_gen_apply<WD>, lds)) return rc;
    hipLaunchKernelGGL((k_gen_apply<WD>), dim3((Lq + TR - 1) / TR, BH), dim3(NT), lds, st, qs, Lq, H, M, d, nv, ldt, T,
                       state_stride, kmax_u, matvec, Y, den_out, shift_out, flushed);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

size_t gen_lds_bwd_side(int d, int ldt) {
  const int ld = ((d + 3) & ~3) + 1;
  return ((size_t)(TR + MB) * ld + (size_t)(TR + MB) * (ldt + 1) + (size_t)2 * TR * (MB + 1) + MB + 2 * TR) * 4;
}

int launch_bwd_ghat(const TensorDev& dY, float* buf, const float* den, const int* exps, float* largest, int L, int BH, int H, int nv, int ldt,
                    hipStream_t st) {
  const size_t rows = (size_t)BH * L;
  if (largest != nullptr)
    hipLaunchKernelGGL(k_bwd_ghat<true>, dim3((L + GMAX_ROWS - 1) / GMAX_ROWS, BH), dim3(256), 0, st, dY, buf, den, exps, largest, L, H, nv, ldt, (size_t)L);
  else
    hipLaunchKernelGGL(k_bwd_ghat<false>, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, dY, buf, den, exps, largest, L, H, nv, ldt, rows);
  FS_LAUNCH_CHECK();
  return 0;
}

int launch_gen_bwd_side(const GenSide& sd, int side, const TensorDev& A, int a_cols, int append_ones, int L, int BH,
                        int H, int M, int d, int nv, int ldt, const float* St, size_t state_stride,
                        const uint32_t* kmax_u, const float* row_shift, const TensorDev& out1, int want_out1,
                        const TensorDev& grad, hipStream_t st) {
  return by_width(d, ldt, [&](auto width) -> int {
    constexpr int WD = width();
    const size_t lds = gen_lds_bwd_side(d, ldt);
    if (int rc = set_lds((const void*)k_gen_bwd_side<WD>, lds)) return rc;
    hipLaunchKernelGGL((k_gen_bwd_side<WD>), dim3((L + TR - 1) / TR, BH), dim3(NT), lds, st, sd, side, A, a_cols, append_ones, L,
                       H, M, d, nv, ldt, St, state_stride, kmax_u, row_shift, out1, want_out1, grad);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

size_t gen_lds_bwd_causal(int d, int ldt) {
  const int ld = ((d + 3) & ~3) + 1;
  return ((size_t)2 * (TR + MB) * ld + (size_t)(2 * TR + MB) * (ldt + 1) + (size_t)5 * TR * (MB + 1) + 2 * MB + 3 * TR) * 4;
}

int launch_gen_bwd_causal(const GenSide& qs, const GenSide& ks, const TensorDev& V, const float* ghat, int L, int BH, int H,
                          int M, int d, int nv, int ldt, int rows_per_seg, int nseg, const uint32_t* kmax_u,
                          const float* row_shift, float* Tstate, float* Rstate, const TensorDev& dQ, const TensorDev& dK,
                          const TensorDev& dV, hipStream_t st) {
  return by_width(d, ldt, [&](auto width) -> int {
    constexpr int WD = width();
    const size_t lds = gen_lds_bwd_causal(d, ldt);
    if (int rc = set_lds((const void*)k_gen_bwd_causal_q<WD>, lds)) return rc;
    if (int rc = set_lds((const void*)k_gen_bwd_causal_k<WD>, lds)) return rc;
    hipLaunchKernelGGL((k_gen_bwd_causal_q<WD>), dim3(nseg, BH), dim3(NTC), lds, st, qs, ks, V, ghat, L, H, M, d, nv, ldt,
                       rows_per_seg, nseg, kmax_u, row_shift, Tstate, dQ);
    FS_LAUNCH_CHECK();
    hipLaunchKernelGGL((k_gen_bwd_causal_k<WD>), dim3(nseg, BH), dim3(NTC), lds, st, qs, ks, V, ghat, L, H, M, d, nv, ldt,
                       rows_per_seg, nseg, kmax_u, row_shift, Rstate, dK, dV);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

int launch_gen_causal(const GenSide& qs, const GenSide& ks, const TensorDev& V, int L, int BH, int H, int M, int d,
                      int nv, int ldt, int rows_per_seg, int nseg, const uint32_t* kmax_u, float* Tstate,
                      const TensorDev& Y, float* den_out, float* shift_out, hipStream_t st, unsigned* flushed) {
  return by_width(d, ldt, [&](auto width) -> int {
    constexpr int WD = width();
    const size_t lds = gen_lds_causal(d, ldt);
    if (int rc = set_lds((const void*)k_gen_causal<WD>, lds)) return rc;
    hipLaunchKernelGGL((k_gen_causal<WD>), dim3(nseg, BH), dim3(NTC), lds, st, qs, ks, V, L, H, M, d, nv, ldt, rows_per_seg,
                       nseg, kmax_u, Tstate, Y, den_out, shift_out, flushed);
    FS_LAUNCH_CHECK();
    return 0;
  });
}

int launch_stats(const TensorDev& X, const TensorDev& Y, int B, int H, int Lx, int Ly, int d, float scale, int groups,
                 int rows_per_chunk, int nchunks, float* part, double* stats, hipStream_t st) {
  if (stats_bf16_supported(X, Y, d)) {
    if (int rc = launch_stats_bf16(X, Y, B * H, H, Lx, Ly, scale, rows_per_chunk, nchunks, part, st)) return rc;
  } else if (stats_wide_supported(X, Y, d)) {
    if (int rc = launch_stats_wide(X, Y, B * H, H, Lx, Ly, scale, rows_per_chunk, nchunks, part, st)) return rc;
  } else {
    const int rc = by_width(d, 0, [&](auto width) -> int {
      constexpr int WD = width();
      const size_t lds = gen_lds_stats(d);
      if (int rc = set_lds((const void*)k_stats_partial<WD>, lds)) return rc;
      hipLaunchKernelGGL((k_stats_partial<WD>), dim3(nchunks, B * H, 2), dim3(NT), lds, st, X, Y, Lx, Ly, H, d, scale,
                         rows_per_chunk, nchunks, part);
      FS_LAUNCH_CHECK();
      return 0;
    });
    if (rc) return rc;
  }
  const size_t total = (size_t)groups * 2 * ((size_t)d * d + d);
  hipLaunchKernelGGL(k_stats_final, dim3((unsigned)((total + 127) / 128)), dim3(128), 0, st, part, B, H, nchunks, d,
                     groups, Lx, Ly, stats);
  FS_LAUNCH_CHECK();
  return 0;
}

}  // namespace fs
