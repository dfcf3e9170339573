// General-shape causal kernels with the state in registers: fp32 matrix instructions, d and dv multiples of four up to 128, M up to
// 512 (other shapes, and those that would be mostly padding here: the causal kernels of kernels_generic.hip, whose state lies in
// memory; with many features and rows that are not narrow: kernels_gen_split.hip).
//
// A workgroup walks a segment of a sequence sixteen tokens at a time; a wave holds 16 FT features: its rows of the state stay in
// accumulators from the first token to the last, and every operand of every product is either such an accumulator, a
// packed accumulator of this chunk, or a row of the chunk in LDS (kernels_gen_rows.hip has the layouts).  Two barriers per
// chunk: one when its rows have arrived, one when the waves' partial output rows are complete; rows of the next
// chunk travel meanwhile.  What bounds them is the fp32 matrix rate (32 cycles per instruction) and the rows of W~, which come from L2
// once per chunk, 13 bytes per cycle and CU.  Causal attention f32 B2 H4 L4096 d64 M256: 175 -> 89 us for this kernel, backward
// pass bf16 B1 H16 L4096 d128 M512: 3300 -> 2560 us for its four (sizes that kernels_gen_split.hip has taken over since).
#include <type_traits>

#include "gen_widths.h"
#include "kernels.h"

namespace fs {
namespace {

using namespace gen;

constexpr int TT = 16;                                   // tokens per chunk
template <int Q> constexpr int LDX = 16 * Q + 4;         // strides of LDS rows: 16-byte reads of a column group and 4-byte
template <int Q> constexpr int LDV = 16 * VT_OF<Q> + 4;  // reads of four rows 4 apart touch every bank once

// Rows of a tensor on their way global -> registers -> LDS, sixteen rows of 16 G numbers, 16 (bf16: 8) bytes per thread and piece.
template <int G, int NW> struct Pieces { u32x4 v[(G + NW - 1) / NW]; };
struct RowSrc {
  const void* ptr;
  int dtype;
  long long base, sl;
  int ncols;               // numbers per row (a multiple of four); column ncols of a live row is `one`, the rest zero
  float scale, one;
};
__device__ __forceinline__ RowSrc row_src(const TensorDev& t, int b, int h, int ncols, float scale, float one) {
  return RowSrc{t.ptr, t.dtype, b * t.sb + h * t.sh, t.sl, ncols, scale, one};
}
template <int G, int NW>
__device__ __forceinline__ void fetch(Pieces<G, NW>& p, const RowSrc& s, int row0, int row_end, int tid) {
#pragma unroll
  for (int i = 0; i < (G + NW - 1) / NW; ++i) {
    const int e = tid + 64 * NW * i, row = min(e / (4 * G), TT - 1), col = 4 * (e % (4 * G));
    const long long at = s.base + (long long)min(row0 + row, row_end - 1) * s.sl + min(col, s.ncols - 4);
    if (s.dtype == 0) {
      p.v[i] = *(const u32x4*)((const float*)s.ptr + at);
    } else {
      const u32x2 r = *(const u32x2*)((const uint16_t*)s.ptr + at);
      p.v[i] = u32x4{r[0], r[1], 0u, 0u};
    }
  }
}
template <int G, int NW>
__device__ __forceinline__ void put(const Pieces<G, NW>& p, const RowSrc& s, float* dst, int ld, int row0, int row_end, int tid) {
#pragma unroll
  for (int i = 0; i < (G + NW - 1) / NW; ++i) {
    const int e = tid + 64 * NW * i, row = e / (4 * G), col = 4 * (e % (4 * G));
    if (row >= TT) continue;
    const u32x4 r = p.v[i];
    f32x4 x = s.dtype == 0 ? __builtin_bit_cast(f32x4, r)
                           : f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xffff0000u), __uint_as_float(r[1] << 16),
                                   __uint_as_float(r[1] & 0xffff0000u)};
    x *= s.scale;
    const bool live = row0 + row < row_end;
    if (!live || col >= s.ncols) x = f32x4{live && col == s.ncols ? s.one : 0.f, 0.f, 0.f, 0.f};
    *(f32x4*)(dst + row * ld + col) = x;
  }
}

// acc[ft]: exponents (without bias) of 16 FT features against the sixteen rows at Xs.  FEATURE_ROWS: rows = features 4 g + r,
// column = token c; else rows = tokens 4 g + r, column = feature c.  The rows of W~ of the next 16-column group are requested
// while one is used (a uniform base and 32-bit offsets, found anew for every chunk: addresses kept across chunks take
// hundreds of registers).
// The first group (first_group) is requested by the caller, ahead of whatever comes before the projection.
__device__ __forceinline__ f32x4 load_wgroup(const float* W, int f, int q, int M, int d, int g) {
  return *(const f32x4*)((const char*)W + (4u * (uint32_t)(min(f, M - 1) * d) + 4u * (uint32_t)min(16 * q + 4 * g, d - 4)));
}
template <int FT>
__device__ __forceinline__ void first_group(f32x4 (&w)[FT], const float* W, int f0, int M, int d, int g, int c) {
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) w[ft] = load_wgroup(W, f0 + 16 * ft + c, 0, M, d, g);
}
template <bool FEATURE_ROWS, int Q, int FT>
__device__ __forceinline__ void project(f32x4 (&acc)[FT], const f32x4 (&w0)[FT], const float* W, int f0, int M, int d, const float* Xs,
                                        int g, int c) {
  f32x4 w[2][FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    acc[ft] = f32x4{0.f, 0.f, 0.f, 0.f};
    w[0][ft] = w0[ft];
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    __builtin_amdgcn_sched_barrier(0);             // (one group ahead and not all of them: registers)
    if (q + 1 < Q) {
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) w[(q + 1) & 1][ft] = load_wgroup(W, f0 + 16 * ft + c, q + 1, M, d, g);
    }
    const f32x4 x = *(const f32x4*)(Xs + c * LDX<Q> + 16 * q + 4 * g);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) acc[ft] = FEATURE_ROWS ? mfma4(w[q & 1][ft][s], x[s], acc[ft]) : mfma4(x[s], w[q & 1][ft][s], acc[ft]);
  }
}

struct WalkArgs {
  GenSide F, S;            // first side (whose rows enter the state), second side (whose rows are the output's)
  TensorDev V, U;          // values of the first side's rows; (gradient walk) left rows of the second side
  int vcols, vone, ucols, uone;
  int L, H, M, d, nv, ldt, rows_per_seg, nseg;
  const uint32_t* kmax_u;
  const float* row_shift;  // [BH][L] shifts of the queries (MODE 1, gradient walks)
  const float* state;      // [BH][nseg][M][ldt], exclusive prefix (forward) or suffix (backward)
  TensorDev out;
  float *den_out, *shift_out;
  unsigned* flushed;
};

// What a token of a side brings to its exponents: - its shift (queries), its row term (keys, whose shift is the key
// maximum), -inf past the end; and an exponent of it, in the order of the other kernels (kernels_gen_rows.hip).
template <bool KEYS>
__device__ __forceinline__ float side_term(const WalkArgs& a, const GenSide& sd, int bh, int row, int row_end) {
  if (row >= row_end) return -INFINITY;
  return KEYS ? sd.rk[(size_t)bh * a.L + row] : -a.row_shift[(size_t)bh * a.L + row];
}
template <bool KEYS>
__device__ __forceinline__ float exponent(float e, float bias, float term, float kmax) {
  return KEYS ? ((e + bias) + term) - kmax : (e + bias) + term;
}

// ---------------------------------------------------------------------------------------------------
// Output walk.  MODE 0 (forwards): first side keys with [V 1], output Y of the queries, whose features are shifted by the
// wave's own maximum of the row; the waves' partial rows are brought to the row's maximum where they are summed.
// MODE 1 (backwards): first side queries with the rows of G1, output dV of the keys.  grid (nseg, B*H), block 64 NW.
//   y_i = P_i T + sum_j tril(P_i S_j) V_j ;  T += S^T V
// ---------------------------------------------------------------------------------------------------
template <int Q, int FT, int NW> constexpr int XCH = TT * (16 * VT_OF<Q> + 1) > FT * 320 ? TT * (16 * VT_OF<Q> + 1) : FT * 320;
template <int Q, int FT, int NW> constexpr size_t walk_lds() {
  return 4 * ((size_t)2 * (2 * TT * LDX<Q> + TT * LDV<Q>) + (size_t)NW * XCH<Q, FT, NW> + NW * TT + 16 * FT * NW);
}

template <int Q, int FT, int NW, int MODE>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) k_gen_walk(WalkArgs a) {
  extern __shared__ __align__(16) float smem[];
  constexpr int VT = VT_OF<Q>, ldx = LDX<Q>, ldv = LDV<Q>, ldo = 16 * VT + 1, xch1 = XCH<Q, FT, NW>;
  constexpr int kBuf = 2 * TT * ldx + TT * ldv;
  float* xch = smem + 2 * kBuf;                    // [wave][token][column]; before that the wave's transposition of first-side features
  float* mw = xch + NW * xch1;                     // [wave][token]: row maxima
  float* bl = mw + NW * TT;                        // biases, -inf behind the last feature
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  int g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), f0 = 16 * FT * w;
  const int pg = group_of(a.F.pgroups, b, h, a.H), M = a.M, d = a.d;
  constexpr bool F_KEYS = MODE == 0;
  const float* W1 = a.F.W + ((size_t)pg * 2 + F_KEYS) * M * d;
  const float* W2 = a.S.W + ((size_t)pg * 2 + !F_KEYS) * M * d;
  const float* bias = a.F.bias + ((size_t)pg * 2) * M;      // (the same on both sides)
  const float kmax = ordered_to_float(a.kmax_u[bh]);
  const int row_beg = seg * a.rows_per_seg, row_end = min(a.L, row_beg + a.rows_per_seg);
  const int nchunk = (row_end - row_beg + TT - 1) / TT;
  const RowSrc xf = row_src(a.F.X, b, h, d, a.F.scale, 0.f), xs = row_src(a.S.X, b, h, d, a.S.scale, 0.f);
  const RowSrc vf = row_src(a.V, b, h, a.vcols, 1.f, a.vone ? 1.f : 0.f);
  auto row_of = [&](int ci) { return row_beg + TT * (MODE ? nchunk - 1 - ci : ci); };

  Pieces<Q, NW> pf, ps;
  Pieces<VT, NW> pv;
  auto fetch_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                       // (nothing of the addresses is kept across chunks: registers)
    const int r0 = row_of(ci);
    fetch<Q, NW>(pf, xf, r0, row_end, tid);
    fetch<Q, NW>(ps, xs, r0, row_end, tid);
    fetch<VT, NW>(pv, vf, r0, row_end, tid);
  };
  auto put_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    float* buf = smem + (ci & 1) * kBuf;
    const int r0 = row_of(ci);
    put<Q, NW>(pf, xf, buf, ldx, r0, row_end, tid);
    put<Q, NW>(ps, xs, buf + TT * ldx, ldx, r0, row_end, tid);
    put<VT, NW>(pv, vf, buf + 2 * TT * ldx, ldv, r0, row_end, tid);
  };
  fetch_chunk(0);
  for (int f = threadIdx.x; f < 16 * FT * NW; f += 64 * NW) bl[f] = f < M ? bias[f] : -INFINITY;
  f32x4 T[FT][VT];
  const float* st = a.state + ((size_t)bh * a.nseg + seg) * M * a.ldt;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int f = f0 + 16 * ft + 4 * g + r;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        const int col = 16 * vt + c;
        const float v = st[(size_t)min(f, M - 1) * a.ldt + min(col, a.ldt - 1)];
        T[ft][vt][r] = f < M && col < a.ldt ? v : 0.f;
      }
    }
  }
  put_chunk(0);
  float* lt = xch + w * xch1;
  for (int ci = 0; ci < nchunk; ++ci) {
    asm volatile("" : "+v"(g), "+v"(c));             // (nothing that follows from the lane is kept across chunks)
    const int row0 = row_of(ci);
    const float* buf = smem + (ci & 1) * kBuf;
    const float addf = side_term<F_KEYS>(a, a.F, bh, row0 + c, row_end);
    const float adds = MODE ? side_term<true>(a, a.S, bh, row0 + c, row_end) : 0.f;
    f32x4 wf[FT];
    first_group(wf, W1, f0, M, d, g, c);
    __syncthreads();
    // features of both sides: rows = features, column = token
    f32x4 sf[FT], p[FT];
    project<true, Q, FT>(sf, wf, W1, f0, M, d, buf, g, c);
    first_group(wf, W2, f0, M, d, g, c);
    project<true, Q, FT>(p, wf, W2, f0, M, d, buf + TT * ldx, g, c);
    __builtin_amdgcn_sched_barrier(0);
    f32x4 br[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) br[ft] = *(const f32x4*)(bl + f0 + 16 * ft + 4 * g);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int r = 0; r < 4; ++r) sf[ft][r] = fast_exp2(exponent<F_KEYS>(sf[ft][r], br[ft][r], addf, kmax));
    if (MODE) {
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[ft][r] = fast_exp2(exponent<true>(p[ft][r], br[ft][r], adds, kmax));
    } else {
      float m = -INFINITY;
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          p[ft][r] += br[ft][r];
          m = fmaxf(m, p[ft][r]);
        }
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      if (g == 0) mw[w * TT + c] = m;
      const float ms = m == -INFINITY ? 0.f : m;         // (a wave behind the last feature)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[ft][r] = fast_exp2(p[ft][r] - ms);
    }
    // the first side's features with tokens as rows, by way of the wave's LDS scratch
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) *(f32x4*)(lt + 320 * ft + 20 * c + 4 * g) = sf[ft];
    // scores of the chunk (rows = first-side tokens 4 g + r, column = second-side token c), and the state's part of the output
    f32x4 sc = {0.f, 0.f, 0.f, 0.f}, y[VT];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) y[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc = mfma4(sf[ft][r], p[ft][r], sc);
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) y[vt] = mfma4(p[ft][r], T[ft][vt][r], y[vt]);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) sc[r] = (MODE ? 4 * g + r >= c : 4 * g + r <= c) ? sc[r] : 0.f;
    // the next chunk's rows travel during the update
    if (ci + 1 < nchunk) fetch_chunk(ci + 1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const float* Vs = buf + 2 * TT * ldx;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      __builtin_amdgcn_sched_barrier(0);
      float s[FT];
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) s[ft] = lt[320 * ft + 20 * (4 * g + r) + c];
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        const float v = Vs[(4 * g + r) * ldv + 16 * vt + c];
        y[vt] = mfma4(sc[r], v, y[vt]);
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) T[ft][vt] = mfma4(s[ft], v, T[ft][vt]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int vt = 0; vt < VT; ++vt)
#pragma unroll
      for (int r = 0; r < 4; ++r) xch[w * xch1 + (4 * g + r) * ldo + 16 * vt + c] = y[vt][r];
    __builtin_amdgcn_sched_barrier(0);
    if (ci + 1 < nchunk) put_chunk(ci + 1);
    __syncthreads();
    // sum over the waves: 4 NW threads per row
    {
      const int row = threadIdx.x / (4 * NW), l = threadIdx.x % (4 * NW);
      float wgt[NW], m = -INFINITY, den = 1.f;
      if (!MODE) {
#pragma unroll
        for (int i = 0; i < NW; ++i) m = fmaxf(m, mw[i * TT + row]);
        den = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          const float mi = mw[i * TT + row];
          wgt[i] = mi == m ? 1.f : fast_exp2(mi - m);
          den += wgt[i] * xch[i * xch1 + row * ldo + a.nv];
        }
      }
      if (row0 + row < row_end) {
        const long long ob = b * a.out.sb + h * a.out.sh + (long long)(row0 + row) * a.out.sl;
        for (int col = l; col < a.nv; col += 4 * NW) {
          float v = 0.f;
#pragma unroll
          for (int i = 0; i < NW; ++i) v += (MODE ? 1.f : wgt[i]) * xch[i * xch1 + row * ldo + col];
          if (!MODE) v = den > 0.f ? v / den : 0.f;
          store_elem(a.out, ob + col, v);
        }
        if (!MODE && l == 0) {
          if (a.flushed != nullptr && !(den > 0.f)) atomicAdd(a.flushed, 1u);
          if (a.den_out != nullptr) {
            a.den_out[(size_t)bh * a.L + row0 + row] = den;
            a.shift_out[(size_t)bh * a.L + row0 + row] = m;
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Gradient walk.  MODE 0 (forwards): first side keys with [V 1], second side queries with left rows G1 -> dQ.  MODE 1 (backwards): first
// side queries with G1, second side keys with left rows [V 1] -> dK.
//   dF_i = Z u_i + sum_j tril(u_i . v_j) F_j ;  dE = F_second * dF ;  gradient = dE W~ (+ row term) ;  Z += F_first^T V
// The state is held transposed (rows = columns of the values, column = feature): as it lies it is the operand of dF.
// grid (nseg, B*H), block 64 NW.
// ---------------------------------------------------------------------------------------------------
template <int Q, int FT, int NW> constexpr size_t gwalk_lds() {
  return 4 * ((size_t)2 * (2 * TT * LDX<Q> + 2 * TT * LDV<Q>) + (size_t)NW * TT * (16 * Q + 1) + NW * TT + 16 * FT * NW + TT * LDX<Q>);
}

template <int Q, int FT, int NW, int MODE>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) k_gen_gwalk(WalkArgs a) {
  extern __shared__ __align__(16) float smem[];
  constexpr int VT = VT_OF<Q>, ldx = LDX<Q>, ldv = LDV<Q>, ldo = 16 * Q + 1, xch1 = TT * ldo;
  constexpr int kBuf = 2 * TT * ldx + 2 * TT * ldv;
  float* xch = smem + 2 * kBuf;                    // [wave][token][coordinate]
  float* rsw = xch + NW * xch1;                    // [wave][token]: row sums of dE
  float* bl = rsw + NW * TT;                       // biases, -inf behind the last feature
  float* cx = bl + 16 * FT * NW;                   // [token][coordinate]: x (C + C^T), where the kernel has a C
  const int seg = blockIdx.x, bh = blockIdx.y, b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  int g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), f0 = 16 * FT * w;
  const int pg = group_of(a.F.pgroups, b, h, a.H), M = a.M, d = a.d;
  constexpr bool F_KEYS = MODE == 0;
  const float* W1 = a.F.W + ((size_t)pg * 2 + F_KEYS) * M * d;
  const float* W2 = a.S.W + ((size_t)pg * 2 + !F_KEYS) * M * d;
  const float* bias = a.F.bias + ((size_t)pg * 2) * M;
  const float kmax = ordered_to_float(a.kmax_u[bh]);
  const int row_beg = seg * a.rows_per_seg, row_end = min(a.L, row_beg + a.rows_per_seg);
  const int nchunk = (row_end - row_beg + TT - 1) / TT;
  const RowSrc xf = row_src(a.F.X, b, h, d, a.F.scale, 0.f), xs = row_src(a.S.X, b, h, d, a.S.scale, 0.f);
  const RowSrc vf = row_src(a.V, b, h, a.vcols, 1.f, a.vone ? 1.f : 0.f), uf = row_src(a.U, b, h, a.ucols, 1.f, a.uone ? 1.f : 0.f);
  const float* th = a.S.theta + (size_t)group_of(a.S.groups, b, h, a.H) * a.S.theta_stride;
  const float* Cmat = (((int)th[2]) & 1) ? nullptr : th + a.S.c_offset;
  auto row_of = [&](int ci) { return row_beg + TT * (MODE ? nchunk - 1 - ci : ci); };

  Pieces<Q, NW> pf, ps;
  Pieces<VT, NW> pv, pu;
  auto fetch_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                       // (nothing of the addresses is kept across chunks: registers)
    const int r0 = row_of(ci);
    fetch<Q, NW>(pf, xf, r0, row_end, tid);
    fetch<Q, NW>(ps, xs, r0, row_end, tid);
    fetch<VT, NW>(pv, vf, r0, row_end, tid);
    fetch<VT, NW>(pu, uf, r0, row_end, tid);
  };
  auto put_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    float* buf = smem + (ci & 1) * kBuf;
    const int r0 = row_of(ci);
    put<Q, NW>(pf, xf, buf, ldx, r0, row_end, tid);
    put<Q, NW>(ps, xs, buf + TT * ldx, ldx, r0, row_end, tid);
    put<VT, NW>(pv, vf, buf + 2 * TT * ldx, ldv, r0, row_end, tid);
    put<VT, NW>(pu, uf, buf + 2 * TT * ldx + TT * ldv, ldv, r0, row_end, tid);
  };
  fetch_chunk(0);
  for (int f = threadIdx.x; f < 16 * FT * NW; f += 64 * NW) bl[f] = f < M ? bias[f] : -INFINITY;
  f32x4 Z[FT][VT];                                  // Z[ft][vt][r]: feature f0 + 16 ft + c, column 16 vt + 4 g + r
  const float* st = a.state + ((size_t)bh * a.nseg + seg) * M * a.ldt;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int f = f0 + 16 * ft + c, fw = min(f, M - 1);
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      const int col = 16 * vt + 4 * g;
      const f32x4 v = *(const f32x4*)(st + (size_t)fw * a.ldt + min(col, a.ldt - 4));
      Z[ft][vt] = f < M && col < a.ldt ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  put_chunk(0);
  for (int ci = 0; ci < nchunk; ++ci) {
    asm volatile("" : "+v"(g), "+v"(c));             // (nothing that follows from the lane is kept across chunks)
    const int row0 = row_of(ci);
    const float* buf = smem + (ci & 1) * kBuf;
    const float* Vs = buf + 2 * TT * ldx;
    const float* Us = Vs + TT * ldv;
    float addf[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) addf[r] = side_term<F_KEYS>(a, a.F, bh, row0 + 4 * g + r, row_end);
    const float adds = side_term<!F_KEYS>(a, a.S, bh, row0 + c, row_end);
    f32x4 wf[FT];
    first_group(wf, W1, f0, M, d, g, c);
    __syncthreads();
    // u_i . v_j (rows = first-side tokens 4 g + r, column = second-side token c), masked, and Z u
    f32x4 am = {0.f, 0.f, 0.f, 0.f}, df[FT];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) df[ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      if (vt % 3 == 0) __builtin_amdgcn_sched_barrier(0);
      const f32x4 u = *(const f32x4*)(Us + c * ldv + 16 * vt + 4 * g), v = *(const f32x4*)(Vs + c * ldv + 16 * vt + 4 * g);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        am = mfma4(v[s], u[s], am);
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) df[ft] = mfma4(Z[ft][vt][s], u[s], df[ft]);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) am[r] = (MODE ? 4 * g + r >= c : 4 * g + r <= c) ? am[r] : 0.f;
    // first side's features, rows = tokens, column = feature: into dF and into the state
    __builtin_amdgcn_sched_barrier(0);
    f32x4 ff[FT];
    project<false, Q, FT>(ff, wf, W1, f0, M, d, buf, g, c);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int r = 0; r < 4; ++r) ff[ft][r] = fast_exp2(exponent<F_KEYS>(ff[ft][r], bl[f0 + 16 * ft + c], addf[r], kmax));
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) df[ft] = mfma4(ff[ft][r], am[r], df[ft]);
    first_group(wf, W2, f0, M, d, g, c);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        if (vt == 0) __builtin_amdgcn_sched_barrier(0);
        const float v = Vs[(4 * g + r) * ldv + 16 * vt + c];
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) Z[ft][vt] = mfma4(v, ff[ft][r], Z[ft][vt]);
      }
    // second side's features, rows = features, column = token; dE = F * dF
    f32x4 fs2[FT];
    project<true, Q, FT>(fs2, wf, W2, f0, M, d, buf + TT * ldx, g, c);
    float rs = 0.f;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const f32x4 br = *(const f32x4*)(bl + f0 + 16 * ft + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        df[ft][r] *= fast_exp2(exponent<!F_KEYS>(fs2[ft][r], br[r], adds, kmax));
        rs += df[ft][r];
      }
    }
    rs += __shfl_xor(rs, 16);
    rs += __shfl_xor(rs, 32);
    if (g == 0) rsw[w * TT + c] = rs;
    // the next chunk's rows travel during the last products
    if (ci + 1 < nchunk) fetch_chunk(ci + 1);
    // gradient rows of this wave's features: dE W~ (wide rows in two halves: registers), a tile's rows of W~ one ahead
    constexpr int DT = Q >= 6 ? Q / 2 : Q, NS = FT * (Q / DT);
    auto load_w = [&](float (&wv)[4][DT], int st) {
      const int ft = st % FT, d0 = DT * (st / FT);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t row = 4u * (uint32_t)(min(f0 + 16 * ft + 4 * g + r, M - 1) * d);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) wv[r][dt] = *(const float*)((const char*)W2 + (row + 4u * (uint32_t)min(16 * (d0 + dt) + c, d - 1)));
      }
    };
    float wv[2][4][DT];
    load_w(wv[0], 0);
    f32x4 gr[DT];
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int ft = st % FT, d0 = DT * (st / FT);
      __builtin_amdgcn_sched_barrier(0);
      if (st + 1 < NS) load_w(wv[(st + 1) & 1], st + 1);
      if (ft == 0) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) gr[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) gr[dt] = mfma4(df[ft][r], wv[st & 1][r][dt], gr[dt]);
      if (ft == FT - 1) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) xch[w * xch1 + (4 * g + r) * ldo + 16 * (d0 + dt) + c] = gr[dt][r];
      }
    }
    // the row term's part, a tile of sixteen columns per wave.  (A thread's own dot products with rows and columns of C cost
    // half as much as everything else: 1024 loads per thread and chunk at d = 128.  Causal backward f32 B2 H8 L1000 d128
    // M256 with a dense C: 1383 -> 851 us.)
    if (Cmat != nullptr) {
      for (int ct = w; ct < Q; ct += NW) {
        const float* xr = buf + TT * ldx + c * ldx + 4 * g;
        const uint32_t col = (uint32_t)min(16 * ct + c, d - 1);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          if (q % 2 == 0) __builtin_amdgcn_sched_barrier(0);
          const uint32_t e = (uint32_t)min(16 * q + 4 * g, d - 4);
          f32x4 cm = *(const f32x4*)((const char*)Cmat + 4u * (col * (uint32_t)d + e));
#pragma unroll
          for (int s = 0; s < 4; ++s) cm[s] += *(const float*)((const char*)Cmat + 4u * ((e + s) * (uint32_t)d + col));
          const f32x4 x = *(const f32x4*)(xr + 16 * q);
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = mfma4(x[s], cm[s], acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) cx[(4 * g + r) * ldx + 16 * ct + c] = acc[r];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (ci + 1 < nchunk) put_chunk(ci + 1);
    __syncthreads();
    {
      const int row = threadIdx.x / (4 * NW), l = threadIdx.x % (4 * NW);
      const float* x = buf + TT * ldx + row * ldx;
      float rsum = 0.f;
#pragma unroll
      for (int i = 0; i < NW; ++i) rsum += rsw[i * TT + row];
      if (row0 + row < row_end) {
        const long long ob = b * a.out.sb + h * a.out.sh + (long long)(row0 + row) * a.out.sl;
        for (int col = l; col < d; col += 4 * NW) {
          float v = 0.f;
#pragma unroll
          for (int i = 0; i < NW; ++i) v += xch[i * xch1 + row * ldo + col];
          const float rc = Cmat != nullptr ? cx[row * ldx + col] : -x[col];
          store_elem(a.out, ob + col, a.S.scale * (v * kLn2 + rsum * rc));
        }
      }
    }
  }
}

// Features per wave and waves: two waves per SIMD where there are tiles for them (one's loads and exponentials beside the
// other's matrix instructions: B2 H4 L4096 d64 M256 156 us against 168 with four waves of 64 features).
template <class F>
int by_features(int M, F launch) {
  if (M <= 64) return launch(std::integral_constant<int, 1>(), std::integral_constant<int, 4>());
  if (M <= 128) return launch(std::integral_constant<int, 1>(), std::integral_constant<int, 8>());
  if (M <= 256) return launch(std::integral_constant<int, 2>(), std::integral_constant<int, 8>());
  return launch(std::integral_constant<int, 4>(), std::integral_constant<int, 8>());
}
template <class K>
int run(K kernel, const WalkArgs& a, int nseg, int BH, int threads, size_t lds, hipStream_t st) {
  if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  hipLaunchKernelGGL(kernel, dim3(nseg, BH), dim3(threads), lds, st, a);
  return hipGetLastError() == hipSuccess ? 0 : 5;
}
template <int MODE>
int run_walk(const WalkArgs& a, int BH, hipStream_t st) {
  return by_width(a.d, a.ldt, [&](auto q) {
    return by_features(a.M, [&](auto ft, auto nw) {
      return run(k_gen_walk<q(), ft(), nw(), MODE>, a, a.nseg, BH, 64 * nw(), walk_lds<q(), ft(), nw()>(), st);
    });
  });
}
template <int MODE>
int run_gwalk(const WalkArgs& a, int BH, hipStream_t st) {
  return by_width(a.d, a.ldt, [&](auto q) {
    return by_features(a.M, [&](auto ft, auto nw) {
      return run(k_gen_gwalk<q(), ft(), nw(), MODE>, a, a.nseg, BH, 64 * nw(), gwalk_lds<q(), ft(), nw()>(), st);
    });
  });
}

}  // namespace

// Rows and values are fetched four numbers at a time, and eight waves hold 64 features each.  A walk is made for the larger of the
// widths of rows and values and for at least 64 features; where most of that is padding the kernels of kernels_generic.hip
// remain, which go through blocks of 32 features and count columns.  (many: more segments than CUs, in the gradients before they
// are shortened.)  Speed of a call on walks against one on those kernels, f32 and bf16:
//   attention, widths even      1 x 192 to 128 x 512, d 8 to 128, M 16 to 512: 1.0 - 2.6 (bf16 d 128 M <= 32: 0.98 - 1.06)
//   attention, uneven, M <= 32  d 8 dv 128  0.82 - 0.95;  d 8 dv 64 and d 64 dv 16  0.92 - 0.99, with many segments 1.1 - 1.3
//   gradients                   few segments 1.1 - 3 (rows per segment: favorsharp_api.hip);  many, even widths 1.06 - 1.9, with a
//                               dense C up to 3, wide rows at M <= 32 0.78 - 0.96 (dense 3);  many, d <= 64 beside dv 128,
//                               M <= 64  0.6 - 0.9 (d 64 dense 1.15);  many, d 128 beside dv 8  0.63 - 0.9 (dense 3)
static bool walk_possible(int d, int dv, int M) { return d % 4 == 0 && dv % 4 == 0 && M <= 512; }
struct WalkWidths { int all; bool even; };
static WalkWidths walk_widths(int d, int dv) {
  const int ldt = (dv + 16) / 16 * 16;
  auto w = [](int d_, int ldt_) { return by_width(d_, ldt_, [](auto q) { return (int)q(); }); };
  const int all = w(d, ldt), rows = w(d, 0), values = w(0, ldt), lo = rows < values ? rows : values;
  return {all, all >= 6 ? lo >= 6 : 2 * lo >= all};
}
bool gen_walk_attention(int d, int dv, int M, bool many) {
  const WalkWidths x = walk_widths(d, dv);
  return walk_possible(d, dv, M) && (M > 32 || x.even || (x.all < 6 && many));
}
bool gen_walk_backward(int d, int dv, int M, bool many) {
  const WalkWidths x = walk_widths(d, dv);
  return walk_possible(d, dv, M) && !(many && M <= 64 && !x.even && x.all >= 6 && d <= 64);
}

int launch_gen_walk(const GenSide& qs, const GenSide& ks, const TensorDev& V, int L, int BH, int H, int M, int d, int nv, int ldt,
                    int rows_per_seg, int nseg, const uint32_t* kmax_u, const float* Tstate, const TensorDev& Y, float* den_out,
                    float* shift_out, hipStream_t st, unsigned* flushed) {
  WalkArgs a{ks, qs, V, V, nv, 1, 0, 0, L, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, nullptr, Tstate, Y, den_out, shift_out, flushed};
  return run_walk<0>(a, BH, st);
}

int launch_gen_bwd_walks(const GenSide& qs, const GenSide& ks, const TensorDev& V, const float* ghat, int L, int BH, int H, int M, int d,
                         int nv, int ldt, int rows_per_seg, int nseg, const uint32_t* kmax_u, const float* row_shift,
                         const float* Tstate, const float* Rstate, const TensorDev& dQ, const TensorDev& dK, const TensorDev& dV,
                         hipStream_t st) {
  const TensorDev G{ghat, 0, (long long)H * L * ldt, (long long)L * ldt, (long long)ldt};
  WalkArgs a{ks, qs, V, G, nv, 1, ldt, 0, L, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, row_shift, Tstate, dQ, nullptr, nullptr, nullptr};
  if (int rc = run_gwalk<0>(a, BH, st)) return rc;
  WalkArgs r{qs, ks, G, V, ldt, 0, nv, 1, L, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, row_shift, Rstate, dV, nullptr, nullptr, nullptr};
  if (int rc = run_walk<1>(r, BH, st)) return rc;
  r.out = dK;
  return run_gwalk<1>(r, BH, st);
}

}  // namespace fs
