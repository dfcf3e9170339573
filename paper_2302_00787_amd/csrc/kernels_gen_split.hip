// General-shape causal kernels on bf16 matrix instructions with fp32 accuracy (split3.h): d and dv multiples of four, M up to 512,
// bf16 rows up to 128 numbers, fp32 rows up to 64 (others: kernels_gen_walk.hip, whose design this is).
//
// A workgroup walks a segment of a sequence 32 tokens at a time; a wave holds 32 features: its part of the state stays in
// accumulators.  More than 256 features go in two launches, the second of which adds the first one's rows to its own (more
// features per wave do not fit its registers: 200 - 365 of them spilled, 920 - 1250 us a walk where two launches take 330).  Rows lie in LDS as bf16 pieces (bf16 tensors: one piece, exact; qk_scale is folded into W~), W~ comes from L2 as
// operand images of pieces, once per chunk.  Every other operand is made of accumulators: two stacked 16-row accumulators are, per
// lane, the eight numbers of an operand whose contraction index runs 16 (e / 4) + 4 g + e % 4 (lane l = (g, c) = (l / 16, l % 16)),
// and value rows are read in that order with the transposing LDS read.
//
// What bounds it: the matrix pipe needs 96 cycles for 16 x 16 x 32 numbers (48 against bf16 tensors; fp32 instructions 256), splitting an
// accumulator pair 28 vector instructions; W~ is 6 bytes per feature and coordinate and chunk from L2.  Two waves per SIMD overlap the two
// pipes about half.  Against fp32 instructions: causal attention f32 B2 H4 L4096 d64 M256 147 -> 107 us (walk 87 -> 61, states 38 -> 25),
// gradients bf16 B1 H16 L4096 d128 M512 3510 -> 1660 (four walks 2570 -> 1325 in eight launches, two states 680 -> 190), results
// of 60 drawn calls 0.93 times as far from 64 bits.
#include <type_traits>

#include "gen_widths.h"
#include "kernels.h"
#include "split3.h"

namespace fs {
namespace {

using namespace gen;

constexpr int TT = 32;                                   // tokens per chunk
constexpr int FT = 2;                                    // tiles of 16 features per wave: one operand
template <int Q> constexpr int KS = (Q + 1) / 2;         // steps of 32 coordinates
template <int Q> constexpr int VTP = (VT_OF<Q> + 1) / 2 * 2;
constexpr int LDR(int cols) { return cols + 8; }         // stride of LDS rows (bf16 numbers)
constexpr int IMG = 512;                                 // numbers of an operand image
// Pieces of numbers below 2^-109 lose bits, so no operand is left there.  Features lie in 2^-126 .. 1 (a causal row may see only keys
// whose features are that far below the largest of the sequence); they are lifted by 2^12 before they are split: one of 2^-126 is then off
// by 2^-20 of itself, less than by the rounding of its exponent, 2^-18.  Output rows and their normalisers have 2^24, which the quotient
// loses; a sum with one feature of either side (dV) has 2^24, one with a feature of one side (R, dQ, dK) 2^12.
// Values, dY and G1 are divided by powers of two, found for each sequence beside the constants (k_prep) and the G1 rows (k_bwd_ghat):
//   V     its largest number is left where it is from 2^-16 to 2^48, brought to one below and to 2^48 above, so that it does not leave the
//         range with the lift, nor with the sums over a million tokens;
//   dY    its largest number is brought to one, so that G1, a normaliser's size off, is neither subnormal nor infinite;
//   G1    its largest number is brought to 2^64 (a product with a value is at most about that: the last column is such a product,
//         summed), so that rows far below the largest have all pieces, down to 2^-125 of it and less.
// (Keys 2^-121 below the largest: outputs up to 1.8e-5 off without the lift, gradients 5e-4, now 3e-7 and 6e-6, as with fp32
// instructions; V or dY near 2^-120, or rows of dY 2^-105 and of V 2^-100 below the largest: up to 1 off where numbers are
// divided by the largest of V and dY alone, 8e-3 undivided, now 2e-7 - 8e-7.  Causal f32 B2 H4 L4096 d64 M256 106.5 -> 108.3 us; gradients
// bf16 B1 H16 L4096 d128 M512 1622 -> 1658, of which the maxima 10.)
constexpr int LIFT = 12;
constexpr float kLift = 1 << LIFT;
constexpr float kLeastSum = 0x1p-125f;                   // kLift^2 times the least fp32 number: below it a normaliser counts as zero

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
__device__ __forceinline__ u32x2 read_tr(const uint16_t* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p)));
}
__device__ __forceinline__ bf16x8 join(u32x2 a, u32x2 b) { return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]}); }

// P pieces of an operand.
template <int P> struct Op { bf16x8 p[P]; };
template <int P>
__device__ __forceinline__ Op<P> row_op(const uint16_t* s, int plane) {       // eight numbers of a row
  Op<P> o;
#pragma unroll
  for (int i = 0; i < P; ++i) o.p[i] = *(const bf16x8*)(s + i * plane);
  return o;
}
template <int P>
__device__ __forceinline__ Op<P> pair_op(const uint16_t* s, int plane) {      // four numbers of a row and the four sixteen further
  Op<P> o;
#pragma unroll
  for (int i = 0; i < P; ++i) o.p[i] = join(*(const u32x2*)(s + i * plane), *(const u32x2*)(s + i * plane + 16));
  return o;
}
template <int P>
__device__ __forceinline__ Op<P> column_op(const uint16_t* s, int ld, int plane) {   // a column of rows 4 g .. and 16 + 4 g ..
  Op<P> o;
#pragma unroll
  for (int i = 0; i < P; ++i) o.p[i] = join(read_tr(s + i * plane), read_tr(s + i * plane + 16 * ld));
  return o;
}
template <int PART = ALL>
__device__ __forceinline__ f32x4 times(const Split3& a, const Op<1>& b, f32x4 c) {
  c = mfma_bf16<PART>(a.l, b.p[0], c);
  c = mfma_bf16<PART>(a.m, b.p[0], c);
  return mfma_bf16<PART>(a.h, b.p[0], c);
}
__device__ __forceinline__ f32x4 times(const Op<1>& a, const Split3& b, f32x4 c) {
  c = mfma_bf16(a.p[0], b.l, c);
  c = mfma_bf16(a.p[0], b.m, c);
  return mfma_bf16(a.p[0], b.h, c);
}
__device__ __forceinline__ Split3 as_split(const Op<3>& a) { return {a.p[0], a.p[1], a.p[2]}; }
template <int PART = ALL>
__device__ __forceinline__ f32x4 times(const Split3& a, const Op<3>& b, f32x4 c) { return mfma3<PART>(a, as_split(b), c); }
__device__ __forceinline__ f32x4 times(const Op<3>& a, const Split3& b, f32x4 c) { return mfma3_t(as_split(a), b, c); }
__device__ __forceinline__ f32x4 times(const Op<1>& a, const Op<3>& b, f32x4 c) { return times(a, as_split(b), c); }
__device__ __forceinline__ f32x4 times(const Op<3>& a, const Op<1>& b, f32x4 c) { return times(as_split(a), b, c); }
__device__ __forceinline__ f32x4 times(const Op<3>& a, const Op<3>& b, f32x4 c) { return mfma3(as_split(a), as_split(b), c); }

// Rows of a tensor on their way global -> registers -> LDS: TT rows of COLS numbers, four numbers per thread and piece of work.
// P == 1: a bf16 tensor, copied; P == 3: an fp32 tensor, split.
struct RowSrc {
  const void* ptr;
  long long base, sl;
  int ncols;               // numbers per row (a multiple of four); column ncols of a live row is `one`, the rest zero
  int one;
};
__device__ __forceinline__ RowSrc row_src(const TensorDev& t, int b, int h, int first, int ncols, int one) {
  return RowSrc{t.ptr, b * t.sb + h * t.sh + first, t.sl, ncols, one};
}
template <int COLS, int NW, int P> struct Fetch {
  static constexpr int N = (TT * COLS / 4 + 64 * NW - 1) / (64 * NW);
  typename std::conditional<P == 1, u32x2, u32x4>::type v[N];
  __device__ __forceinline__ void get(const RowSrc& s, int row0, int row_end, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = tid + 64 * NW * i, row = min(e / (COLS / 4), TT - 1), col = 4 * (e % (COLS / 4));
      const long long at = s.base + (long long)min(row0 + row, row_end - 1) * s.sl + min(col, s.ncols - 4);
      if constexpr (P == 1) v[i] = *(const u32x2*)((const uint16_t*)s.ptr + at);
      else v[i] = *(const u32x4*)((const float*)s.ptr + at);
    }
  }
  // exponent: the numbers are divided by 2^exponent
  __device__ __forceinline__ void put(const RowSrc& s, uint16_t* dst, int row0, int row_end, int tid, int exponent = 0) {
    constexpr int LD = LDR(COLS), PLANE = TT * LD;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int e = tid + 64 * NW * i, row = e / (COLS / 4), col = 4 * (e % (COLS / 4));
      if (row >= TT) continue;
      const bool live = row0 + row < row_end, in = live && col < s.ncols, one = live && s.one && col == s.ncols;
      uint16_t* at = dst + row * LD + col;
      if constexpr (P == 1) {
        u32x2 x = v[i];
        if (__builtin_amdgcn_readfirstlane(exponent) != 0) {                 // (exact but for numbers that leave the exponent range)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            x[j] = __float_as_uint(ldexpf(__uint_as_float(x[j] << 16), -exponent)) >> 16 |
                   (__float_as_uint(ldexpf(__uint_as_float(x[j] & 0xffff0000u), -exponent)) & 0xffff0000u);
        }
        *(u32x2*)at = in ? x : u32x2{one ? 0x3f80u : 0u, 0u};
      } else {
        f32x4 x = __builtin_bit_cast(f32x4, v[i]);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = ldexpf(x[j], -exponent);
        x = in ? x : f32x4{one ? 1.f : 0.f, 0.f, 0.f, 0.f};
        const Split3 q = split3_each(x, x);
        const u32x4 h = __builtin_bit_cast(u32x4, q.h), m = __builtin_bit_cast(u32x4, q.m), l = __builtin_bit_cast(u32x4, q.l);
        *(u32x2*)at = u32x2{h[0], h[1]};
        *(u32x2*)(at + PLANE) = u32x2{m[0], m[1]};
        *(u32x2*)(at + 2 * PLANE) = u32x2{l[0], l[1]};
      }
    }
  }
};

// The exponents that V and G1 are divided by, of their largest numbers.
__device__ __forceinline__ int value_exponent(float largest) {
  const int e = __builtin_amdgcn_frexp_expf(largest);
  return e < -16 ? e : max(e - 48, 0);
}
__device__ __forceinline__ int left_exponent(float largest) { return __builtin_amdgcn_frexp_expf(largest) - 64; }

struct SplitArgs {
  GenSide F, S;            // first side (whose rows enter the state), second side (whose rows are the output's)
  TensorDev V, U;          // values of the first side's rows; (gradient walk) left rows of the second side
  int vcols, vone, ucols, uone;
  int L, BH, H, M, d, nv, ldt, rows_per_seg, nseg, ntile;
  const uint16_t* img;     // [pgroups][2][ntile][KS][3][IMG]: W~ times qk_scale, a lane's feature against eight coordinates
  const uint16_t* img_t;   // [pgroups][2][ntile / 2][2 KS][3][IMG]: a lane's coordinate against eight features
  uint32_t* kmax_u;
  const float* part;       // partial key maxima (k_gen_kmax) or nullptr: kmax_u has the maximum
  int npart;
  const float *vmax, *dmax;    // [BH][nvmax] partial maxima of |V|, |dY|; behind k_bwd_ghat dmax has those of |G1|, of GMAX_ROWS rows
  int nvmax;
  int* exps;               // [BH] exponents that V is divided by; (gradients) [3][BH], those of dY and G1 behind them
  const float* row_shift;  // [BH][L] shifts of the queries
  float* state;            // [BH][nseg][M][ldt]: sums of the segments (written), exclusive prefix or suffix (read)
  TensorDev out;
  float *den_out, *shift_out;
  unsigned* flushed;
  int tile0;               // the launch's first tile of features
  int bh0, nbh;            // its first sequence, sequences
  float *part_out, *part_in;   // [nbh][L][ldp] rows of a launch that is not the last, of the one before it
  int ldp;
};

// (a uniform base and a 32-bit offset found anew for every chunk: addresses kept across chunks are spilled, and a spilled address is
// a memory latency ahead of the load)
__device__ __forceinline__ uint32_t image_lane(int lane) {
  uint32_t at = 16u * (uint32_t)lane;
  asm volatile("" : "+v"(at));
  return at;
}
__device__ __forceinline__ Split3 image_op(const uint16_t* img, uint32_t at) {
  const char* p = (const char*)img;
  return {*(const bf16x8*)(p + at), *(const bf16x8*)(p + 2 * IMG + at), *(const bf16x8*)(p + 4 * IMG + at)};
}
template <int Q>
__device__ __forceinline__ const uint16_t* side_image(const SplitArgs& a, const uint16_t* img, int pg, int side) {
  return img + ((size_t)pg * 2 + side) * a.ntile * KS<Q> * 3 * IMG;
}

// Segment and sequence of a workgroup.  Workgroups go to the eight XCDs in turn; the segments of a sequence go to one XCD, one after
// the other, so that its L2 holds the images they all read (16 heads, d 128, M 512: 6 MB for an XCD that serves all of them).
__device__ __forceinline__ void segment_of(int& seg, int& bh, int bh0) {
  const unsigned total = gridDim.x * gridDim.y, id = blockIdx.x + gridDim.x * blockIdx.y, xcd = id % 8, per = total / 8, rest = total % 8;
  const unsigned at = xcd * per + min(xcd, rest) + id / 8;
  const int at_bh = at / gridDim.x;
  seg = at - at_bh * gridDim.x;
  bh = bh0 + at_bh;
}

// Exponents (without bias) of N tiles of 16 features, from f0 / 16 on, against the chunk's rows at Xs.  FEATURE_ROWS: rows = features
// 4 g + r, column = token c; else rows = tokens, column = feature.  Two steps of W~ are on their way while one is used.
template <bool FEATURE_ROWS, int Q, int N, int XP>
__device__ __forceinline__ void project(f32x4 (&acc)[N][2], const uint16_t* W, const uint16_t* Xs, int lane) {
  constexpr int K = KS<Q>, STEPS = N * K, LD = LDR(32 * K), PLANE = TT * LD, AHEAD = 2;
  const int g = lane >> 4, c = lane & 15;
  const uint32_t at = image_lane(lane);
  asm volatile("" : "+s"(W));
  Split3 w[AHEAD + 1];
#pragma unroll
  for (int s = 0; s < AHEAD && s < STEPS; ++s) w[s] = image_op(W + (size_t)s * 3 * IMG, at);
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    __builtin_amdgcn_sched_barrier(0);
    if (s + AHEAD < STEPS) w[(s + AHEAD) % (AHEAD + 1)] = image_op(W + (size_t)(s + AHEAD) * 3 * IMG, at);
    const int n = s / K, k = s % K;
    const Split3& ww = w[s % (AHEAD + 1)];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const Op<XP> x = row_op<XP>(Xs + (16 * t + c) * LD + 32 * k + 8 * g, PLANE);
      const f32x4 z = k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[n][t];
      acc[n][t] = FEATURE_ROWS ? times(ww, x, z) : times(x, ww, z);
    }
  }
}

// What a token of a side brings to its exponents: - its shift (queries), its row term (keys, whose shift is the key
// maximum), -inf past the end; and an exponent of it, in the order of the other kernels (kernels_gen_rows.hip).
template <bool KEYS>
__device__ __forceinline__ float side_term(const SplitArgs& a, const GenSide& sd, int bh, int row, int row_end) {
  if (row >= row_end) return -INFINITY;
  return KEYS ? sd.rk[(size_t)bh * a.L + row] : -a.row_shift[(size_t)bh * a.L + row];
}
template <bool KEYS>
__device__ __forceinline__ float exponent(float e, float bias, float term, float kmax) {
  return KEYS ? ((e + bias) + term) - kmax : (e + bias) + term;
}

// ---------------------------------------------------------------------------------------------------
// State of a segment: sum over its rows of F (features) x V.  KEYS: keys with [V 1]; else queries with the rows of G1.
// grid (nseg, B*H, blocks of 32 NW features), block 64 NW.
// ---------------------------------------------------------------------------------------------------
template <int Q, int NW, int XP, int VP> constexpr size_t state_lds() {
  return 2 * (size_t)TT * (XP * LDR(32 * KS<Q>) + VP * LDR(16 * VT_OF<Q>));
}
template <int Q, int NW, int XP, int VP, bool KEYS>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) k_split_state(SplitArgs a) {
  extern __shared__ __align__(16) uint16_t lds16[];
  constexpr int VT = VT_OF<Q>, XC = 32 * KS<Q>, VC = 16 * VT, LDV = LDR(VC), VPLANE = TT * LDV;
  uint16_t *Xs = lds16, *Vs = Xs + XP * TT * LDR(XC);
  int seg, bh;
  segment_of(seg, bh, a.bh0);
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  int g = lane >> 4, c = lane & 15;
  a.tile0 = FT * NW * blockIdx.z;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fw = 16 * FT * w, f0 = 16 * a.tile0 + fw;
  const int pg = group_of(a.F.pgroups, b, h, a.H), M = a.M;
  const uint16_t* W = side_image<Q>(a, a.img, pg, KEYS) + (size_t)(a.tile0 + FT * w) * KS<Q> * 3 * IMG;
  const float* bias = a.F.bias + (size_t)pg * 2 * M;
  const int row_beg = seg * a.rows_per_seg, row_end = min(a.L, row_beg + a.rows_per_seg);
  const RowSrc xf = row_src(a.F.X, b, h, 0, a.d, 0), vf = row_src(a.V, b, h, 0, a.vcols, a.vone);
  Fetch<XC, NW, XP> px;
  Fetch<VC, NW, VP> pv;
  // (the first partial maxima of each lane are requested ahead of the rows: their reduction waits for no more than them)
  const bool first = seg == 0 && blockIdx.z == 0;             // leaves what was found for the kernels behind this one
  const int nmax = KEYS ? a.nvmax : (a.L + GMAX_ROWS - 1) / GMAX_ROWS;
  const float *vmax = (KEYS ? a.vmax : a.dmax) + (size_t)bh * nmax, *kpart = a.part + (size_t)bh * a.npart;
  float vm = vmax[min(lane, nmax - 1)], km = KEYS && a.part != nullptr ? kpart[min(lane, a.npart - 1)] : 0.f, kmax = 0.f;
  px.get(xf, row_beg, row_end, threadIdx.x);
  pv.get(vf, row_beg, row_end, threadIdx.x);
  for (int i = lane + 64; i < nmax; i += 64) vm = fmaxf(vm, vmax[i]);
  if (KEYS && a.part != nullptr)
    for (int i = lane + 64; i < a.npart; i += 64) km = fmaxf(km, kpart[i]);
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    if (KEYS) km = fmaxf(km, __shfl_xor(km, s));
    vm = fmaxf(vm, __shfl_xor(vm, s));
  }
  const int ve = KEYS ? value_exponent(vm) : left_exponent(vm);
  if (KEYS) {
    kmax = a.part != nullptr ? km : ordered_to_float(a.kmax_u[bh]);
    if (first && a.dmax != nullptr) {
      float dm = 0.f;
      for (int i = lane; i < nmax; i += 64) dm = fmaxf(dm, a.dmax[(size_t)bh * nmax + i]);
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) dm = fmaxf(dm, __shfl_xor(dm, s));
      if (threadIdx.x == 0) a.exps[a.BH + bh] = __builtin_amdgcn_frexp_expf(dm);
    }
    if (first && threadIdx.x == 0) {
      if (a.part != nullptr) a.kmax_u[bh] = float_to_ordered(km);
      a.exps[bh] = ve;
    }
  } else if (first && threadIdx.x == 0) {
    a.exps[2 * a.BH + bh] = ve;
  }
  float bf[FT];
  f32x4 T[FT][VT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int f = f0 + 16 * ft + c;
    bf[ft] = f < M ? bias[f] : -INFINITY;
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) T[ft][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int row0 = row_beg; row0 < row_end; row0 += TT) {
    asm volatile("" : "+v"(g), "+v"(c));             // (nothing that follows from the lane is kept across chunks)
    __syncthreads();
    px.put(xf, Xs, row0, row_end, threadIdx.x);
    pv.put(vf, Vs, row0, row_end, threadIdx.x, ve);
    __syncthreads();
    if (row0 + TT < row_end) {
      px.get(xf, row0 + TT, row_end, threadIdx.x);
      pv.get(vf, row0 + TT, row_end, threadIdx.x);
    }
    float add[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) add[t][r] = side_term<KEYS>(a, a.F, bh, row0 + 16 * t + 4 * g + r, row_end);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      f32x4 s[1][2];
      project<false, Q, 1, XP>(s, W + (size_t)ft * KS<Q> * 3 * IMG, Xs, lane);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[0][t][r] = kLift * fast_exp2(exponent<KEYS>(s[0][t][r], bf[ft], add[t][r], kmax));
      const Split3 so = split3(s[0][0], s[0][1]);
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        const Op<VP> v = column_op<VP>(Vs + (4 * g + (c >> 2)) * LDV + 16 * vt + 4 * (c & 3), LDV, VPLANE);
        T[ft][vt] = times(so, v, T[ft][vt]);
      }
    }
  }
  float* out = a.state + ((size_t)bh * a.nseg + seg) * M * a.ldt;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int vt = 0; vt < VT; ++vt)
      if (16 * vt < a.ldt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = f0 + 16 * ft + 4 * g + r;
          if (m < M) out[(size_t)m * a.ldt + 16 * vt + c] = T[ft][vt][r];
        }
      }
}

// ---------------------------------------------------------------------------------------------------
// Output walk.  MODE 0 (forwards): first side keys with [V 1], output Y of the queries, whose features are shifted by the
// wave's own maximum of the row; the waves' partial rows are brought to the row's maximum where they are summed.
// MODE 1 (backwards): first side queries with the rows of G1, output dV of the keys.  The partial rows of more than 80 columns meet in
// two blocks, the one with the normaliser first.  grid (nseg, B*H), block 64 NW.
//   y_i = P_i T + sum_j tril(P_i S_j) V_j ;  T += S^T V
// ---------------------------------------------------------------------------------------------------
template <int Q> constexpr int VB = VT_OF<Q> < 5 ? VT_OF<Q> : 5;        // tiles of columns per block
constexpr int LDS_F = 36;                                // stride of a wave's feature rows in LDS: 32 features and padding
template <int Q> constexpr int XCH = TT * (16 * VB<Q> + 1) > 3 * TT * LDS_F / 2 ? TT * (16 * VB<Q> + 1) : 3 * TT * LDS_F / 2;
template <int Q, int NW, int XP, int VP> constexpr size_t walk_lds() {
  return 4 * ((size_t)NW * XCH<Q> + NW * TT + 16 * FT * NW) + 2 * (size_t)TT * (2 * XP * LDR(32 * KS<Q>) + VP * LDR(16 * VT_OF<Q>));
}

template <int Q, int NW, int XP, int VP, int MODE>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) k_split_walk(SplitArgs a) {
  extern __shared__ __align__(16) uint16_t lds16[];
  constexpr int VT = VT_OF<Q>, XC = 32 * KS<Q>, VC = 16 * VT, LDV = LDR(VC), VPLANE = TT * LDV, ldo = 16 * VB<Q> + 1, XROWS = XP * TT * LDR(XC);
  uint16_t *Xf = lds16, *Xs = Xf + XROWS, *Vs = Xs + XROWS;
  float* xch = (float*)(Vs + VP * VPLANE);         // [wave][token][column]; before that the wave's transposition of first-side features
  float* mw = xch + NW * XCH<Q>;                   // [wave][token]: row maxima
  float* bl = mw + NW * TT;                        // biases, -inf behind the last feature
  int seg, bh;
  segment_of(seg, bh, a.bh0);
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  int g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fw = 16 * FT * w, f0 = 16 * a.tile0 + fw;
  const int pg = group_of(a.F.pgroups, b, h, a.H), M = a.M;
  constexpr bool F_KEYS = MODE == 0;
  const size_t wave_w = (size_t)(a.tile0 + FT * w) * KS<Q> * 3 * IMG;
  const uint16_t* W1 = side_image<Q>(a, a.img, pg, F_KEYS) + wave_w;
  const uint16_t* W2 = side_image<Q>(a, a.img, pg, !F_KEYS) + wave_w;
  const float* bias = a.F.bias + (size_t)pg * 2 * M;        // (the same on both sides)
  const float kmax = ordered_to_float(a.kmax_u[bh]);
  int ve = MODE ? a.exps[2 * a.BH + bh] : a.exps[bh];                                    // of the values, of the output
  int back = MODE ? ve + a.exps[a.BH + bh] - 2 * LIFT : a.den_out == nullptr ? ve : 0;
  asm("" : "+v"(ve), "+v"(back));                    // (scalar registers are what runs out)
  const int row_beg = seg * a.rows_per_seg, row_end = min(a.L, row_beg + a.rows_per_seg);
  const int nchunk = (row_end - row_beg + TT - 1) / TT;
  const RowSrc xf = row_src(a.F.X, b, h, 0, a.d, 0), xs = row_src(a.S.X, b, h, 0, a.d, 0), vf = row_src(a.V, b, h, 0, a.vcols, a.vone);
  auto row_of = [&](int ci) { return row_beg + TT * (MODE ? nchunk - 1 - ci : ci); };

  Fetch<XC, NW, XP> pf, ps;
  Fetch<VC, NW, VP> pv;
  auto fetch_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                       // (nothing of the addresses is kept across chunks: registers)
    const int r0 = row_of(ci);
    pf.get(xf, r0, row_end, tid);
    ps.get(xs, r0, row_end, tid);
    pv.get(vf, r0, row_end, tid);
  };
  auto put_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int r0 = row_of(ci);
    pf.put(xf, Xf, r0, row_end, tid);
    ps.put(xs, Xs, r0, row_end, tid);
    pv.put(vf, Vs, r0, row_end, tid, ve);
  };
  fetch_chunk(0);
  for (int f = threadIdx.x; f < 16 * FT * NW; f += 64 * NW) bl[f] = 16 * a.tile0 + f < M ? bias[16 * a.tile0 + f] : -INFINITY;
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
  uint16_t* lt = (uint16_t*)(xch + w * XCH<Q>);      // [3][token][32 features]
  for (int ci = 0; ci < nchunk; ++ci) {
    asm volatile("" : "+v"(g), "+v"(c));             // (nothing that follows from the lane is kept across chunks)
    const int row0 = row_of(ci);
    float addf[2], adds[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      addf[t] = side_term<F_KEYS>(a, a.F, bh, row0 + 16 * t + c, row_end);
      adds[t] = MODE ? side_term<true>(a, a.S, bh, row0 + 16 * t + c, row_end) : 0.f;
    }
    __syncthreads();
    // features of both sides: rows = features, column = token
    f32x4 sf[FT][2], p[FT][2];
    project<true, Q, FT, XP>(sf, W1, Xf, lane);
    project<true, Q, FT, XP>(p, W2, Xs, lane);
    __builtin_amdgcn_sched_barrier(0);
    float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const f32x4 br = *(const f32x4*)(bl + fw + 16 * ft + 4 * g);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sf[ft][t][r] = kLift * fast_exp2(exponent<F_KEYS>(sf[ft][t][r], br[r], addf[t], kmax));
          if (MODE) {
            p[ft][t][r] = kLift * fast_exp2(exponent<true>(p[ft][t][r], br[r], adds[t], kmax));
          } else {
            p[ft][t][r] += br[r];
            m[t] = fmaxf(m[t], p[ft][t][r]);
          }
        }
    }
    if (!MODE) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        m[t] = fmaxf(m[t], __shfl_xor(m[t], 16));
        m[t] = fmaxf(m[t], __shfl_xor(m[t], 32));
        if (g == 0) mw[w * TT + 16 * t + c] = m[t];
        const float ms = m[t] == -INFINITY ? 0.f : m[t];         // (a wave behind the last feature)
#pragma unroll
        for (int ft = 0; ft < FT; ++ft)
#pragma unroll
          for (int r = 0; r < 4; ++r) p[ft][t][r] = kLift * fast_exp2(p[ft][t][r] - ms);
      }
    }
    f32x4 sc[2][2], y[2][VT];      // scores (rows = first-side tokens, column = second-side token), output rows
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      sc[0][t] = sc[1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) y[t][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const uint16_t* vcol = Vs + (4 * g + (c >> 2)) * LDV + 4 * (c & 3);
    __builtin_amdgcn_sched_barrier(0);
    {
      Split3 so[2], po[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        so[t] = split3(sf[0][t], sf[1][t]);
        po[t] = split3(p[0][t], p[1][t]);
        // the first side's features with tokens as the contraction, by way of the wave's LDS scratch
        const bf16x8 pieces[3] = {so[t].h, so[t].m, so[t].l};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const u32x4 q = __builtin_bit_cast(u32x4, pieces[i]);
          uint16_t* at = lt + i * TT * LDS_F + (16 * t + c) * LDS_F + 4 * g;
          *(u32x2*)at = u32x2{q[0], q[1]};
          *(u32x2*)(at + 16) = u32x2{q[2], q[3]};
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int tf = 0; tf < 2; ++tf)
          if (MODE ? tf >= t : tf <= t) sc[tf][t] = mfma3(so[tf], po[t], sc[tf][t]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        __builtin_amdgcn_sched_barrier(0);             // (registers: here and below)
        const Split3 ts = split3(T[0][vt], T[1][vt]);
        y[0][vt] = mfma3(po[0], ts, y[0][vt]);
        y[1][vt] = mfma3(po[1], ts, y[1][vt]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int tf = 0; tf < 2; ++tf)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int first = 16 * tf + 4 * g + r, second = 16 * t + c;
          sc[tf][t][r] = (MODE ? first >= second : first <= second) ? sc[tf][t][r] : 0.f;
        }
    }
    {
      Split3 su[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        su[i] = as_split(column_op<3>(lt + (4 * g + (c >> 2)) * LDS_F + 16 * i + 4 * (c & 3), LDS_F, TT * LDS_F));
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        __builtin_amdgcn_sched_barrier(0);
        const Op<VP> v = column_op<VP>(vcol + 16 * vt, LDV, VPLANE);
        T[0][vt] = times(su[0], v, T[0][vt]);
        T[1][vt] = times(su[1], v, T[1][vt]);
      }
    }
    if (ci + 1 < nchunk) fetch_chunk(ci + 1);          // the next chunk's rows travel meanwhile
    {
      Split3 so[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) so[t] = split3(sc[0][t], sc[1][t]);
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        __builtin_amdgcn_sched_barrier(0);
        const Op<VP> v = column_op<VP>(vcol + 16 * vt, LDV, VPLANE);
        y[0][vt] = times<MODE ? ALL : LOW>(so[0], v, y[0][vt]);
        y[1][vt] = times<MODE ? HIGH : ALL>(so[1], v, y[1][vt]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // the waves' rows summed, 2 NW threads per row
    const int row = threadIdx.x / (2 * NW), l = threadIdx.x % (2 * NW);
    const bool live = row0 + row < row_end;
    const size_t rec = (size_t)bh * a.L + row0 + row, prec = (size_t)(bh - a.bh0) * a.L + row0 + row;
    float wgt[NW], wpart = 0.f, mm = -INFINITY, den = 1.f;
#pragma unroll
    for (int vb = (VT - 1) / VB<Q> * VB<Q>; vb >= 0; vb -= VB<Q>) {
      if (vb > a.nv / 16) continue;                              // (no columns there)
      const bool with_den = vb + VB<Q> > a.nv / 16;
      if (!with_den) __syncthreads();                            // the last block's rows have been summed
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int vt = vb; vt < vb + VB<Q> && vt < VT; ++vt)
#pragma unroll
          for (int r = 0; r < 4; ++r) xch[w * XCH<Q> + (16 * t + 4 * g + r) * ldo + 16 * (vt - vb) + c] = y[t][vt][r];
      __syncthreads();
      const int base = 16 * vb, cols = min(16 * VB<Q>, a.nv - base);
      const float* at = xch + row * ldo;
      if (!MODE && with_den) {                                   // shifts and normaliser
#pragma unroll
        for (int i = 0; i < NW; ++i) mm = fmaxf(mm, mw[i * TT + row]);
        float before = -INFINITY;
        if (a.part_in != nullptr && live) before = a.part_in[prec * a.ldp + a.ldt];
        mm = fmaxf(mm, before);
        wpart = before == -INFINITY ? 0.f : fast_exp2(before - mm);
        den = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          const float mi = mw[i * TT + row];
          wgt[i] = mi == mm ? 1.f : fast_exp2(mi - mm);
          den += wgt[i] * at[i * XCH<Q> + a.nv - base];
        }
        if (a.part_in != nullptr && live) den += wpart * a.part_in[prec * a.ldp + a.nv];
        if (live && l == 0) {
          if (a.part_out != nullptr) {
            a.part_out[prec * a.ldp + a.nv] = den;
            a.part_out[prec * a.ldp + a.ldt] = mm;
          } else {
            if (a.flushed != nullptr && !(den > kLeastSum)) atomicAdd(a.flushed, 1u);
            if (a.den_out != nullptr) {
              a.den_out[rec] = den > kLeastSum ? den : 0.f;
              a.shift_out[rec] = mm;
            }
          }
        }
      }
      if (live) {
        const long long ob = b * a.out.sb + h * a.out.sh + (long long)(row0 + row) * a.out.sl;
        for (int col = l; col < cols; col += 2 * NW) {
          float v = 0.f;
#pragma unroll
          for (int i = 0; i < NW; ++i) v += (MODE ? 1.f : wgt[i]) * at[i * XCH<Q> + col];
          if (a.part_in != nullptr) v += (MODE ? 1.f : wpart) * a.part_in[prec * a.ldp + base + col];
          if (a.part_out != nullptr) {
            a.part_out[prec * a.ldp + base + col] = v;
          } else {
            if (!MODE) v = den > kLeastSum ? ldexpf(v / den, back) : 0.f;
            else v = ldexpf(v, back);
            store_elem(a.out, ob + base + col, v);
          }
        }
      }
    }
    if (ci + 1 < nchunk) put_chunk(ci + 1);
  }
}

// ---------------------------------------------------------------------------------------------------
// Gradient walk.  MODE 0 (forwards): first side keys with [V 1], second side queries with left rows G1 -> dQ.  MODE 1 (backwards): first
// side queries with G1, second side keys with left rows [V 1] -> dK.
//   dF_i = Z u_i + sum_j tril(u_i . v_j) F_j ;  dE = F_second * dF ;  gradient = dE W~ (+ row term) ;  Z += F_first^T V
// The state is held transposed (rows = columns of the values, column = feature): as it lies it is the operand of dF.  The gradient's
// coordinates go in blocks of 64: the waves' partial rows of a block fit in LDS, its accumulators in registers.
// grid (nseg, B*H), block 64 NW.
// ---------------------------------------------------------------------------------------------------
template <int Q> constexpr int GC = Q < 4 ? 16 * Q : 64;       // coordinates per block
template <int Q, int NW, int XP, int VP, int UP> constexpr size_t gwalk_lds() {
  return 4 * ((size_t)NW * TT * (GC<Q> + 1) + NW * TT + 16 * FT * NW + TT * (16 * Q + 4)) +
         2 * (size_t)TT * (2 * XP * LDR(32 * KS<Q>) + (VP + UP) * LDR(16 * VTP<Q>));
}

template <int Q, int NW, int XP, int MODE>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) k_split_gwalk(SplitArgs a) {
  extern __shared__ __align__(16) uint16_t lds16[];
  constexpr int VP = MODE ? 3 : XP, UP = MODE ? XP : 3;
  constexpr int VT = VT_OF<Q>, NV = VTP<Q> / 2, XC = 32 * KS<Q>, VC = 16 * VTP<Q>, LDX = LDR(XC), LDV = LDR(VC);
  constexpr int XPLANE = TT * LDX, VPLANE = TT * LDV, DT = GC<Q> / 16, ldo = GC<Q> + 1, ldc = 16 * Q + 4;
  uint16_t *Xf = lds16, *Xs = Xf + XP * XPLANE, *Vs = Xs + XP * XPLANE, *Us = Vs + VP * VPLANE;
  float* xch = (float*)(Us + UP * VPLANE);         // [wave][token][coordinate]
  float* rsw = xch + NW * TT * ldo;                // [wave][token]: row sums of dE
  float* bl = rsw + NW * TT;                       // biases, -inf behind the last feature
  float* cx = bl + 16 * FT * NW;                   // [token][coordinate]: x (C + C^T), where the kernel has a C
  int seg, bh;
  segment_of(seg, bh, a.bh0);
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  int g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), fw = 16 * FT * w, f0 = 16 * a.tile0 + fw;
  const int pg = group_of(a.F.pgroups, b, h, a.H), M = a.M, d = a.d;
  constexpr bool F_KEYS = MODE == 0;
  const size_t wave_w = (size_t)(a.tile0 + FT * w) * KS<Q> * 3 * IMG;
  const uint16_t* W1 = side_image<Q>(a, a.img, pg, F_KEYS) + wave_w;
  const uint16_t* W2 = side_image<Q>(a, a.img, pg, !F_KEYS) + wave_w;
  const uint16_t* Wt = side_image<Q>(a, a.img_t, pg, !F_KEYS) + wave_w;
  const float* bias = a.F.bias + (size_t)pg * 2 * M;
  const float kmax = ordered_to_float(a.kmax_u[bh]), scale = a.S.scale;
  int ve = a.exps[bh], ge = a.exps[2 * a.BH + bh], back = ve + ge + a.exps[a.BH + bh] - LIFT;
  asm("" : "+v"(ve), "+v"(ge), "+v"(back));
  const int row_beg = seg * a.rows_per_seg, row_end = min(a.L, row_beg + a.rows_per_seg);
  const int nchunk = (row_end - row_beg + TT - 1) / TT;
  const RowSrc xf = row_src(a.F.X, b, h, 0, d, 0), xs = row_src(a.S.X, b, h, 0, d, 0);
  const RowSrc vf = row_src(a.V, b, h, 0, a.vcols, a.vone), uf = row_src(a.U, b, h, 0, a.ucols, a.uone);
  const float* th = a.S.theta + (size_t)group_of(a.S.groups, b, h, a.H) * a.S.theta_stride;
  const float* Cmat = (((int)th[2]) & 1) || a.part_out != nullptr ? nullptr : th + a.S.c_offset;
  auto row_of = [&](int ci) { return row_beg + TT * (MODE ? nchunk - 1 - ci : ci); };

  Fetch<XC, NW, XP> pf, ps;
  Fetch<VC, NW, VP> pv;
  Fetch<VC, NW, UP> pu;
  auto fetch_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                       // (nothing of the addresses is kept across chunks: registers)
    const int r0 = row_of(ci);
    pf.get(xf, r0, row_end, tid);
    ps.get(xs, r0, row_end, tid);
    pv.get(vf, r0, row_end, tid);
    pu.get(uf, r0, row_end, tid);
  };
  auto put_chunk = [&](int ci) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int r0 = row_of(ci);
    pf.put(xf, Xf, r0, row_end, tid);
    ps.put(xs, Xs, r0, row_end, tid);
    pv.put(vf, Vs, r0, row_end, tid, MODE ? ge : ve);
    pu.put(uf, Us, r0, row_end, tid, MODE ? ve : ge);
  };
  // four numbers of a second-side row as they are
  auto x_four = [&](int row, int col) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = XP - 1; i >= 0; --i) {
      const u32x2 q = *(const u32x2*)(Xs + i * XPLANE + row * LDX + col);
      x += f32x4{__uint_as_float(q[0] << 16), __uint_as_float(q[0] & 0xffff0000u), __uint_as_float(q[1] << 16), __uint_as_float(q[1] & 0xffff0000u)};
    }
    return x;
  };
  fetch_chunk(0);
  for (int f = threadIdx.x; f < 16 * FT * NW; f += 64 * NW) bl[f] = 16 * a.tile0 + f < M ? bias[16 * a.tile0 + f] : -INFINITY;
  f32x4 Z[FT][VT];                                  // Z[ft][vt][r]: feature f0 + 16 ft + c, column 16 vt + 4 g + r
  const float* st = a.state + ((size_t)bh * a.nseg + seg) * M * a.ldt;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const int f = f0 + 16 * ft + c, fc = min(f, M - 1);
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
      const int col = 16 * vt + 4 * g;
      const f32x4 v = *(const f32x4*)(st + (size_t)fc * a.ldt + min(col, a.ldt - 4));
      Z[ft][vt] = f < M && col < a.ldt ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  put_chunk(0);
  for (int ci = 0; ci < nchunk; ++ci) {
    asm volatile("" : "+v"(g), "+v"(c));             // (nothing that follows from the lane is kept across chunks)
    const int row0 = row_of(ci);
    __syncthreads();
    // u_i . v_j (rows = first-side tokens, column = second-side token), masked, and Z u
    f32x4 am[2][2], df[FT][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      am[0][t] = am[1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) df[ft][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int pr = 0; pr < NV; ++pr) {
      __builtin_amdgcn_sched_barrier(0);
      Op<UP> u[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) u[t] = pair_op<UP>(Us + (16 * t + c) * LDV + 32 * pr + 4 * g, VPLANE);
#pragma unroll
      for (int tf = 0; tf < 2; ++tf) {
        const Op<VP> v = pair_op<VP>(Vs + (16 * tf + c) * LDV + 32 * pr + 4 * g, VPLANE);
#pragma unroll
        for (int t = 0; t < 2; ++t)
          if (MODE ? tf >= t : tf <= t) am[tf][t] = times(v, u[t], am[tf][t]);
      }
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) {
        __builtin_amdgcn_sched_barrier(0);
        const f32x4 none = {0.f, 0.f, 0.f, 0.f};
        const Split3 z = split3(Z[ft][2 * pr], 2 * pr + 1 < VT ? Z[ft][2 * pr + 1 < VT ? 2 * pr + 1 : 0] : none);
#pragma unroll
        for (int t = 0; t < 2; ++t) df[ft][t] = times(z, u[t], df[ft][t]);
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int tf = 0; tf < 2; ++tf)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int first = 16 * tf + 4 * g + r, second = 16 * t + c;
          am[tf][t][r] = (MODE ? first >= second : first <= second) ? am[tf][t][r] : 0.f;
        }
    __builtin_amdgcn_sched_barrier(0);
    // first side's features, rows = tokens, column = feature: into dF and into the state
    float addf[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) addf[t][r] = side_term<F_KEYS>(a, a.F, bh, row0 + 16 * t + 4 * g + r, row_end);
    const uint16_t* vcol = Vs + (4 * g + (c >> 2)) * LDV + 4 * (c & 3);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      f32x4 ff[1][2];
      project<false, Q, 1, XP>(ff, W1 + (size_t)ft * KS<Q> * 3 * IMG, Xf, lane);
      const float bf = bl[fw + 16 * ft + c];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) ff[0][t][r] = kLift * fast_exp2(exponent<F_KEYS>(ff[0][t][r], bf, addf[t][r], kmax));
      const Split3 fo = split3(ff[0][0], ff[0][1]);
      df[ft][0] = mfma3<MODE ? ALL : LOW>(fo, split3(am[0][0], am[1][0]), df[ft][0]);
      df[ft][1] = mfma3<MODE ? HIGH : ALL>(fo, split3(am[0][1], am[1][1]), df[ft][1]);
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        if (vt % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        Z[ft][vt] = times(column_op<VP>(vcol + 16 * vt, LDV, VPLANE), fo, Z[ft][vt]);
      }
    }
    // second side's features, rows = features, column = token; dE = F * dF
    __builtin_amdgcn_sched_barrier(0);
    float adds[2], rs[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t) adds[t] = side_term<!F_KEYS>(a, a.S, bh, row0 + 16 * t + c, row_end);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      f32x4 fs2[1][2];
      project<true, Q, 1, XP>(fs2, W2 + (size_t)ft * KS<Q> * 3 * IMG, Xs, lane);
      const f32x4 br = *(const f32x4*)(bl + fw + 16 * ft + 4 * g);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          df[ft][t][r] *= fast_exp2(exponent<!F_KEYS>(fs2[0][t][r], br[r], adds[t], kmax));
          rs[t] += df[ft][t][r];
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      rs[t] += __shfl_xor(rs[t], 16);
      rs[t] += __shfl_xor(rs[t], 32);
      if (g == 0) rsw[w * TT + 16 * t + c] = rs[t];
    }
    __builtin_amdgcn_sched_barrier(0);
    // the row term's part, a tile of sixteen columns and tokens per wave
    if (Cmat != nullptr) {
      for (int ct = w; ct < 2 * Q; ct += NW) {
        const int t = ct & 1, col = 16 * (ct >> 1) + c;
        const uint32_t cl = (uint32_t)min(col, d - 1);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          if (q % 2 == 0) __builtin_amdgcn_sched_barrier(0);
          const uint32_t e = (uint32_t)min(16 * q + 4 * g, d - 4);
          f32x4 cm = *(const f32x4*)((const char*)Cmat + 4u * (cl * (uint32_t)d + e));
#pragma unroll
          for (int s = 0; s < 4; ++s) cm[s] += *(const float*)((const char*)Cmat + 4u * ((e + s) * (uint32_t)d + cl));
          const f32x4 x = x_four(16 * t + c, 16 * q + 4 * g) * scale;      // (zero past the row)
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = mfma4(x[s], cm[s], acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) cx[(16 * t + 4 * g + r) * ldc + col] = acc[r];
      }
    }
    // gradient rows of this wave's features: dE W~, a block of coordinates after the other
#pragma unroll
    for (int d0 = 0; d0 < 16 * Q; d0 += GC<Q>) {
      f32x4 gr[2][DT];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) gr[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      constexpr int STEPS = FT / 2 * DT;
      Split3 wt[3];
      const uint32_t at = image_lane(lane);
      const uint16_t* wc = Wt + (size_t)(d0 / 16) * 3 * IMG;
      asm volatile("" : "+s"(wc));
      auto image = [&](int s) { return image_op(wc + ((size_t)(s / DT) * 2 * KS<Q> + s % DT) * 3 * IMG, at); };
      wt[0] = image(0);
      wt[1] = image(1);
#pragma unroll
      for (int pr = 0; pr < FT / 2; ++pr) {
        Split3 de[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) de[t] = split3(df[2 * pr][t], df[2 * pr + 1][t]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const int s = pr * DT + dt;
          __builtin_amdgcn_sched_barrier(0);
          if (s + 2 < STEPS) wt[(s + 2) % 3] = image(s + 2);
#pragma unroll
          for (int t = 0; t < 2; ++t) gr[t][dt] = mfma3(de[t], wt[s % 3], gr[t][dt]);
        }
      }
      if (d0 > 0) __syncthreads();       // the last block's rows have been summed
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 4; ++r) xch[(w * TT + 16 * t + 4 * g + r) * ldo + 16 * dt + c] = gr[t][dt][r];
      if (d0 + GC<Q> >= 16 * Q && ci + 1 < nchunk) fetch_chunk(ci + 1);      // the next chunk's rows travel meanwhile
      __syncthreads();
      {
        const int row = threadIdx.x / (2 * NW), l = threadIdx.x % (2 * NW);
        float rsum = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) rsum += rsw[i * TT + row];
        if (row0 + row < row_end) {
          const size_t rec = (size_t)(bh - a.bh0) * a.L + row0 + row;
          if (a.part_in != nullptr) rsum += a.part_in[rec * a.ldp + d];
          if (a.part_out != nullptr && d0 == 0 && l == 0) a.part_out[rec * a.ldp + d] = rsum;
          const long long ob = b * a.out.sb + h * a.out.sh + (long long)(row0 + row) * a.out.sl;
          for (int col = l; col < min(GC<Q>, d - d0); col += 2 * NW) {
            float v = 0.f;
#pragma unroll
            for (int i = 0; i < NW; ++i) v += xch[(i * TT + row) * ldo + col];
            if (a.part_in != nullptr) v += a.part_in[rec * a.ldp + d0 + col];
            if (a.part_out != nullptr) {
              a.part_out[rec * a.ldp + d0 + col] = v;
              continue;
            }
            float rc;
            if (Cmat != nullptr) {
              rc = cx[row * ldc + d0 + col];
            } else {
              rc = 0.f;
#pragma unroll
              for (int i = XP - 1; i >= 0; --i) rc -= bf16_bits_to_f32(Xs[i * XPLANE + row * LDX + d0 + col]);
              rc *= scale;
            }
            store_elem(a.out, ob + d0 + col, ldexpf(v * kLn2 + scale * (rsum * rc), back));
          }
        }
      }
    }
    if (ci + 1 < nchunk) {
      __syncthreads();                   // (the rows have been read)
      put_chunk(ci + 1);
    }
  }
}

// Waves of 32 features, and launches of at most eight of them.
template <bool BF16, class F>
int by_features(int M, F launch) {
  if constexpr (BF16)
    if (M <= 128) return launch(std::integral_constant<int, 4>());
  return launch(std::integral_constant<int, 8>());
}
int tiles_of(int M) { return M <= 128 ? 8 : M <= 256 ? 16 : 32; }
int launches_of(int M) { return M <= 256 ? 1 : 2; }
// Widths and pieces of a row: two widths of fp32 rows, three of bf16 rows.
int width_of(int d, int ldt) { return d <= 32 && ldt <= 48 ? 2 : d <= 64 && ldt <= 80 ? 4 : 8; }
template <class F>
int by_rows(int d, int ldt, int dtype, F launch) {
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 3> three;
  const int q = width_of(d, ldt);
  if (q == 2) return dtype ? launch(std::integral_constant<int, 2>(), one) : launch(std::integral_constant<int, 2>(), three);
  if (q == 4) return dtype ? launch(std::integral_constant<int, 4>(), one) : launch(std::integral_constant<int, 4>(), three);
  return launch(std::integral_constant<int, 8>(), one);
}
template <class K>
int run(K kernel, const SplitArgs& a, dim3 grid, int threads, size_t lds, hipStream_t st) {
  if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, a);
  return hipGetLastError() == hipSuccess ? 0 : 5;
}
template <bool KEYS>
int run_state(const SplitArgs& a, int BH, hipStream_t st) {
  return by_rows(a.d, a.ldt, a.F.X.dtype, [&](auto q, auto xp) {
    return by_features<xp() == 1>(a.M, [&](auto nw) {
      constexpr int VP = KEYS ? xp() : 3;
      return run(k_split_state<q(), nw(), xp(), VP, KEYS>, a, dim3(a.nseg, BH, launches_of(a.M)), 64 * nw(), state_lds<q(), nw(), xp(), VP>(), st);
    });
  });
}
// launch(args) once, or twice for as many sequences at a time as `part` has room for the rows of the first launch
template <class F>
int in_launches(SplitArgs a, int BH, F launch) {
  const int n = launches_of(a.M), batch = n > 1 ? gen_split_part_sequences(BH, a.L, a.d, a.nv) : BH;
  float* part = a.part_out;
  for (a.bh0 = 0; a.bh0 < BH; a.bh0 += batch) {
    a.nbh = BH - a.bh0 < batch ? BH - a.bh0 : batch;
    for (int i = 0; i < n; ++i) {
      a.tile0 = 16 * i;
      a.part_out = i + 1 < n ? part : nullptr;
      a.part_in = i > 0 ? part : nullptr;
      if (int rc = launch(a)) return rc;
    }
  }
  return 0;
}
template <int MODE>
int run_walk(const SplitArgs& args, int BH, hipStream_t st) {
  return in_launches(args, BH, [&](const SplitArgs& a) {
    return by_rows(a.d, a.ldt, a.F.X.dtype, [&](auto q, auto xp) {
      return by_features<xp() == 1>(a.M, [&](auto nw) {
        constexpr int VP = MODE ? 3 : xp();
        return run(k_split_walk<q(), nw(), xp(), VP, MODE>, a, dim3(a.nseg, a.nbh), 64 * nw(), walk_lds<q(), nw(), xp(), VP>(), st);
      });
    });
  });
}
template <int MODE>
int run_gwalk(const SplitArgs& args, int BH, hipStream_t st) {
  return in_launches(args, BH, [&](const SplitArgs& a) {
    return by_rows(a.d, a.ldt, a.F.X.dtype, [&](auto q, auto xp) {
      return by_features<xp() == 1>(a.M, [&](auto nw) {
        constexpr int VP = MODE ? 3 : xp(), UP = MODE ? xp() : 3;
        return run(k_split_gwalk<q(), nw(), xp(), MODE>, a, dim3(a.nseg, a.nbh), 64 * nw(), gwalk_lds<q(), nw(), xp(), VP, UP>(), st);
      });
    });
  });
}
SplitArgs split_args(const GenSide& f, const GenSide& s, const GenSplit& sp, int L, int BH, int H, int M, int d, int nv, int ldt, int rows_per_seg,
                     int nseg, uint32_t* kmax_u, const float* row_shift, float* state) {
  SplitArgs a{};
  a.F = f; a.S = s;
  a.L = L; a.BH = BH; a.H = H; a.M = M; a.d = d; a.nv = nv; a.ldt = ldt; a.rows_per_seg = rows_per_seg; a.nseg = nseg; a.ntile = tiles_of(M);
  a.vmax = sp.vmax; a.dmax = sp.dmax; a.nvmax = (L + VMAX_ROWS - 1) / VMAX_ROWS; a.exps = sp.exps;
  a.img = sp.img; a.img_t = sp.img_t; a.part_out = sp.part; a.ldp = gen_split_part_row(d, nv);
  a.kmax_u = kmax_u; a.row_shift = row_shift; a.state = state;
  return a;
}
}  // namespace

// Which calls they take.  Speed of a causal call against one on the kernels of kernels_gen_walk.hip (380 drawn calls, 256 - 32768
// head-tokens), where a chunk is 16 tokens and a wave 16 features: with few features or narrow rows the chain of a chunk is what
// a call waits for, and there it is shorter.
//   attention  f32   M <= 64 0.71 - 0.84;  M 100, 128 0.85 - 1.01;  M 200, 256: d 8, 16 0.86 - 0.90, d 24 .. 64 1.03 - 1.28
//              bf16  M <= 64 0.81 - 1.06;  M >= 100: d 8, 16 0.96 - 1.13, d 24 .. 128 1.04 - 1.48
//   gradients  f32   M <= 64 0.72 - 0.82;  M 100, 128 0.86 - 1.08;  M 200, 256: d 8, 16 0.91 - 0.97, d 24 .. 64 1.10 - 1.40
//              bf16  M <= 64 0.69 - 0.99;  M >= 100: d 8, 16 1.04 - 1.07, d 24 .. 128 1.15 - 1.50 (d 80 M 100, 128 0.96 - 1.04)
// and, as features pad to 128, 256 or 512, over numbers between those (2 x 700, 16 x 1024 and 32 x 2048 head-tokens, d 24 .. 128)
//   attention  f32   M 129 .. 256 1.18 - 1.67, 257 .. 512 1.19 - 1.70;  bf16  65 .. 128 1.33 - 1.89, 129 .. 256 1.39 - 2.07, 257 .. 512 1.33 - 1.96
//   gradients  f32   M 129 .. 256 1.17 - 2.04, 257 .. 512 1.14 - 1.93;  bf16  65 .. 128 1.42 - 2.04, 129 .. 256 1.34 - 2.45, 257 .. 512 1.22 - 2.56
static bool split_rows(int d, int dv, int dtype) {
  const int ldt = (dv + 16) / 16 * 16;
  return d % 4 == 0 && dv % 4 == 0 && d > 16 && width_of(d, 0) == width_of(0, ldt) && (dtype || width_of(d, ldt) < 8);
}
bool gen_split_attention(int d, int dv, int M, int dtype) { return split_rows(d, dv, dtype) && M > (dtype ? 64 : 128) && M <= 512; }
bool gen_split_backward(int d, int dv, int M, int dtype) {
  return split_rows(d, dv, dtype) && M > (!dtype || (d > 64 && d <= 96) ? 128 : 64) && M <= 512;
}
// Sequences of a chunk or two: half of a chunk of 32 tokens is padding where a chunk of 16 has none, and the start of a workgroup counts.
// Speed against the same kernels, 1 - 1024 sequences, M 129 - 512 (bf16 from 70; the lower figures of bf16 are those of M 70):
//   tokens       8, 16        17 .. 32      48           64           80           96
//   f32   d 24   0.70 - 0.85  0.92 - 1.06   0.83 - 0.92  0.96 - 1.08  0.95 - 1.06  1.06 - 1.18
//         d 64   0.73 - 0.90  1.02 - 1.12   0.89 - 1.00  1.06 - 1.18  0.98 - 1.15  1.10 - 1.33
//   bf16  d 24   0.76 - 0.90  0.96 - 1.10   0.93 - 1.01  1.05 - 1.20  1.02 - 1.20  1.15 - 1.33
//         d 128  0.74 - 0.95  0.96 - 1.30   0.95 - 1.19  1.10 - 1.45  1.22 - 1.48  1.08 - 1.67
// (80 tokens of f32 d 24: below one only from 256 sequences on; bf16 d 128 M 129 .. at 48 tokens 1.01 and more)
bool gen_split_length(int BH, int L, int d, int M, int dtype) {
  if (L > 80) return true;
  if (dtype) return L > 48 || (M > 128 && L > 16 && (L <= 32 || d > 32));
  return d > 32 ? L > 48 || (L > 16 && L <= 32) : L > 48 && BH < 256;
}
int gen_split_part_row(int d, int dv) { return (d > dv ? d : dv) + 20; }
// Sequences whose partial rows are there at a time: 256 MB of them, one at least.
int gen_split_part_sequences(int BH, int L, int d, int dv) {
  const size_t one = sizeof(float) * (size_t)L * gen_split_part_row(d, dv), n = ((size_t)256 << 20) / one;
  return n < 1 ? 1 : n < (size_t)BH ? (int)n : BH;
}
GenSplitShape gen_split_shape(int d, int dv, int M) {
  const int q = width_of(d, (dv + 16) / 16 * 16);
  return {tiles_of(M), q == 2 ? 1 : q == 4 ? 2 : 4, launches_of(M) > 1, M <= 128 ? 4 : 8};
}

int launch_split_state(const GenSide& side, const GenSplit& sp, bool keys, const TensorDev& V, int L, int BH, int H, int M, int d, int nv,
                       int ldt, int rows_per_seg, int nseg, uint32_t* kmax_u, const float* part, int npart, const float* row_shift,
                       float* state, hipStream_t st) {
  SplitArgs a = split_args(side, side, sp, L, BH, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, row_shift, state);
  a.V = V; a.vcols = keys ? nv : ldt; a.vone = keys; a.part = part; a.npart = npart;
  return keys ? run_state<true>(a, BH, st) : run_state<false>(a, BH, st);
}

int launch_split_walk(const GenSide& qs, const GenSide& ks, const GenSplit& sp, const TensorDev& V, int L, int BH, int H, int M, int d,
                      int nv, int ldt, int rows_per_seg, int nseg, uint32_t* kmax_u, float* Tstate, const TensorDev& Y, float* den_out,
                      float* shift_out, hipStream_t st, unsigned* flushed) {
  SplitArgs a = split_args(ks, qs, sp, L, BH, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, nullptr, Tstate);
  a.V = V; a.vcols = nv; a.vone = 1; a.out = Y; a.den_out = den_out; a.shift_out = shift_out; a.flushed = flushed;
  return run_walk<0>(a, BH, st);
}

int launch_split_bwd_walks(const GenSide& qs, const GenSide& ks, const GenSplit& sp, const TensorDev& V, const float* ghat, int L, int BH,
                           int H, int M, int d, int nv, int ldt, int rows_per_seg, int nseg, uint32_t* kmax_u, const float* row_shift,
                           float* Tstate, float* Rstate, const TensorDev& dQ, const TensorDev& dK, const TensorDev& dV, hipStream_t st) {
  const TensorDev G{ghat, 0, (long long)H * L * ldt, (long long)L * ldt, (long long)ldt};
  SplitArgs a = split_args(ks, qs, sp, L, BH, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, row_shift, Tstate);
  a.V = V; a.vcols = nv; a.vone = 1; a.U = G; a.ucols = ldt; a.out = dQ;
  if (int rc = run_gwalk<0>(a, BH, st)) return rc;
  SplitArgs r = split_args(qs, ks, sp, L, BH, H, M, d, nv, ldt, rows_per_seg, nseg, kmax_u, row_shift, Rstate);
  r.V = G; r.vcols = ldt; r.U = V; r.ucols = nv; r.uone = 1; r.out = dV;
  if (int rc = run_walk<1>(r, BH, st)) return rc;
  r.out = dK;
  return run_gwalk<1>(r, BH, st);
}

}  // namespace fs
