// Kernel operator K^(alpha)(X, Y) C for a few right-hand sides (Section 2.1, the problem statement): out = P (S^T C)
// with fp32 rows, fp32 arithmetic (split3.h: numbers as three bf16 pieces on the bf16 matrix instructions) and every scale kept
// (Section 2.3: the exp(alpha |.|^2) factors, D, M^-1/2).  Shapes: d a multiple of 4 up to 64, M a multiple of 16, n <= 16 columns.
//
// Four launches: k_op_pre (projection constants as operand images of pieces), k_op_state (one workgroup per 64 key rows:
// S^T C of those rows, every tile of 16 features on its own largest exponent), k_op_reduce (sum over the workgroups per tile, on
// the tile's largest shift, as operand images), k_op_apply (one workgroup per 64 query rows: P T, every wave on its rows' largest
// exponents, brought together and scaled back at the end).
//
// A workgroup is eight waves; a wave owns every eighth 16-feature tile (query side: pair of tiles).  The pieces of the workgroup's 64
// rows are operands in registers for the whole kernel, the projection slice of a tile is read from its image one tile ahead.
// MFMA operand layout (v_mfma_f32_16x16x32_bf16): A[l%16][8(l/16)..+7], B[8(l/16)..+7][l%16], D[4(l/16)+r][l%16]; two stacked D tiles
// are an operand whose contraction index runs 16(e/4) + 4(l/16) + e%4.
//   key side    E = X W^T   (A = rows, B = W~)   -> lane <-> feature, registers <-> rows 4g .. 4g+3: two row tiles are an operand of
//               T_tile += S^T C (B = C in the same order of rows)
//   query side  E^T = W X^T (A = W~, B = rows)   -> lane <-> row, registers <-> features: two feature tiles are an operand of
//               out^T += T^T P^T (A = T in the same order of features)
// Exponents live in the log2 domain.  Shifts, where there have to be any, are largest exponents of what a wave has in its registers
// anyway, so no factor can overflow and none that matters can vanish, and they are applied back at the end through the exponent field: a sum of shifts
// may leave the fp32 exponent range although the result does not.
// Pieces of numbers below 2^-109 lose bits (split3.h), so no operand is left there: right-hand sides are split relative to the largest of
// their column among the workgroup's rows, the state relative to the largest of the column (powers of two, taken back through the
// exponent field), and features are lifted by kLift.  (All of C near 2^-110 / 2^-115 / 2^-120: results up to 8e-4 / 3e-2 / 0.8 off
// without that, with fp32 instructions 4e-6 .. 2e-4, now as for C near one, up to 4e-6.)
//
// What bounds it: matrix pipe, exponentials and splits are 3 - 4 us of each of the two main kernels (256 workgroups of c2), the rest is
// the launch and the chain rows -> operands -> first tile.  With fp32 instructions and Cauchy-Schwarz bounds over all features as
// shifts (N 16384, d 32, M 512, n 8): k_op_state 25.3 us, now 15.0, k_op_apply
// 20.7 and 9.8, the call 52.3 and 29.2; 40 calls of N 256 .. 32768, d 8 .. 64: results 0.56 times as far from 64 bits.
#include <algorithm>

#include "fast_common.h"
#include "split3.h"

namespace fs {
namespace op {

constexpr int RW = 64;          // rows per workgroup
constexpr int NTH = 512;        // threads per workgroup: eight waves, two per SIMD
constexpr int NWV = NTH / 64;
constexpr int NC = 16;          // right-hand-side columns (padded)
constexpr int DMAX = 64;
constexpr int IMG = 512;        // numbers of an operand image: 64 lanes x 8
constexpr int LIFT = 12;        // binary exponent of the factor on the features of either side
constexpr float kLift = 1 << LIFT;
constexpr int FAR = 64;         // parts of the state from larger right-hand sides are stored at 2^-LIFT, not 2^LIFT (sums near the largest number)
constexpr int NONE = -1000;     // exponent of a column of zeros
// (the kernels are instantiated for KS = 1 and 2 contraction steps of a projection: d <= 32 and d <= 64; numbers past d are zero)

struct OpArgs {
  TensorDev X;            // rows of this side ([N, d] f32)
  const float* theta;     // one parameter set
  const uint16_t* W;      // this side's [M/16][KS][3][IMG]: pieces of W~, log2e folded in
  const float* bias;      // [M]
  const float* C;         // [Ny][n]
  float* Tpart;           // [nwg][M][NC]
  float* tshift;          // [M/16][nwg]
  int* cexp;              // [nwg][NC]: binary exponents of the columns of C, in the workgroup's rows
  const int* cstar;       // [NC]: the largest of them
  const uint16_t* T;      // [pairs of tiles][3][IMG]: pieces of the state
  const float* tstar;     // [M/16]
  float* out;             // [Nx][n]
  int N, d, M, n, nwg;
  float scale, alpha;
};

// Where the contraction has room behind the d numbers of a row, two more are the bias against one and one against the row term: the
// exponent then is a single sum of exact products, rounded once.  (Added afterwards, d = 8 and 16 have results up to 1.4
// times as far from 64 bits as sums of fp32 products that start from bias and row term.)
__host__ __device__ __forceinline__ bool terms_in_product(int d) { return d % 32 != 0; }

// ---------------------------------------------------------------------------------------------------
// Projection constants (Section 4, evaluation recipe): W~[side][m,:] = log2e omega_m^T B_side, bias[m] = log2e
// (omega_m^T A omega_m + log D - 1/2 log M), the same for both sides.  grid (M/4, 2), block 256: a wave per feature, lane c
// handles column c.
// ---------------------------------------------------------------------------------------------------
template <int KS>
__global__ void __launch_bounds__(256) k_op_pre(const float* theta, const float* Omega, int M, int d, uint16_t* W, float* bias) {
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), side = blockIdx.y, c = threadIdx.x & 63;
  const float* om = Omega + (size_t)m * d;
  const float* Bm = theta + FS_THETA_HEADER_ + d + (side ? (size_t)d * d : 0);
  const float* A = theta + FS_THETA_HEADER_;
  float acc = 0.f, q = 0.f;
  if (c < d) {
    // sixteen rows of B requested at a time (d is a multiple of 4): the loop is a chain of memory latencies otherwise
    for (int l0 = 0; l0 < d; l0 += 16) {
      float o[16], bv[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int l = min(l0 + i, d - 1);
        o[i] = l0 + i < d ? om[l] : 0.f;
        bv[i] = Bm[l * d + c];
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) acc += o[i] * bv[i];
    }
    acc *= kLog2e;
    q = A[c] * om[c] * om[c];
  }
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) q += __shfl_xor(q, s);
  const float bm = kLog2e * (q + theta[0] - 0.5f * logf((float)M));
  if (terms_in_product(d)) acc = c == d ? bm : (c == d + 1 ? 1.f : acc);
  if (c < 32 * KS) {
    const size_t image = (((size_t)side * (M >> 4) + (m >> 4)) * KS + (c >> 5)) * 3;
    split3_store(W + image * IMG + ((c & 31) / 8 * 16 + (m & 15)) * 8 + (c & 7), IMG, acc);
  }
  if (side == 0 && c == 0) bias[m] = bm;
}

template <int KS> struct RowsLds {
  u32x4 x[KS][4][3][64];          // pieces of the rows, scaled by qk_scale (zero past the end): operand images of 16 rows
  float rt[RW];                   // row term log2e (x^T C x + alpha |x|^2), zero where it is in the product
  float xf[RW][DMAX + 1];         // the rows themselves, where the row terms need them
};

// Rows to LDS and from there to registers, row terms.
template <int KS>
__device__ __forceinline__ void stage_rows(RowsLds<KS>& sm, const OpArgs& a, int side, int row0, Split3 (&x)[KS][4]) {
  const float* Xp = (const float*)a.X.ptr;
  const bool iso = ((int)a.theta[2]) & 1;
  const int t = threadIdx.x;
  if (t < RW * 4 * KS) {                                   // eight numbers of a row each
    const int r = t / (4 * KS), ch = t % (4 * KS), col = 8 * ch;
    f32x4 v[2];
    const float* p = Xp + (long long)min(row0 + r, a.N - 1) * a.X.sl;
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = *(const f32x4*)(p + min(col + 4 * i, a.d - 4));      // (rows start at multiples of 16 bytes)
    float n2 = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      v[i] = row0 + r < a.N && col + 4 * i < a.d ? v[i] * a.scale : f32x4{0.f, 0.f, 0.f, 0.f};
      n2 += (v[i][0] * v[i][0] + v[i][1] * v[i][1]) + (v[i][2] * v[i][2] + v[i][3] * v[i][3]);
    }
    n2 += __shfl_xor(n2, 1);
    n2 += __shfl_xor(n2, 2);
    if (KS == 2) n2 += __shfl_xor(n2, 4);
    const float rt = kLog2e * ((a.alpha - 0.5f) * n2);
    if (!iso) {
#pragma unroll
      for (int i = 0; i < 8; ++i) sm.xf[r][col + i] = v[i >> 2][i & 3];
    } else if (ch == 0) {
      sm.rt[r] = terms_in_product(a.d) ? 0.f : rt;
    }
    if (terms_in_product(a.d)) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (col + 4 * i == a.d) v[i] = f32x4{1.f, iso ? rt : 0.f, 0.f, 0.f};
    }
    const Split3 s = split3(v[0], v[1]);
    const int at = (ch & 3) * 16 + (r & 15);
    sm.x[ch >> 2][r >> 4][0][at] = __builtin_bit_cast(u32x4, s.h);
    sm.x[ch >> 2][r >> 4][1][at] = __builtin_bit_cast(u32x4, s.m);
    sm.x[ch >> 2][r >> 4][2][at] = __builtin_bit_cast(u32x4, s.l);
  }
  __syncthreads();
  if (!iso) {                                              // eight threads per row
    const int r = t >> 3, part = t & 7;
    const float* Cm = a.theta + FS_THETA_HEADER_ + a.d + (2 + (side ? 1 : 0)) * (size_t)a.d * a.d;
    float n2 = 0.f, qf = 0.f;
    for (int i = part; i < a.d; i += 8) {
      const float xi = sm.xf[r][i];
      n2 += xi * xi;
      float s = 0.f;
      for (int j = 0; j < a.d; ++j) s += Cm[i * a.d + j] * sm.xf[r][j];
      qf += xi * s;
    }
    n2 += __shfl_xor(n2, 1); n2 += __shfl_xor(n2, 2); n2 += __shfl_xor(n2, 4);
    qf += __shfl_xor(qf, 1); qf += __shfl_xor(qf, 2); qf += __shfl_xor(qf, 4);
    if (part == 0) {
      const float rt = kLog2e * (qf + a.alpha * n2);
      sm.rt[r] = terms_in_product(a.d) ? 0.f : rt;
      if (terms_in_product(a.d)) {
        const int col = a.d + 1;
        split3_store((uint16_t*)&sm.x[col >> 5][r >> 4][0][(col & 31) / 8 * 16 + (r & 15)] + (col & 7), IMG, rt);
      }
    }
    __syncthreads();
  }
  const int lane = t & 63;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      x[ks][tt].h = __builtin_bit_cast(bf16x8, sm.x[ks][tt][0][lane]);
      x[ks][tt].m = __builtin_bit_cast(bf16x8, sm.x[ks][tt][1][lane]);
      x[ks][tt].l = __builtin_bit_cast(bf16x8, sm.x[ks][tt][2][lane]);
    }
}

// The shift of features whose largest exponent is m.  None where they and their products stay well inside the fp32 range anyway: a
// shift's own rounding is a relative error of all of them (d = 8: results 1.1 - 1.6 times as far from 64 bits with it).
__device__ __forceinline__ float shift_of(float m) { return fabsf(m) <= 30.f || m == -INFINITY ? 0.f : m; }

__device__ __forceinline__ Split3 load_image(const uint16_t* img, int lane) {
  const u32x4* p = (const u32x4*)img + lane;
  return {__builtin_bit_cast(bf16x8, p[0]), __builtin_bit_cast(bf16x8, p[IMG / 8]), __builtin_bit_cast(bf16x8, p[2 * (IMG / 8)])};
}
template <int KS>
__device__ __forceinline__ void load_slice(Split3 (&w)[KS], const uint16_t* W, int ft, int lane) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) w[ks] = load_image(W + ((size_t)ft * KS + ks) * 3 * IMG, lane);
}

// ---------------------------------------------------------------------------------------------------
// Key side: Tpart[wg] = sum over the workgroup's rows j of exp2(E2_jm - t) C_j, t = the largest exponent of the tile of
// features, to tshift.  grid ceil(Ny / 64), block 512.
// ---------------------------------------------------------------------------------------------------
template <int KS>
__global__ void __launch_bounds__(NTH, 2) k_op_state(OpArgs a) {
  __shared__ RowsLds<KS> sm;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, c = lane & 15;
  const int row0 = blockIdx.x * RW, ntile = a.M >> 4;
  Split3 wr[KS], wn[KS];
  load_slice(wr, a.W, min(w, ntile - 1), lane);
  // right-hand sides of rows 4g .. 4g + 3 of the row tiles, column c
  f32x4 cv[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 16 * tt + 4 * g + r;
      const float v = a.C[(size_t)min(row, a.N - 1) * a.n + min(c, a.n - 1)];
      cv[tt][r] = row < a.N && c < a.n ? v : 0.f;
    }
  Split3 x[KS][4], cs[2];
  stage_rows<KS>(sm, a, 1, row0, x);
  float big = 0.f;
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) big = fmaxf(big, fabsf(cv[tt][r]));
  big = fmaxf(big, __shfl_xor(big, 16));
  big = fmaxf(big, __shfl_xor(big, 32));
  const int ce = big > 0.f ? __builtin_amdgcn_frexp_expf(big) : NONE;
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r) cv[tt][r] = ldexpf(cv[tt][r], -ce);
  if (w == 0 && g == 0) a.cexp[blockIdx.x * NC + c] = ce;
  cs[0] = split3(cv[0], cv[1]);
  cs[1] = split3(cv[2], cv[3]);
  f32x4 add[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int r = 0; r < 4; ++r)   // rows past the end: -inf, their features are exactly zero
      add[tt][r] = row0 + 16 * tt + 4 * g + r < a.N ? sm.rt[16 * tt + 4 * g + r] : -INFINITY;
  for (int ft = w; ft < ntile; ft += NWV) {
    const float bm = terms_in_product(a.d) ? 0.f : a.bias[16 * ft + c];
    if (ft + NWV < ntile) load_slice(wn, a.W, ft + NWV, lane);
    f32x4 e[4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) e[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) e[tt] = mfma3(x[ks][tt], wr[ks], e[tt]);
    float shift = -INFINITY;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      e[tt] = (e[tt] + bm) + add[tt];
      shift = fmaxf(shift, fmaxf(fmaxf(e[tt][0], e[tt][1]), fmaxf(e[tt][2], e[tt][3])));
    }
    shift = shift_of(fast::wave_max(shift));
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int r = 0; r < 4; ++r) e[tt][r] = kLift * fast_exp2(e[tt][r] - shift);
    f32x4 t = mfma3(split3(e[0], e[1]), cs[0], f32x4{0.f, 0.f, 0.f, 0.f});
    t = mfma3(split3(e[2], e[3]), cs[1], t);
    float* out = a.Tpart + ((size_t)blockIdx.x * a.M + 16 * ft + 4 * g) * NC + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(size_t)r * NC] = ldexpf(t[r], ce - (ce > FAR ? 2 * LIFT : 0));
    if (lane == 0) a.tshift[(size_t)ft * a.nwg + blockIdx.x] = shift;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) wr[ks] = wn[ks];
  }
}

// T = 2^-c* sum_wg Tpart[wg] 2^(t_wg - t*), t* = max t_wg of the tile.  grid M / 4, block 1024: four features per workgroup, the
// workgroups' partial states dealt to the sixteen waves.  (A last tile without a partner gets one of zeros.)
__global__ void __launch_bounds__(1024) k_op_reduce(const float* Tpart, const float* tshift, const int* cexp, uint16_t* T, float* tstar, int* cstar,
                                                    int nwg, int M) {
  __shared__ float red[16][2], part[16][64];
  __shared__ int cred[16][NC];
  const int ft = blockIdx.x >> 2, q = threadIdx.x >> 6, l = threadIdx.x & 63;
  const float* sh = tshift + (size_t)ft * nwg;
  const float* p = Tpart + (size_t)blockIdx.x * 64 + l;
  const size_t total = (size_t)M * NC;
  int cs = NONE;
#pragma unroll
  for (int u = 0; u < 4; ++u) cs = max(cs, cexp[min((int)threadIdx.x + 1024 * u, nwg * NC - NC + (l & 15))]);
  for (int i = threadIdx.x + 4096; i < nwg * NC; i += 1024) cs = max(cs, cexp[i]);
  // the first sixteen parts of a wave are requested ahead of the shifts
  float v[16], s16[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int i = min(q + 16 * u, nwg - 1);
    v[u] = p[i * total];
    s16[u] = sh[i];
  }
  float ts = -INFINITY;
  for (int i = threadIdx.x; i < nwg; i += 1024) ts = fmaxf(ts, sh[i]);
  ts = fast::wave_max(ts);
  cs = max(cs, __shfl_xor(cs, 16));
  cs = max(cs, __shfl_xor(cs, 32));
  if (l < NC) cred[q][l] = cs;
  const float any = __any(cs > FAR) ? 1.f : 0.f;
  if (l == 0) {
    red[q][0] = ts;
    red[q][1] = any;
  }
  __syncthreads();
  ts = red[0][0];
  float far = red[0][1];
#pragma unroll
  for (int i = 1; i < 16; ++i) {
    ts = fmaxf(ts, red[i][0]);
    far = fmaxf(far, red[i][1]);
  }
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u) acc += q + 16 * u < nwg ? v[u] * fast_exp2(s16[u] - ts) : 0.f;
#pragma unroll 4
  for (int i = q + 256; i < nwg; i += 16) acc += p[i * total] * fast_exp2(sh[i] - ts);
  int down = 0;
  if (far > 0.f) {                                   // (there are parts at 2^-LIFT: those at 2^LIFT are brought down)
    cs = NONE;
    for (int i = 0; i < 16; ++i) cs = max(cs, cred[i][l & 15]);
    if (cs > FAR) {
      down = 2 * LIFT;
      acc = 0.f;
      for (int i = q; i < nwg; i += 16) acc += ldexpf(p[i * total], cexp[i * NC + (l & 15)] > FAR ? 0 : -down) * fast_exp2(sh[i] - ts);
    }
  }
  part[q][l] = acc;
  __syncthreads();
  if (q == 0) {
#pragma unroll
    for (int i = 1; i < 16; ++i) {
      acc += part[i][l];
      cs = max(cs, cred[i][l & 15]);
    }
    acc = ldexpf(acc, down - cs);
    if (blockIdx.x == 0 && l < NC) cstar[l] = cs;
    const int f = (blockIdx.x & 3) * 4 + (l >> 4), n = l & 15;        // feature of the tile, column
    uint16_t* at = T + (size_t)(ft >> 1) * 3 * IMG + ((f >> 2) * 16 + n) * 8 + (f & 3);
    split3_store(at + 4 * (ft & 1), IMG, acc);
    if ((ft & 1) == 0 && 16 * (ft + 1) >= M) split3_store(at + 4, IMG, 0.f);
  }
  if ((blockIdx.x & 3) == 0 && threadIdx.x == 0) tstar[ft] = ts;
}

// ---------------------------------------------------------------------------------------------------
// Query side: out_i = sum over waves 2^(s_iw) sum_m exp2(E1_im + t*_m - s_iw) T_m, s_iw = the row's largest exponent in the wave's
// tiles so far (its sums are rescaled where it grows).  grid ceil(Nx / 64), block 512.
// ---------------------------------------------------------------------------------------------------
template <int KS>
__global__ void __launch_bounds__(NTH, 2) k_op_apply(OpArgs a) {
  __shared__ union {
    RowsLds<KS> rows;
    struct {
      float xo[NWV][RW][NC + 1];      // partial out^T tiles of the waves: [wave][row][column]
      float sh[NWV][RW];              // their shifts
    } o;
  } sm;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, c = lane & 15;
  const int row0 = blockIdx.x * RW, ntile = a.M >> 4, npair = (ntile + 1) >> 1;
  auto second = [&](int p) { return min(2 * p + 1, ntile - 1); };      // (a last tile without a partner: itself, with T = 0)
  Split3 wr[2][KS];
  load_slice(wr[0], a.W, min(2 * w, ntile - 1), lane);
  load_slice(wr[1], a.W, second(w), lane);
  Split3 x[KS][4];
  stage_rows<KS>(sm.rows, a, 0, row0, x);
  float add[4], rm[4], s[4];      // row terms, largest exponents so far, shifts
  f32x4 o[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) {
    add[tt] = sm.rows.rt[16 * tt + c];
    rm[tt] = s[tt] = -INFINITY;
    o[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int p = w; p < npair; p += NWV) {
    const Split3 T = load_image(a.T + (size_t)p * 3 * IMG, lane);
    f32x4 e[2][4], bm[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ft = i ? second(p) : 2 * p;
      bm[i] = (terms_in_product(a.d) ? f32x4{0.f, 0.f, 0.f, 0.f} : *(const f32x4*)(a.bias + 16 * ft + 4 * g)) + a.tstar[ft];
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) e[i][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) e[i][tt] = mfma3(wr[i][ks], x[ks][tt], e[i][tt]);
      if (p + NWV < npair) load_slice(wr[i], a.W, i ? second(p + NWV) : 2 * (p + NWV), lane);
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      float m = -INFINITY;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        e[i][tt] = (e[i][tt] + bm[i]) + add[tt];
        m = fmaxf(m, fmaxf(fmaxf(e[i][tt][0], e[i][tt][1]), fmaxf(e[i][tt][2], e[i][tt][3])));
      }
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      rm[tt] = fmaxf(rm[tt], m);
      const float sn = shift_of(rm[tt]);
      o[tt] *= s[tt] == sn ? 1.f : fast_exp2(s[tt] - sn);
      s[tt] = sn;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) e[i][tt][r] = kLift * fast_exp2(e[i][tt][r] - sn);
      o[tt] = mfma3(T, split3(e[0][tt], e[1][tt]), o[tt]);
    }
  }
  // o[tt]: rows = columns 4g + r of the right-hand side, column = row 16 tt + c of the workgroup
  __syncthreads();                 // (in place of the rows)
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) sm.o.xo[w][16 * tt + c][4 * g + r] = o[tt][r];
    if (g == 0) sm.o.sh[w][16 * tt + c] = s[tt];
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < RW * a.n; idx += NTH) {
    const int r = idx / a.n, col = idx - r * a.n;
    if (row0 + r < a.N) {
      float m = sm.o.sh[0][r], v = 0.f;
#pragma unroll
      for (int wv = 1; wv < NWV; ++wv) m = fmaxf(m, sm.o.sh[wv][r]);
#pragma unroll
      for (int wv = 0; wv < NWV; ++wv) {
        const float sw = sm.o.sh[wv][r];
        v += sm.o.xo[wv][r][col] * (sw == m ? 1.f : fast_exp2(sw - m));
      }
      const float whole = floorf(m);
      a.out[(size_t)(row0 + r) * a.n + col] = ldexpf(v * fast_exp2(m - whole), (int)fminf(fmaxf(whole, -1000.f), 1000.f) + a.cstar[col] - 2 * LIFT);
    }
  }
}

}  // namespace op

bool op_supported(int dtype_x, int dtype_y, int d, int M, int n) {
  return dtype_x == 0 && dtype_y == 0 && d % 4 == 0 && d <= op::DMAX && M % 16 == 0 && n <= op::NC;
}

// Floats of workspace: pieces of W~ (both sides), partial states, pieces of the state, biases, shifts and exponents.
static int op_steps(int d) { return d <= 32 ? 1 : 2; }
size_t op_workspace_floats(int Ny, int d, int M) {
  const size_t nwg = (Ny + op::RW - 1) / op::RW, ntile = M >> 4;
  return 2 * ntile * op_steps(d) * 3 * op::IMG / 2 + nwg * M * op::NC + (ntile + 1) / 2 * 3 * op::IMG / 2 + M + nwg * ntile + ntile + (nwg + 1) * op::NC + 64;
}

#define FS_LAUNCH_CHECK() do { if (hipGetLastError() != hipSuccess) return 5; } while (0)

namespace op {
template <int KS>
static int launch(const float* theta, const TensorDev& X, const TensorDev& Y, int Nx, int Ny, int d, float scale, float alpha,
                  const float* Omega, int M, const float* C, int n, float* out, float* ws, hipStream_t st) {
  const int nwg = (Ny + RW - 1) / RW, ntile = M >> 4;
  const size_t side = (size_t)ntile * KS * 3 * IMG;
  uint16_t* W = (uint16_t*)(((uintptr_t)ws + 15) & ~(uintptr_t)15);
  uint16_t* T = W + 2 * side;
  float* Tpart = (float*)(T + (size_t)((ntile + 1) / 2) * 3 * IMG);
  float* bias = Tpart + (size_t)nwg * M * NC;
  float* tshift = bias + M;
  float* tstar = tshift + (size_t)nwg * ntile;
  int* cexp = (int*)(tstar + ntile);
  int* cstar = cexp + (size_t)nwg * NC;
  hipLaunchKernelGGL(k_op_pre<KS>, dim3(M / 4, 2), dim3(256), 0, st, theta, Omega, M, d, W, bias);
  FS_LAUNCH_CHECK();
  OpArgs a;
  a.theta = theta; a.bias = bias; a.C = C; a.Tpart = Tpart; a.tshift = tshift; a.cexp = cexp; a.T = T;
  a.tstar = tstar; a.cstar = cstar; a.out = out; a.d = d; a.M = M; a.n = n; a.nwg = nwg; a.scale = scale; a.alpha = alpha;
  a.X = Y; a.N = Ny; a.W = W + side;
  hipLaunchKernelGGL(k_op_state<KS>, dim3(nwg), dim3(NTH), 0, st, a);
  FS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_op_reduce, dim3(M / 4), dim3(1024), 0, st, Tpart, tshift, cexp, T, tstar, cstar, nwg, M);
  FS_LAUNCH_CHECK();
  a.X = X; a.N = Nx; a.W = W;
  hipLaunchKernelGGL(k_op_apply<KS>, dim3((Nx + RW - 1) / RW), dim3(NTH), 0, st, a);
  FS_LAUNCH_CHECK();
  return 0;
}
}  // namespace op

int launch_op_matvec(const float* theta, const TensorDev& X, const TensorDev& Y, int Nx, int Ny, int d, float scale,
                     float alpha, const float* Omega, int M, const float* C, int n, float* out, float* ws, hipStream_t st) {
  return op_steps(d) == 1 ? op::launch<1>(theta, X, Y, Nx, Ny, d, scale, alpha, Omega, M, C, n, out, ws, st)
                          : op::launch<2>(theta, X, Y, Nx, Ny, d, scale, alpha, Omega, M, C, n, out, ws, st);
}

}  // namespace fs
