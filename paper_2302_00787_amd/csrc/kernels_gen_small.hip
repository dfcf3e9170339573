// Non-causal attention of short sequences in one launch: constants, key maximum, state and outputs of a sequence by one workgroup.
// d up to 32 in fours, up to 256 keys, few features, queries and sequences as gen_small_supported says; fp32 arithmetic on v_mfma_f32_16x16x4_f32.
//
// Such a call is a chain of launches and memory latencies (f32 L 256 d 16 M 64: five launches of 3 - 9 us, 23 us, for 0.1 us of
// work at the card's rates).  Here rows, values and parameters are requested at once at the start, everything else stays in
// registers and LDS, and there are five barriers.  Layouts as in kernels_gen_rows.hip: lane l = (g, c) = (l / 16, l % 16), a row's numbers
// 16 q + 4 g .. + 3 are four contraction steps, an accumulator register is an operand.  Wave w takes every eighth tile of 16 keys, then
// of 16 queries.  f32 L 256 d 16 M 64: 24.9 -> 14.3 us.
#include <type_traits>

#include "gen_widths.h"
#include "kernels.h"

namespace fs {
namespace {

using namespace gen;

constexpr int SW = 8, SNT = 64 * SW;         // waves, threads
constexpr int KT = 2;                        // tiles of keys per wave: 16 SW KT keys

struct SmallArgs {
  TensorDev Q, K, V, Y;
  const float *theta, *Omega;
  int groups, omega_groups, H, Lq, Lk, d, M, nv;
  float scale;
  unsigned* flushed;
  int count;               // one workgroup: it writes the counter of zero normalisers itself
};

template <int BF>
__device__ __forceinline__ f32x4 load4(const TensorDev& t, long long at) {
  if constexpr (BF) {
    const u32x2 p = *(const u32x2*)((const uint16_t*)t.ptr + at);
    return f32x4{__uint_as_float(p[0] << 16), __uint_as_float(p[0] & 0xffff0000u), __uint_as_float(p[1] << 16), __uint_as_float(p[1] & 0xffff0000u)};
  } else {
    return *(const f32x4*)((const float*)t.ptr + at);
  }
}

template <int Q, int MT> constexpr int small_lds_floats() {
  constexpr int LDW = 16 * Q + 4, LDT = 16 * VT_OF<Q> + 1, F = 16 * MT, DQ = 16 * Q;
  constexpr int part = SW * F * LDT, stage = F * LDW + 2 * DQ * LDW;
  return 2 * F * LDW + 2 * F + F * LDT + 2 * SW + (part > stage ? part : stage);
}

// grid (B*H), block 512.
template <int Q, int MT, int BF>
__global__ void __launch_bounds__(SNT, 2) k_gen_small(SmallArgs a) {
  extern __shared__ __align__(16) float smem[];
  constexpr int VT = VT_OF<Q>, LDW = 16 * Q + 4, LDT = 16 * VT + 1, F = 16 * MT, DQ = 16 * Q, NO = F * DQ / SNT, NB = (2 * DQ * DQ + SNT - 1) / SNT;
  static_assert(DQ <= F, "A lies in F numbers");
  float* W = smem;                           // [2][F][LDW]: W~, zero past the features and past the row
  float* bl = W + 2 * F * LDW;               // biases, -inf past the features
  float* As = bl + F;                        // diagonal of A
  float* T = As + F;                         // [F][LDT] the state
  float* wmax = T + F * LDT;                 // [SW] largest exponents of the waves
  int* zeros = (int*)(wmax + SW);            // rows with a zero normaliser, by wave
  float* part = wmax + 2 * SW;               // [SW][F][LDT] the waves' parts of the state; before that omega and B1, B2
  float *om = part, *Bs = part + F * LDW;
  const int bh = blockIdx.x, b = bh / a.H, h = bh % a.H, d = a.d, M = a.M;
  const int t = threadIdx.x, lane = t & 63, g = lane >> 4, c = lane & 15, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* th = a.theta + (size_t)group_of(a.groups, b, h, a.H) * (FS_THETA_HEADER_ + (size_t)d + 4 * (size_t)d * d);
  const float* omg = a.Omega + (size_t)group_of(a.omega_groups, b, h, a.H) * M * d;
  const long long kb = b * a.K.sb + h * a.K.sh, vb = b * a.V.sb + h * a.V.sh, qb = b * a.Q.sb + h * a.Q.sh, yb = b * a.Y.sb + h * a.Y.sh;

  // ---- everything the kernel starts from is requested at once
  f32x4 x[KT][Q];
  float v[KT][4][VT];
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    const int row = 16 * (w + SW * i) + c;
#pragma unroll
    for (int q = 0; q < Q; ++q) x[i][q] = load4<BF>(a.K, kb + (long long)min(row, a.Lk - 1) * a.K.sl + min(16 * q + 4 * g, d - 4));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const long long at = vb + (long long)min(16 * (w + SW * i) + 4 * g + r, a.Lk - 1) * a.V.sl;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) v[i][r][vt] = load_elem(a.V, at + min(16 * vt + c, a.nv - 1));
    }
  }
  f32x4 xq[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) xq[q] = load4<BF>(a.Q, qb + (long long)min(16 * w + c, a.Lq - 1) * a.Q.sl + min(16 * q + 4 * g, d - 4));
  const float logD = th[0];
  const bool iso = ((int)th[2]) & 1;
  {
    float ro[NO], rb[NB], ra;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      const int e = t + SNT * i;
      ro[i] = omg[(size_t)min(e / DQ, M - 1) * d + min(e % DQ, d - 1)];
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int e = t + SNT * i, s = e / (DQ * DQ) & 1;
      rb[i] = th[FS_THETA_HEADER_ + d + (size_t)s * d * d + (size_t)min(e / DQ % DQ, d - 1) * d + min(e % DQ, d - 1)];
    }
    ra = th[FS_THETA_HEADER_ + min(t, d - 1)];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      const int e = t + SNT * i, m = e / DQ, l = e % DQ;
      om[m * LDW + l] = m < M && l < d ? ro[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int e = t + SNT * i, l = e / DQ % DQ, cc = e % DQ;
      if (e < 2 * DQ * DQ) Bs[(e / DQ) * LDW + cc] = l < d && cc < d ? rb[i] : 0.f;
    }
    if (t < DQ) As[t] = t < d ? ra : 0.f;
  }
  __syncthreads();
  // ---- W~ = log2e omega B, biases
  for (int e = t; e < 2 * F * DQ; e += SNT) {
    const int s = e / (F * DQ), m = e / DQ % F, cc = e % DQ;
    float acc = 0.f;
#pragma unroll
    for (int l = 0; l < DQ; ++l) acc += om[m * LDW + l] * Bs[(s * DQ + l) * LDW + cc];
    W[(s * F + m) * LDW + cc] = acc * kLog2e;
  }
  if (t < F) {
    float q = 0.f;
#pragma unroll
    for (int l = 0; l < DQ; ++l) q += As[l] * om[t * LDW + l] * om[t * LDW + l];
    bl[t] = t < M ? kLog2e * (q + logD - 0.5f * logf((float)M)) : -INFINITY;
  }
  // ---- keys: row terms x C x, by way of lanes into accumulator order
  const float* Cm = th + FS_THETA_HEADER_ + d + 3 * (size_t)d * d;
  float rt[KT][4];
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    float p = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      x[i][q] = 16 * q + 4 * g < d ? x[i][q] * a.scale : f32x4{0.f, 0.f, 0.f, 0.f};
      if (iso)
#pragma unroll
        for (int r = 0; r < 4; ++r) p += x[i][q][r] * x[i][q][r];
    }
    if (iso) {
      p *= -0.5f;
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) {          // (C x)[16 q + 4 g + r] of token c
        f32x4 cx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          const f32x4 cr = *(const f32x4*)(Cm + (size_t)min(16 * q + c, d - 1) * d + min(16 * k + 4 * g, d - 4));
#pragma unroll
          for (int s = 0; s < 4; ++s) cx = mfma4(cr[s], x[i][k][s], cx);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) p += x[i][q][r] * cx[r];
      }
    }
    p += __shfl_xor(p, 16);
    p += __shfl_xor(p, 32);
#pragma unroll
    for (int r = 0; r < 4; ++r) rt[i][r] = 16 * (w + SW * i) + 4 * g + r < a.Lk ? kLog2e * __shfl(p, 4 * g + r) : -INFINITY;
  }
  __syncthreads();
  // ---- exponents (rows = tokens, column = feature) and their maximum
  f32x4 e[KT][MT];
  float m = -INFINITY;
#pragma unroll
  for (int ft = 0; ft < MT; ++ft) {
    const float bf = bl[16 * ft + c];
#pragma unroll
    for (int i = 0; i < KT; ++i) e[i][ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const f32x4 wr = *(const f32x4*)(W + (F + 16 * ft + c) * LDW + 16 * q + 4 * g);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < KT; ++i) e[i][ft] = mfma4(x[i][q][s], wr[s], e[i][ft]);
    }
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        e[i][ft][r] = (e[i][ft][r] + bf) + rt[i][r];
        m = fmaxf(m, e[i][ft][r]);
      }
  }
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) m = fmaxf(m, __shfl_xor(m, s));
  if (lane == 0) wmax[w] = m;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SW; ++i) m = fmaxf(m, wmax[i]);
  // ---- state: the wave's part, then the sum over the waves
#pragma unroll
  for (int i = 0; i < KT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool live = 16 * (w + SW * i) + 4 * g + r < a.Lk;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt) {
        const int col = 16 * vt + c;
        v[i][r][vt] = live && col <= a.nv ? (col < a.nv ? v[i][r][vt] : 1.f) : 0.f;
      }
    }
#pragma unroll
  for (int ft = 0; ft < MT; ++ft) {
    f32x4 s[VT];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) s[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float f = fast_exp2(e[i][ft][r] - m);
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) s[vt] = mfma4(f, v[i][r][vt], s[vt]);
      }
#pragma unroll
    for (int vt = 0; vt < VT; ++vt)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[(w * F + 16 * ft + 4 * g + r) * LDT + 16 * vt + c] = s[vt][r];
  }
  __syncthreads();
  for (int i = t; i < F * LDT; i += SNT) {
    float s[SW];
#pragma unroll
    for (int k = 0; k < SW; ++k) s[k] = part[k * F * LDT + i];
    T[i] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
  }
  __syncthreads();
  // ---- queries
  int zero = 0;
  for (int tile = w; 16 * tile < a.Lq; tile += SW) {
#pragma unroll
    for (int q = 0; q < Q; ++q) xq[q] = 16 * q + 4 * g < d ? xq[q] * a.scale : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 p[MT];                             // rows = features, column = token
    float mx = -INFINITY;
#pragma unroll
    for (int ft = 0; ft < MT; ++ft) {
      p[ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const f32x4 wr = *(const f32x4*)(W + (16 * ft + c) * LDW + 16 * q + 4 * g);
#pragma unroll
        for (int s = 0; s < 4; ++s) p[ft] = mfma4(wr[s], xq[q][s], p[ft]);
      }
      const f32x4 br = *(const f32x4*)(bl + 16 * ft + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[ft][r] += br[r];
        mx = fmaxf(mx, p[ft][r]);
      }
    }
    const int next = 16 * (tile + SW) + c;   // the next tile's rows travel meanwhile
#pragma unroll
    for (int q = 0; q < Q; ++q) xq[q] = load4<BF>(a.Q, qb + (long long)min(next, a.Lq - 1) * a.Q.sl + min(16 * q + 4 * g, d - 4));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    f32x4 y[VT];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) y[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ft = 0; ft < MT; ++ft)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float f = fast_exp2(p[ft][r] - mx);
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) y[vt] = mfma4(f, T[(16 * ft + 4 * g + r) * LDT + 16 * vt + c], y[vt]);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * tile + 4 * g + r;
      float den = 0.f;
#pragma unroll
      for (int vt = 0; vt < VT; ++vt)
        if (vt == a.nv >> 4) den = y[vt][r];
      den = __shfl(den, 16 * g + (a.nv & 15));
      if (row < a.Lq) {
        zero += c == 0 && !(den > 0.f);
#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
          if (16 * vt + c < a.nv) store_elem(a.Y, yb + (long long)row * a.Y.sl + 16 * vt + c, den > 0.f ? y[vt][r] / den : 0.f);
      }
    }
  }
  zero += __shfl_xor(zero, 16);
  zero += __shfl_xor(zero, 32);
  if (!a.count) {
    if (lane == 0 && zero != 0) atomicAdd(a.flushed, (unsigned)zero);
    return;
  }
  if (lane == 0) zeros[w] = zero;
  __syncthreads();
  if (t == 0) {
    unsigned n = 0;
    for (int i = 0; i < SW; ++i) n += (unsigned)zeros[i];
    *a.flushed = n;
  }
}

template <class F>
int by_small(int d, int M, int dtype, F launch) {
  const std::integral_constant<int, 0> f32;
  const std::integral_constant<int, 1> bf16;
  const std::integral_constant<int, 1> q1;
  const std::integral_constant<int, 2> q2, m2;
  const std::integral_constant<int, 4> m4;
  if (d <= 16) return M <= 32 ? (dtype ? launch(q1, m2, bf16) : launch(q1, m2, f32)) : (dtype ? launch(q1, m4, bf16) : launch(q1, m4, f32));
  return M <= 32 ? (dtype ? launch(q2, m2, bf16) : launch(q2, m2, f32)) : (dtype ? launch(q2, m4, bf16) : launch(q2, m4, f32));
}

}  // namespace

// Which calls.  Times as five launches / this one, us.
// Rows of 32 numbers, 64 features and 256 keys are what LDS holds of the waves' parts of the state (eight waves, two tiles of keys each,
// their exponents in registers until the maximum is known).
// Queries: a workgroup takes all queries of its sequence, 128 at a time, where the five launches spread them over the chip.  From 96
// sequences on it is faster for any number of them (16384 queries: f32 d16 M64 416 / 310, bf16 d32 M64 554 / 509; 80 sequences 354 /
// 310, 469 / 508).  With fewer it may take only so many passes:
//   1 sequence    d32 M64 256 queries 28.7 / 25.5, 512 28.5 / 32.7;  d16 M64 512 30 / 21, 1024 31 / 30 (bf16 28 / 33), 65536 39 / 1203;
//                 d16 M32 1024 28 / 22, 2048 28 / 34
//   48 sequences  d32 M64 256 32 / 28, 512 33.7 / 35.3;  d16 M64 1024 36 / 32, 2048 48 / 51;  d16 M32 2048 37 / 36, 4096 53 / 61
// Tokens: sequences of a few tiles leave most of its waves without any, which counts once the sequences are several times the CUs
// (bf16, as many queries as keys):
//   1024 sequences  d8 M64 32 keys 39 / 49, 48 keys 50 / 49
//   2048 sequences  d32 M64 64 keys 137 / 154, 80 keys 171 / 171;  d32 M24 32 keys 67 / 71, 48 keys 83 / 72
//   8192 sequences  d8 M64 96 keys 361 / 405, 128 keys 445 / 405 (one query: 265 / 345);  d32 M24 96 keys 362 / 309
// 256 x 256 d16 M64 53 / 20, 2048 x 256 d32 M64 358 / 200.
bool gen_small_supported(int BH, int Lq, int Lk, int d, int dv, int M) {
  if (d % 4 || Lk > 16 * SW * KT || M > 64 || !(d <= 16 ? dv < 32 : d <= 32 && dv < 48)) return false;
  const int passes = (Lq + 16 * SW - 1) / (16 * SW), few = d > 16 ? 2 : M > 32 ? 4 : 8;
  if (BH < 96 && (long long)passes * (112 - BH) > 112 * few) return false;
  const int least = M > 32 ? (BH > 2048 ? 128 : BH > 1024 ? 80 : BH > 512 ? 48 : 1) : (BH > 2048 ? 96 : BH > 1024 && d > 16 ? 48 : 1);
  return (long long)Lq + Lk >= 2 * least;
}

int launch_gen_small(const TensorDev& Q, const TensorDev& K, const TensorDev& V, const TensorDev& Y, const float* theta, int groups,
                     const float* Omega, int omega_groups, int BH, int H, int Lq, int Lk, int d, int nv, int M, float scale,
                     unsigned* flushed, hipStream_t st) {
  if (BH > 1)
    if (int rc = launch_fill_u32(flushed, 0u, 1, st)) return rc;
  SmallArgs a{Q, K, V, Y, theta, Omega, groups, omega_groups, H, Lq, Lk, d, M, nv, scale, flushed, BH == 1};
  return by_small(d, M, Q.dtype, [&](auto q, auto mt, auto bf) {
    auto kernel = k_gen_small<q(), mt(), bf()>;
    const int lds = 4 * small_lds_floats<q(), mt()>();
    if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) {
      (void)hipGetLastError();
      return 2;
    }
    hipLaunchKernelGGL(kernel, dim3(BH), dim3(SNT), lds, st, a);
    return hipGetLastError() == hipSuccess ? 0 : 5;
  });
}

}  // namespace fs
