// Closed-form DERF parameter fits on the device: one workgroup per parameter group, fp64, no host round trip.
//
// Input: the data statistics of a group (mu4 = mean x, mu5 = mean y, M1 = mean x x^T, M2 = mean y y^T; Theorems on
// ADERF and SDERF), as the statistics kernels leave them.  Output: one theta block per group (layout in
// favorsharp.h) and one status word per group.
//
// The symmetric eigenproblems (M1, M2, and N = M1 + mu4 mu5^T + mu5 mu4^T + M2) are reduced to tridiagonal form by
// Householder reflections with the matrix in registers; eigenvalues from Sturm sequences, secants within the intervals that
// these keep, all of them side by side; eigenvectors of the tridiagonal matrix from twisted factorisations (Fernando; Parlett and Dhillon), one lane
// per vector; the reflections are then applied to them (`eig_tridiagonal`).  Where eigenvalues (nearly) coincide such
// vectors are not orthogonal by themselves: there the tridiagonal matrix is finished by implicit QR steps instead.
// The singular value problem of the ADERF matrix Lambda1^(1/2) Q1^T Q2 Lambda2^(1/2) is solved by the one-sided
// (Hestenes) Jacobi iteration on its columns, whose normalised columns are the left singular vectors, in the
// round-robin ordering: a round rotates d/2 disjoint index pairs at once, a few lanes per pair, one barrier per round,
// the matrix in LDS.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace fs {

namespace {

constexpr int FIT_NT = 512;      // threads per workgroup (256 and 1024 were measured: 30 % slower / no faster)
constexpr int FIT_DMAX = 128;
// A pair of columns counts as orthogonal below this cosine.  The statistics carry fp32 rounding of the inputs'
// products, so nothing is gained by iterating to the last bits of fp64.
constexpr double kJacobiEps = 1e-13;
// A sweep is followed by another one only if it met a pair above this cosine: the iteration converges quadratically,
// so a sweep whose largest cosine is below 1e-8 leaves nothing above 1e-15 behind, and the sweep that would only
// confirm that is not run.
constexpr double kJacobiAgain = 1e-8;

// Scalar minimiser of log(1-4A) - 1/2 log(1-8A) + phi/(1-8A)  (appendix lemma on the scalar objective).
__device__ __forceinline__ double a_star(double phi) {
  const double t = 2.0 * phi + 1.0;
  return (1.0 - 2.0 * phi - sqrt(t * t + 8.0 * phi)) / 16.0;
}

// Sum over a group of w consecutive lanes (w a power of two, groups aligned); every lane gets the same bits.
__device__ __forceinline__ double lanes_sum(double v, int w) {
  for (int m = w >> 1; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

struct FitShared {
  double nrm[3][FIT_DMAX];   // column norms after an iteration (eigenvalues / singular values, unsorted)
  double sgn[3][FIT_DMAX];   // sign that makes the largest component of an eigenvector positive
  int ord[3][FIT_DMAX];      // ord[k] = column with the k-th largest norm
  double red_row[FIT_DMAX];  // per-row scale factors of the results
  double red[8];             // scalars shared by the workgroup
  int twist[FIT_DMAX];
  int row[FIT_DMAX];         // rows of the matrix in the order of the eigenproblem: those with off-diagonal entries first
  int flag;
};

// Tangent of the Jacobi rotation that annihilates the off-diagonal entry `off` of a 2 x 2 block whose diagonal
// entries differ by `diff`: t = sign(z) / (|z| + sqrt(1 + z^2)), z = diff / (2 off).  The rotation must be orthogonal
// to fp64 accuracy, its angle need not be (an error of 1e-6 of the angle leaves 1e-6 of the pair's off-diagonal entry
// for the next sweep): fp32 with the hardware reciprocal and square root.  0, inf or NaN when there is nothing to
// rotate (the callers skip those).
__device__ __forceinline__ float rotation_tangent(float diff, float off) {
  const float zeta = diff * __builtin_amdgcn_rcpf(2.f * off);
  return copysignf(1.f, zeta) * __builtin_amdgcn_rcpf(fabsf(zeta) + __builtin_amdgcn_sqrtf(1.f + zeta * zeta));
}

// Cosine 1 / sqrt(1 + t^2) of the rotation with tangent t, |t| <= 1, to fp64 accuracy: the fp32 hardware estimate
// and two Newton steps (relative error 1e-7 -> 1e-14 -> below the rounding of fp64).
__device__ __forceinline__ double rotation_cosine(double t) {
  const double x = 1.0 + t * t;
  double c = (double)__builtin_amdgcn_rsqf((float)x);
  c = c * (1.5 - 0.5 * x * c * c);
  c = c * (1.5 - 0.5 * x * c * c);
  return c;
}

// Batched access to a pair of columns for the sizes where every lane of a pair handles exactly NI elements
// (n = NI x lanes per pair: 32, 64, 128 with 512 threads).  Every request is issued before the first use, so a pair
// costs one memory latency, not one per element as in the general loops (whose stores may alias the next loads).
template <int NI>
__device__ __forceinline__ void fetch_pair(const double* xp, const double* xq, int r0, int tpp, double (&x)[NI], double (&y)[NI]) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = r0 + i * tpp;
    x[i] = xp[r];
    y[i] = xq[r];
  }
}
// (xp, xq) <- (c xp - s xq, s xp + c xq) on those elements.
template <int NI>
__device__ __forceinline__ void store_rotated(double* xp, double* xq, int r0, int tpp, const double (&x)[NI], const double (&y)[NI],
                                              double c, double s) {
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int r = r0 + i * tpp;
    xp[r] = c * x[i] - s * y[i];
    xq[r] = s * x[i] + c * y[i];
  }
}

// One-sided Jacobi on the columns of g (n x n, column c at g + c * ldg): g <- g R with mutually orthogonal columns.
// All FIT_NT threads must call; n <= FIT_DMAX.  Inlined at each call site so that the compiler knows g to be in LDS.
// NI > 0: n = NI x (lanes per pair), batched accesses; NI = 0: any n.
template <int NI>
__device__ __forceinline__ void jacobi_columns(double* g, int n, int ldg, FitShared& sh) {
  const int np = (n + 1) / 2;        // pairs per round
  const int m = 2 * np;              // players of the tournament (player n is a bye when n is odd)
  int tpp = 64;                      // lanes per pair
  while (tpp * np > FIT_NT) tpp >>= 1;
  const int t = threadIdx.x, pair = t / tpp, r0 = t % tpp;
  constexpr int NA = NI > 0 ? NI : 1;
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (t == 0) sh.flag = 0;
    __syncthreads();
    // round-robin: player m-1 stays, the others walk round a circle of m-1 seats; in round `round` pair 0 is
    // (m-1, round), pair k is (round + k, round - k) modulo m-1.  The two seats advance by one per round.
    int pa = pair % (m - 1), pb = (m - 1 - pair) % (m - 1);
    for (int round = 0; round < m - 1; ++round) {
      if (pair < np) {
        int p = pair == 0 ? m - 1 : pa;
        int q = pair == 0 ? round : pb;
        if (p > q) { const int s = p; p = q; q = s; }
        if (q < n) {
          double* gp = g + (size_t)p * ldg;
          double* gq = g + (size_t)q * ldg;
          double al = 0.0, be = 0.0, ga = 0.0;
          double x[NA], y[NA];
          if constexpr (NI > 0) {
            fetch_pair<NA>(gp, gq, r0, tpp, x, y);
#pragma unroll
            for (int i = 0; i < NA; ++i) { al += x[i] * x[i]; be += y[i] * y[i]; ga += x[i] * y[i]; }
          } else {
            for (int r = r0; r < n; r += tpp) {
              const double a = gp[r], b = gq[r];
              al += a * a; be += b * b; ga += a * b;
            }
          }
          al = lanes_sum(al, tpp); be = lanes_sum(be, tpp); ga = lanes_sum(ga, tpp);
          // tangent in fp32, cosine and sine from it in fp64
          const float tn32 = rotation_tangent((float)(be - al), (float)ga);
          if (ga * ga > kJacobiEps * kJacobiEps * al * be && tn32 != 0.f && isfinite(tn32)) {
            const double tn = (double)tn32;
            const double c = rotation_cosine(tn), s = c * tn;
            if constexpr (NI > 0) {
              store_rotated<NA>(gp, gq, r0, tpp, x, y, c, s);
            } else {
              for (int r = r0; r < n; r += tpp) {
                const double a = gp[r], b = gq[r];
                gp[r] = c * a - s * b;
                gq[r] = s * a + c * b;
              }
            }
            if (r0 == 0 && ga * ga > kJacobiAgain * kJacobiAgain * al * be) sh.flag = 1;
          }
        }
      }
      pa = pa + 1 == m - 1 ? 0 : pa + 1;
      pb = pb + 1 == m - 1 ? 0 : pb + 1;
      __syncthreads();
    }
    const int again = sh.flag;
    __syncthreads();
    if (!again) break;
  }
}

// Place of v[t] in the descending order of v[0 .. n), ties by index.  The bits are compared, not the values: a total
// order, so that the places are a permutation (they become column indices) whatever the statistics were, NaN included.
__device__ __forceinline__ int descending_place(const double* v, int n, int t) {
  auto key = [](double x) {
    const long long b = __double_as_longlong(x + 0.0);       // (-0 counts as 0)
    return b < 0 ? b ^ 0x7fffffffffffffffll : b;
  };
  const long long mine = key(v[t]);
  int place = 0;
  for (int i = 0; i < n; ++i) {
    const long long k = key(v[i]);
    place += (k > mine || (k == mine && i < t)) ? 1 : 0;
  }
  return place;
}

// Singular values and left singular vectors of an n x n matrix in global memory (g, column-major with stride n): g <- g R
// with orthogonal columns; their norms, the singular values, and the norms' order go to slot k.  The matrix is copied to
// LDS for the iteration (column stride n + 1: columns start in different banks) and back afterwards.
__device__ __forceinline__ void decompose_columns(double* g, int n, int k, FitShared& sh, double* lds) {
  const int t = threadIdx.x, nn = n * n, ld = n + 1;
  for (int e = t; e < nn; e += FIT_NT) lds[(e / n) * ld + e % n] = g[e];
  __syncthreads();
  // (the sizes with a batched form: n = 64, 4 elements per lane, n = 128, 16; else the general one)
  if (n == 64) jacobi_columns<4>(lds, n, ld, sh);
  else if (n == 128) jacobi_columns<16>(lds, n, ld, sh);
  else jacobi_columns<0>(lds, n, ld, sh);
  if (t < n) {
    double s2 = 0.0;
    for (int r = 0; r < n; ++r) s2 += lds[(size_t)t * ld + r] * lds[(size_t)t * ld + r];
    sh.nrm[k][t] = sqrt(s2);
  }
  __syncthreads();
  if (t < n) sh.ord[k][descending_place(sh.nrm[k], n, t)] = t;
  for (int e = t; e < nn; e += FIT_NT) g[e] = lds[(e / n) * ld + e % n];
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------------
// Symmetric eigenproblem by reduction to tridiagonal form, one workgroup, everything in fp64.
//
// What bounds it is latency (one workgroup per matrix, a few matrices per call), so the design counts dependent steps:
// the reduction has one barrier per column against two barriers per rotation round of a Jacobi iteration, which
// needs (n - 1) x 6 - 8 rounds; everything after the reduction has no barrier per step at all.  Measured against a
// two-sided Jacobi iteration (8 matrices of 64: k_fit_device 686 -> 89 us; 16 matrices of 128: 7290 -> 313 us).
// ---------------------------------------------------------------------------------------------------

// Gap between neighbouring eigenvalues (in units of the norm) below which vectors from twisted factorisations are not
// used.  The eigenvalues carry an ulp or two of the norm, so the inner product of two vectors is about that over their
// gap: up to 2.5e-16 / gap on matrices of 2 .. 128 with pairs 1e-10 .. 1e-7 apart.  2.5e-8 at this limit, below the
// rounding of the fp32 results (6e-8); at a limit of 1e-10 it was up to 2e-6.
constexpr double kMinGap = 1e-8;
// Off-diagonal entries (in units of the norm) that the QR steps take for zero: below the rounding of the reduction.
constexpr double kQrTiny = 1e-16;

__device__ __forceinline__ double rcp64(double x) {        // hardware estimate and two Newton steps
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double rsqrt64(double x) {      // the estimate and one step of third order
  const double r = __builtin_amdgcn_rsq(x), h = fma(-x * r, r, 1.0);
  return fma(fma(h, 0.375, 0.5), h * r, r);
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141, kMirror16 = 0x140;      // DPP controls
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Exchanges the odd 16-lane rows of x with the even rows of y and adds: rows 0, 2 of the result are the sums of x over
// the row pairs (0, 1), (2, 3), rows 1, 3 those of y.
__device__ __forceinline__ double add_rows16(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double add_halves32(double x, double y) {     // the same with the two halves of the wave
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double sum8(double v) {         // over aligned groups of 8 lanes
  v += dpp64<kXor1>(v);
  v += dpp64<kXor2>(v);
  return v + dpp64<kMirror8>(v);
}
__device__ __forceinline__ double sum64(double v) {        // over the wave
  v = sum8(v);
  v += dpp64<kMirror16>(v);
  v = add_rows16(v, v);
  return add_halves32(v, v);
}
// The same through the matrix pipe: lane 16 k + 4 b + i of the first factor is entry (i, k) of block b, so that a product with ones is
// the sum over the rows of lanes and a second one that over groups of four.  (Six steps of lane swaps and adds, each waiting
// for the last, are 240 cycles.)
__device__ __forceinline__ double wave_sum(double v) {
  v = __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0);
  v = __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0);
  v += dpp64<kMirror8>(v);
  return v + dpp64<kMirror16>(v);
}
__device__ __forceinline__ double max64(double v) {        // over the wave
  v = fmax(v, dpp64<kXor1>(v));
  v = fmax(v, dpp64<kXor2>(v));
  v = fmax(v, dpp64<kMirror8>(v));
  v = fmax(v, dpp64<kMirror16>(v));
  auto pair = [](const auto& lo, const auto& hi) {
    return fmax(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
  };
  unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
  v = pair(__builtin_amdgcn_permlane16_swap(lo, lo, false, false), __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
  lo = (unsigned)__double2loint(v);
  hi = (unsigned)__double2hiint(v);
  return pair(__builtin_amdgcn_permlane32_swap(lo, lo, false, false), __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
}

// Eigenvalues and vectors of a tridiagonal matrix by implicit QR steps with Wilkinson shifts (Golub and Van Loan, section
// 8.3), for matrices with (nearly) equal eigenvalues: a product of rotations is orthogonal whatever the gaps are.
// (diagonal, .) pairs `de`, off-diagonal `es`, both of NP, at most 2 in size.  NP / 64 waves call it, a lane per component:
// lane i of them carries row i of the vectors (component i of vector j at Z[j NP + i], the identity at the start) through
// every rotation; the rotations themselves are a serial chain, which each wave computes on a copy of the matrix of its own
// (`mine`, 2 NP doubles): no barrier, no exchange.  The chain bounds it: about 1.1 n^2 rotations (fewer where blocks
// split off), each 14 dependent fp64 operations, 110 - 150 ns.  Measured against a two-sided Jacobi iteration on the
// original matrix, which is as orthogonal: fits of rank-2 rows, 8 heads, d 16 / 64 / 128 155 / 874 / 6796 -> 114 / 685 /
// 2303 us.  The eigenvalues, in no order, stay in mine[0 .. n).
template <int NP>
__device__ __forceinline__ void tridiagonal_qr(const f64x2* de, const double* es, int n, double* Z, double* mine) {
  const int lane = threadIdx.x & 63;
  double *dg = mine, *of = mine + NP, *zr = Z + (threadIdx.x & (NP - 1));
#pragma unroll
  for (int h = 0; h < NP / 64; ++h) {
    dg[lane + 64 * h] = de[lane + 64 * h].x;
    of[lane + 64 * h] = es[lane + 64 * h];
  }
  int q = n - 1;
  for (int left = 30 * n; left > 0; --left) {
    // what the lanes stored in the last step is read by all of them in this one
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    unsigned long long zero[2] = {0, 0};             // bit i: entry i is negligible (or NaN: the iteration ends)
#pragma unroll
    for (int h = 0; h < NP / 64; ++h) zero[h] = __ballot(!(fabs(of[lane + 64 * h]) > kQrTiny));
    auto below = [](const unsigned long long (&m)[2], int i) {      // highest set bit under bit i, or -1
      if (NP > 64 && i > 64) {
        const unsigned long long hi = m[1] << (128 - i);
        if (hi) return i - 1 - __clzll(hi);
      }
      const unsigned long long lo = i > 0 ? m[0] << (64 - min(i, 64)) : 0;
      return lo ? min(i, 64) - 1 - __clzll(lo) : -1;
    };
    const unsigned long long live[2] = {~zero[0], ~zero[1]};
    q = below(live, q) + 1;                          // the last unreduced block: p .. q
    if (q == 0) break;
    const int p = below(zero, q) + 1;
    const double dq = dg[q], b = of[q - 1], dl = 0.5 * (dg[q - 1] - dq);
    const double h2 = dl * dl + b * b;
    const double mu = dq - b * b * rcp64(dl + copysign(h2 * rsqrt64(h2), dl));
    double a = dg[p], e = of[p], g = dg[p + 1], en = of[p + 1], x = a - mu, w = e, y0 = zr[p * NP], y1 = zr[(p + 1) * NP];
    for (int k = p; k < q; ++k) {                    // rotate rows and columns k, k + 1: (x, w) -> (r, 0)
      const int kn = min(k + 2, q);
      const double gn = dg[kn], en2 = of[kn], yn = zr[kn * NP];
      const double r2 = x * x + w * w;
      double c = 1.0, s = 0.0, r = 0.0;
      if (r2 > 1e-290) {
        const double ir = rsqrt64(r2);
        c = x * ir;
        s = w * ir;
        r = r2 * ir;
      }
      if (k > p) of[k - 1] = r;
      const double u0 = c * a + s * e, u1 = c * e + s * g, v0 = c * e - s * a, v1 = c * g - s * e;
      dg[k] = c * u0 + s * u1;
      x = c * v0 + s * v1;                           // the entry (k, k + 1), and beyond it the bulge
      a = c * v1 - s * v0;
      w = s * en;
      e = c * en;
      zr[k * NP] = c * y0 + s * y1;
      y0 = c * y1 - s * y0;
      g = gn;
      en = en2;
      y1 = yn;
    }
    dg[q] = a;
    of[q - 1] = x;
    zr[q * NP] = y0;
  }
}

// LDS of `eig_tridiagonal` (doubles; NP = 32 RJ): reflectors [NP][NP], two vectors of NP, (diagonal, e^2) pairs, e,
// eigenvalues, partial norms, partial minima with their rows (one per thread; the QR steps' matrices); for NP = 64 also the
// multipliers of the twisted factorisations [2][NP][NP] (the QR steps' vectors; NP = 128: in place of the reflectors).
constexpr size_t tri_lds_doubles(int NP) { return (size_t)(NP == 64 ? 3 : 1) * NP * NP + 11 * (size_t)NP + FIT_NT + FIT_NT / 2; }

constexpr int TRI_WAVES = 4;      // waves that hold the matrix of eig_tridiagonal, one per SIMD, every fourth column each

// a: the matrix, entry (lane + 64 h, wave + 4 q) in a[q][h] of the first four waves, zero outside n x n
// (destroyed).  Any symmetric matrix: the statistics' matrices are positive semidefinite only up to the
// rounding of their fp32 sums, and where large means cancel that rounding is all there is.  Eigenvalues go to slot k of
// the shared block with their order and the signs of the vectors, eigenvector j to column j of v (column-major with stride
// ldv, component i in row sh.row[i]; may be the start of lds).  scr: 2 n n doubles of global scratch (NP = 128).  Statistics that are
// not finite give parameters that are not finite.
template <int RJ>
__device__ __forceinline__ void eig_tridiagonal(double (&a)[8 * RJ][RJ / 2], int n, double* v, int ldv, double* scr, int k_slot,
                                                FitShared& sh, double* lds) {
  constexpr int NP = 32 * RJ, RH = NP / 64, TW = TRI_WAVES, NQ0 = NP / TW, QB = NQ0 / 4;
  constexpr bool kInLds = NP == 64;
  double* refl = lds;                                // reflector k: refl[k * NP + i], zero for i <= k
  double* col = refl + (size_t)NP * NP;
  double* pv = col + NP;
  f64x2* de = (f64x2*)(pv + NP);                     // (d_i, e_{i-1}^2)
  double* es = (double*)(de + NP);
  double* lam = es + NP;
  double* nsq = lam + NP;                            // [2][NP]
  double* part_val = nsq + 2 * NP;
  int* part_arg = (int*)(part_val + FIT_NT);
  double* mul = part_val + FIT_NT + FIT_NT / 2;      // NP = 64: [2][n][n]
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);

  // ---- Householder reduction: A <- H A H with H = I - tau v v^T, column by column: v = x - beta e (x: the entries of column k
  // below the diagonal, e: unit vector k + 1, beta = -sign(x_0) |x|), tau = 1 / (|x| (|x| + |x_0|)), y = A v,
  // A <- A - tau (v y^T + (y - tau (v^T y) v) v^T).  What bounds a step is the latency of its dependent fp64 operations and of
  // its passes through LDS (a wave per SIMD).  A lane holds rows and a wave columns: A x takes no exchange between lanes, the
  // numbers of a wave's columns (x_j, y_j) are broadcast reads of LDS.  The product is taken with the raw column, beside the chain of
  // the norm: A v = A x - beta A e, A e being column k + 1, and v^T A v likewise from x^T A x.  From the parts of the product
  // every wave has the next column for itself (column k + 1 after the update), so there is one barrier per column.  Column k + 1
  // is finished then and goes without its share of beta; finished rows go on being rotated, their norms stay.  The loop over
  // blocks of a quarter of the columns is unrolled so that finished columns are skipped at compile time.  Against a thread per 8 x 2
  // entries with rows and columns both over lanes, u made before the product and two barriers a column: 2060 -> 1700 cycles per
  // column at n = 64, 2700 -> 2600 at n = 128.
  double* prt = lam;                                 // [2][4][NP] parts of A x, by wave and row (lam, nsq, part_val: not yet in use)
  double* sw = prt + 8 * NP;                         // [2][4] x^T A x, a part per wave
  double* xy = sw + 8 + 3 * NQ0 * wave;              // y, x of the wave's columns, [2] x
  double x[RH], ax[RH] = {};                         // x, and the wave's part of A x
  {
    if (wave == 0)
#pragma unroll
      for (int h = 0; h < RH; ++h) col[lane + 64 * h] = a[0][h];
    if (wave == 1)
#pragma unroll
      for (int h = 0; h < RH; ++h) pv[lane + 64 * h] = a[0][h];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < RH; ++h) {
      const int i = lane + 64 * h;
      x[h] = i > 0 ? col[i] : 0.0;
      if (t == 0 && h == 0) de[0].x = col[0];
    }
    if (wave < TW) {
#pragma unroll
      for (int h = 0; h < RH; ++h)
        if ((lane & (TW - 1)) == wave) xy[NQ0 + (lane + 64 * h) / TW] = x[h];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int q = 0; q < NQ0 / 2; ++q) {
        const f64x2 xj = ((const f64x2*)(xy + NQ0))[q];
#pragma unroll
        for (int h = 0; h < RH; ++h) ax[h] += a[2 * q][h] * xj.x + a[2 * q + 1][h] * xj.y;
      }
    }
    __syncthreads();
  }
  auto columns = [&](auto Q0) {
    constexpr int q0 = Q0();
#pragma unroll 1
    for (int k = TW * q0; k < min(n - 2, TW * (q0 + QB)); ++k) {
      double* pk = prt + 4 * NP * (k & 1);
      double* sk = sw + 4 * (k & 1);
      double *xo = xy + NQ0 * (1 + (k & 1)), *xn = xy + NQ0 * (2 - (k & 1));      // x of this step and the next
      double *c2p = k & 1 ? col : pv, *c2n = k & 1 ? pv : col;      // column k + 1, and k + 2 after this step
      double beta = 0.0, tau = 0.0, x0 = 0.0;
      if (wave < TW) {
        double n2 = 0.0, xax = 0.0;
#pragma unroll
        for (int h = 0; h < RH; ++h) n2 += x[h] * x[h];
        n2 = wave_sum(n2);
#pragma unroll
        for (int h = 0; h < RH; ++h) {
          pk[NP * wave + lane + 64 * h] = ax[h];
          xax += x[h] * ax[h];
        }
        xax = wave_sum(xax);
        if (lane == 0) sk[wave] = xax;
        const int l0 = (k + 1) & 63;                 // x_0 = x of row k + 1
        double xs = x[0];
        if constexpr (RH == 2) xs = k + 1 < 64 ? x[0] : x[RH - 1];
        x0 = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(xs), l0), __builtin_amdgcn_readlane(__double2loint(xs), l0));
        if (n2 > 1e-290) {
          const double nrm = n2 * rsqrt64(n2);
          beta = -copysign(nrm, x0);
          tau = rcp64(fma(nrm, fabs(x0), n2));
        }
      }
      __syncthreads();
      if (wave < TW) {
        const f64x2 s01 = *(const f64x2*)sk, s23 = *(const f64x2*)(sk + 2);
        const double a11 = c2p[k + 1];
        const double ax0 = (pk[k + 1] + pk[NP + k + 1]) + (pk[2 * NP + k + 1] + pk[3 * NP + k + 1]);
        const double y0 = ax0 - beta * a11, v0 = x0 - beta;          // y and v of row k + 1
        const double c = tau * (((s01.x + s01.y) + (s23.x + s23.y)) - beta * (ax0 + y0));
        double tv[RH], ty[RH];
#pragma unroll
        for (int h = 0; h < RH; ++h) {
          const int i = lane + 64 * h;
          const double c2 = c2p[i];
          const double y = ((pk[i] + pk[NP + i]) + (pk[2 * NP + i] + pk[3 * NP + i])) - beta * c2;
          const double v = i == k + 1 ? v0 : x[h];
          if (wave == 0) refl[(size_t)k * NP + i] = i == k ? tau : v;
          tv[h] = tau * v;
          ty[h] = tau * (y - c * v);
          const double full = c2 - ty[h] * v0 - tv[h] * y0;
          if (wave == 0 && i == k + 1) {
            de[k + 1].x = full;
            es[k] = beta;
          }
          x[h] = i > k + 1 ? full : 0.0;
          if ((lane & (TW - 1)) == wave) {
            xn[i / TW] = x[h];
            xy[i / TW] = y;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        double s[RH][2] = {};
#pragma unroll
        for (int q = q0 / 2; q < NQ0 / 2; ++q) {     // the update, and the product with the next x
          const f64x2 xj = ((const f64x2*)xo)[q], yj = ((const f64x2*)xy)[q], nj = ((const f64x2*)xn)[q];
#pragma unroll
          for (int h = 0; h < RH; ++h) {
            a[2 * q][h] = fma(-tv[h], yj.x, fma(-ty[h], xj.x, a[2 * q][h]));
            a[2 * q + 1][h] = fma(-tv[h], yj.y, fma(-ty[h], xj.y, a[2 * q + 1][h]));
            s[h][0] = fma(a[2 * q][h], nj.x, s[h][0]);
            s[h][1] = fma(a[2 * q + 1][h], nj.y, s[h][1]);
          }
        }
#pragma unroll
        for (int h = 0; h < RH; ++h) ax[h] = s[h][0] + s[h][1];
        if (wave == ((k + 2) & (TW - 1))) {
          const int q = (k + 2) / TW - q0;           // at most the first column of the next block
          auto pick = [&](double lo, double hi, int bit) { return q & bit ? hi : lo; };
#pragma unroll
          for (int h = 0; h < RH; ++h) {
            double r = pick(pick(a[q0][h], a[q0 + 1][h], 1), pick(a[q0 + 2][h], a[q0 + 3][h], 1), 2);
            if constexpr (QB == 8)
              r = pick(r, pick(pick(a[q0 + 4][h], a[q0 + 5][h], 1), pick(a[q0 + 6][h], a[q0 + 7][h], 1), 2), 4);
            if constexpr (q0 + QB < NQ0) r = pick(r, a[q0 + QB][h], QB);
            c2n[lane + 64 * h] = r;
          }
        }
      }
    }
  };
  columns(std::integral_constant<int, 0>());
  columns(std::integral_constant<int, QB>());
  columns(std::integral_constant<int, 2 * QB>());
  columns(std::integral_constant<int, 3 * QB>());
  __syncthreads();
  if (n > 1 && t == n - 1) {                         // the last two columns
    de[n - 1].x = (n & 1 ? col : pv)[n - 1];
    es[n - 2] = t < 64 ? x[0] : x[RH - 1];
  }
  for (int k = wave; k < n - 2; k += FIT_NT / 64) {  // reflectors as u = v sqrt(tau), |u|^2 = 2 (tau waits in entry k)
    double* u = refl + (size_t)k * NP;
    const double tau = u[k], f = tau > 0.0 ? tau * rsqrt64(tau) : 0.0;
#pragma unroll
    for (int h = 0; h < RH; ++h) {
      const int i = lane + 64 * h;
      u[i] = i == k ? 0.0 : f * u[i];
    }
  }
  __syncthreads();
  // in units of the largest Gershgorin radius about zero (every wave finds it for itself), which no eigenvalue exceeds
  // in size; off-diagonal entries at least 1e-17 (far below the rounding of the reduction), so that no Sturm sequence and
  // no factorisation meets an exact split; entries behind the matrix keep the sign of a sequence
  double scale = 0.0;
#pragma unroll
  for (int q = 0; q < NP / 64; ++q) {
    const int i = lane + 64 * q;
    if (i < n) {
      const double r = fabs(de[i].x) + (i > 0 ? fabs(es[i - 1]) : 0.0) + (i < n - 1 ? fabs(es[i]) : 0.0);
      scale = fmax(scale, r < 1e120 ? r : 1e300);
    }
  }
  scale = max64(scale);
  if (!(scale > 1e-120 && scale < 1e120)) scale = 1.0;     // a matrix of zeros, or one that is not finite
  {
    const double inv = rcp64(scale);
    double dd = 2.0, e2 = 1e-34;
    if (t < NP) {
      if (t < n) dd = de[t].x * inv;
      if (t >= 1 && t < n) { const double e = fmax(fabs(es[t - 1] * inv), 1e-17); e2 = e * e; }
    }
    double ee = 0.0;
    if (t < n - 1) { ee = es[t] * inv; if (fabs(ee) < 1e-17) ee = 1e-17; }
    __syncthreads();
    if (t < NP) { de[t] = f64x2{dd, e2}; es[t] = ee; }
    __syncthreads();
  }

  // ---- eigenvalues: 256 / NP lanes per eigenvalue.  They split its interval into as many parts + 1 until it holds no other
  // eigenvalue; then they stand about the zero of the secant through the characteristic polynomial at its ends, at distances that
  // shrink with the secant's error (to the square of the interval).  Which part is kept is decided by the Sturm counts
  // alone, and a step whose guess missed is followed by a split into equal parts.  (Equal parts throughout, 24 steps at n = 64 and 35
  // at n = 128: 51 k and 139 k cycles, now 37 k and 98 k.)  The sequence of leading
  // minors in its three-term form: one dependent multiply-add per row, rescaled every 16 rows (a factor of at least
  // 1e-34 per two rows: no underflow before).  One wave per SIMD: with twice the lanes (and a quarter fewer steps) the
  // waves share the fp64 issue slots (50 k -> 60 k cycles at n = 64).
  if (t < 256) {
    constexpr int S = 256 / NP;
    const int j = t / S, sec = t % S;
    const double frac = (double)(sec + 1) / (double)(S + 1);
    constexpr double kFirst = 1.0 / 16.0;
    // the ends of the interval, the polynomial m 2^e there, the eigenvalues below
    double lo = -1.0 - 1e-9, hi = 1.0 + 1e-9, lo_m = 0.0, hi_m = 0.0;
    int lo_e = 0, hi_e = 0, lo_cnt = 0, hi_cnt = n;
    double eta = 0.0;                                // distance from the guess, in intervals; 0: equal parts
    bool done = j >= n;
    // Steps: equal parts, and so every second step at the least, leave a third (n <= 64: a fifth) of the interval: 36 of them from 2 down
    // to 3e-17, 72 steps if every guess missed.  Spectra of all kinds (graded over 15 decades, clusters 1e-9 wide) take up to 38.
    for (int it = 0; it < 74; ++it) {
      const double w = hi - lo, third = fma(w, frac, lo);
      double x = third, in = 0.0;
      if (eta > 0.0) {
        const double ratio = ldexp(fabs(hi_m), hi_e - lo_e) * rcp64(fabs(lo_m));
        const double r = fma(w, rcp64(1.0 + ratio), lo), least = fma(fabs(r), 1.2e-16, 3e-17);
        in = fmax((S == 4 ? eta * eta : eta) * w, least);
        const double out = fmax(eta * w, 2.0 * in);
        const double d = S == 4 && (sec == 0 || sec == 3) ? out : in;
        x = sec < S / 2 ? r - d : r + d;
        x = x > lo && x < hi ? x : third;        // (outside, or not a number)
      }
      double p1 = 1.0, p2 = 0.0;
      unsigned bits = 0;
      int cnt = 0, ex_sum = 0;
      for (int i0 = 0; i0 < n; i0 += 16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const f64x2 c = de[i0 + i];
          const double p = fma(c.x - x, p1, -(c.y * p2));
          p2 = p1;
          p1 = p;
          bits = __builtin_amdgcn_alignbit(bits, (unsigned)__double2hiint(p), 31);     // shift the sign in
        }
        cnt += __popc((bits ^ (bits >> 1)) & 0xffffu);
        const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = ldexp(p1, -ex);
        p2 = ldexp(p2, -ex);
        ex_sum += ex;
      }
      const bool up = cnt <= j && x > lo, down = cnt > j && x < hi;
      double nlo = up ? x : lo, nhi = down ? x : hi, nlo_m = up ? p1 : lo_m, nhi_m = down ? p1 : hi_m;
      int nlo_e = up ? ex_sum : lo_e, nhi_e = down ? ex_sum : hi_e, nlo_cnt = up ? cnt : lo_cnt, nhi_cnt = down ? cnt : hi_cnt;
      auto over = [&](auto CTRL) {                   // the larger lower end, the smaller upper end of two lanes
        constexpr int ctrl = CTRL();
        const double ol = dpp64<ctrl>(nlo), oh = dpp64<ctrl>(nhi), olm = dpp64<ctrl>(nlo_m), ohm = dpp64<ctrl>(nhi_m);
        const int ole = __builtin_amdgcn_update_dpp(0, nlo_e, ctrl, 0xf, 0xf, true);
        const int ohe = __builtin_amdgcn_update_dpp(0, nhi_e, ctrl, 0xf, 0xf, true);
        const int olc = __builtin_amdgcn_update_dpp(0, nlo_cnt, ctrl, 0xf, 0xf, true);
        const int ohc = __builtin_amdgcn_update_dpp(0, nhi_cnt, ctrl, 0xf, 0xf, true);
        const bool l = ol > nlo, h = oh < nhi;
        nlo = l ? ol : nlo;
        nlo_m = l ? olm : nlo_m;
        nlo_e = l ? ole : nlo_e;
        nlo_cnt = l ? olc : nlo_cnt;
        nhi = h ? oh : nhi;
        nhi_m = h ? ohm : nhi_m;
        nhi_e = h ? ohe : nhi_e;
        nhi_cnt = h ? ohc : nhi_cnt;
      };
      over(std::integral_constant<int, kXor1>());
      if constexpr (S == 4) over(std::integral_constant<int, kXor2>());
      if (!done) {
        lo = nlo;
        lo_m = nlo_m;
        lo_e = nlo_e;
        lo_cnt = nlo_cnt;
        hi = nhi;
        hi_m = nhi_m;
        hi_e = nhi_e;
        hi_cnt = nhi_cnt;
        const double wn = hi - lo;
        if (eta > 0.0) {                             // the guess is good to the square of eta, to eta, or not
          if (wn <= 2.5 * in) eta = fmin(4.0 * eta * eta, kFirst);
          else if (!(S == 4 && wn <= 2.5 * eta * w)) eta = 0.0;
        } else if (lo_cnt == j && hi_cnt == j + 1) {
          eta = kFirst;
        }
        done = wn <= fma(fmax(fabs(lo), fabs(hi)), 2.3e-16, 3e-17);
      }
      if (!__any(!done)) break;
    }
    if (sec == 0) lam[j] = 0.5 * (lo + hi);
  }
  if (t == 0) sh.flag = 0;
  __syncthreads();
  if (t < n - 1 && !(lam[t + 1] - lam[t] > kMinGap)) sh.flag = 1;
  __syncthreads();
  const bool close = sh.flag;

  // what the last stage starts from: the components of the vector that a thread holds there, sixteen vectors a wave, four lanes
  // (a row of lanes apart) per vector, each with rows 2 part + 8 q + {0, 1}
  constexpr int NQ = NP / 8;
  const int part = lane >> 4, vec = 16 * wave + (lane & 15);
  const bool holds = 16 * wave < NP;
  double z[2 * NQ];
  if (close) {
    double* Z = kInLds ? mul : refl;
    if (!kInLds) {                                   // (the reflectors wait in global memory)
      for (int e = t; e < n * n; e += FIT_NT) scr[e] = refl[(size_t)(e / n) * NP + e % n];
      __syncthreads();
    }
    for (int e = t; e < NP * NP; e += FIT_NT) Z[e] = e / NP == e % NP ? 1.0 : 0.0;
    __syncthreads();
    if (t < NP) {
      double* mine = part_val + wave * 2 * NP;
      tridiagonal_qr<NP>(de, es, n, Z, mine);
      if (wave == 0) {
#pragma unroll
        for (int h = 0; h < NP / 64; ++h) lam[lane + 64 * h] = mine[lane + 64 * h];
      }
    }
    __syncthreads();
    if (t < n) sh.twist[t] = descending_place(lam, n, t);
#pragma unroll
    for (int q = 0; q < 2 * NQ; ++q) z[q] = Z[min(vec, NP - 1) * NP + 2 * part + 8 * (q >> 1) + (q & 1)];
    __syncthreads();
    if (!kInLds) {
      for (int e = t; e < n * NP; e += FIT_NT) refl[e] = e % NP < n ? scr[(size_t)(e / NP) * n + e % NP] : 0.0;
      __syncthreads();
    }
  } else {
    // ---- eigenvectors of the tridiagonal matrix.  Forward and backward factorisations of T - lambda_j, a lane per j:
    // l_i = e_i / D+_i and u_i = e_i / D-_{i+1}; the twist index r minimises |gamma_i| (largest component of the vector).
    // The pivots are quotients of successive minors, so that the chain from row to row is the minors' recurrence and the
    // divisions run beside it.
    double* fl = kInLds ? mul : scr;                   // l_i of vector j at fl[i * n + j], later its component i (i < r)
    double* bu = fl + (size_t)n * n;                   // u_i, later component i + 1 (i >= r)
    constexpr int NW = NP / 64;                        // waves per direction
    constexpr double kTiny = 1e-30;                    // smallest pivot (far below the error of the eigenvalue)
    const int vj = min(t & (NP - 1), n - 1);
    const bool mine = (t & (NP - 1)) < n, fwd = wave < NW, bwd = wave >= NW && wave < 2 * NW;
    const double lj = lam[vj];
    if (fwd || bwd) {
      const int r0 = fwd ? 0 : n - 1, step = fwd ? 1 : -1, eoff = fwd ? 0 : -1;
      double* out = (fwd ? fl : bu) + vj;
      double p1 = 1.0, p2 = 0.0, e2 = 0.0;
      auto row = [&](int i) {
        const double e = es[i + eoff];
        double p = fma(de[i].x - lj, p1, -(e2 * p2));
        p = copysign(fmax(fabs(p), kTiny * fabs(p1)), p);
        out[(i + eoff) * n] = e * p1 * rcp64(p);       // (lanes past the last vector repeat it)
        e2 = e * e;
        p2 = p1;
        p1 = p;
      };
      int i0 = 0;
      for (; i0 + 8 <= n - 1; i0 += 8) {
#pragma unroll
        for (int m = 0; m < 8; ++m) row(r0 + step * (i0 + m));
        const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = ldexp(p1, -ex);
        p2 = ldexp(p2, -ex);
      }
      for (; i0 < n - 1; ++i0) row(r0 + step * i0);
    }
    __syncthreads();
    {   // gamma_i = d_i - lambda - u_i e_i - l_{i-1} e_{i-1}: NT / NP threads per vector, a range of rows each
      constexpr int NC = FIT_NT / NP;
      const int c = t / NP, len = (n + NC - 1) / NC;
      double best = 1e300;
      int arg = 0;
      for (int i0 = c * len; i0 < min(n, (c + 1) * len); i0 += 16) {
        double ub[16], lb[16];             // (sixteen rows' loads in flight; clamped, as es is zero past the last row)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          ub[q] = bu[(size_t)min(i0 + q, max(n - 2, 0)) * n + vj];
          lb[q] = fl[(size_t)min(max(i0 + q - 1, 0), max(n - 2, 0)) * n + vj];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int i = i0 + q;
          if (i < min(n, (c + 1) * len)) {
            double g = de[i].x - lj;
            if (i < n - 1) g -= ub[q] * es[i];
            if (i > 0) g -= lb[q] * es[i - 1];
            if (fabs(g) < best) { best = fabs(g); arg = i; }
          }
        }
      }
      part_val[t] = best;
      part_arg[t] = arg;
    }
    __syncthreads();
    int rtw = part_arg[t & (NP - 1)];
    {
      double best = part_val[t & (NP - 1)];
#pragma unroll
      for (int i = (t & (NP - 1)) + NP; i < FIT_NT; i += NP)
        if (part_val[i] < best) { best = part_val[i]; rtw = part_arg[i]; }
    }
    if (fwd && mine) {
      double z = 1.0, q = 0.0;
      for (int i0 = n - 2; i0 >= 0; i0 -= 16) {
        double l[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) l[m] = fl[(size_t)max(i0 - m, 0) * n + vj];
#pragma unroll
        for (int m = 0; m < 16; ++m)
          if (i0 - m >= 0 && i0 - m < rtw) {
            z *= -l[m];
            q += z * z;
            fl[(size_t)(i0 - m) * n + vj] = z;
          }
      }
      nsq[vj] = q;
    } else if (bwd && mine) {
      double z = 1.0, q = 0.0;
      for (int i0 = 0; i0 < n - 1; i0 += 16) {
        double u[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) u[m] = bu[(size_t)min(i0 + m, n - 2) * n + vj];
#pragma unroll
        for (int m = 0; m < 16; ++m)
          if (i0 + m < n - 1 && i0 + m >= rtw) {
            z *= -u[m];
            q += z * z;
            bu[(size_t)(i0 + m) * n + vj] = z;
          }
      }
      nsq[NP + vj] = q;
    }
    if (t < NP) sh.twist[t] = rtw;
    __syncthreads();
    if (holds) {
      const int jc = min(vec, n - 1), rt = sh.twist[jc];
      const double sc = vec < n ? rsqrt64(1.0 + nsq[jc] + nsq[NP + jc]) : 0.0;
#pragma unroll
      for (int q = 0; q < 2 * NQ; ++q) {
        const int i = 2 * part + 8 * (q >> 1) + (q & 1), ic = min(i, n - 1);
        const double x = *(i < rt ? fl + (size_t)ic * n + jc : bu + (size_t)max(ic - 1, 0) * n + jc);
        z[q] = i < n ? (i == rt ? sc : x * sc) : 0.0;
      }
    }
  }

  // ---- the reflections applied to the vectors, their products summed over the parts by the matrix pipe.
  // (sixteen reflectors per block, so that the rows above them are skipped at compile time; the next reflector is
  // requested while the current one is used)
  if (holds) {
#pragma unroll
    for (int jb = NP / 16 - 1; jb >= 0; --jb) {
      const int ktop = min(n - 3, 16 * jb + 15);
      if (ktop < 16 * jb) continue;
      auto load = [&](f64x2 (&u)[NQ], int k) {
        const f64x2* up = (const f64x2*)(refl + (size_t)max(k, 0) * NP) + part;
#pragma unroll
        for (int q = 2 * jb; q < NQ; ++q) u[q] = up[4 * q];
      };
      auto reflect = [&](const f64x2 (&u)[NQ]) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 2 * jb; q < NQ; ++q) {
          s[2 * (q & 1)] += u[q].x * z[2 * q];
          s[2 * (q & 1) + 1] += u[q].y * z[2 * q + 1];
        }
        const double sm = -__builtin_amdgcn_mfma_f64_4x4x4f64(1.0, (s[0] + s[1]) + (s[2] + s[3]), 0.0, 0, 0, 0);
#pragma unroll
        for (int q = 2 * jb; q < NQ; ++q) {
          z[2 * q] = fma(u[q].x, sm, z[2 * q]);
          z[2 * q + 1] = fma(u[q].y, sm, z[2 * q + 1]);
        }
      };
      f64x2 ua[NQ], ub[NQ];
      load(ua, ktop);
      int k = ktop;
#pragma unroll 1
      for (; k > 16 * jb; k -= 2) {
        load(ub, k - 1);
        reflect(ua);
        load(ua, k - 2);
        reflect(ub);
      }
      if (k == 16 * jb) reflect(ua);
    }
  }
  __syncthreads();                                   // (v may be where the reflectors are)
  // results: vectors, and per vector the sign that makes its largest component positive (lowest index on ties)
  if (holds) {
    double big = 0.0;
    int at = 0;
#pragma unroll
    for (int q = 0; q < 2 * NQ; ++q) {
      const int i = 2 * part + 8 * (q >> 1) + (q & 1);
      if (vec < n && i < n) v[(size_t)vec * ldv + sh.row[i]] = z[q];
      if (fabs(z[q]) > fabs(big)) { big = z[q]; at = i; }
    }
    for (int m = 16; m < 64; m <<= 1) {
      const double ob = __shfl_xor(big, m, 64);
      const int oa = __shfl_xor(at, m, 64);
      if (fabs(ob) > fabs(big) || (fabs(ob) == fabs(big) && oa < at)) { big = ob; at = oa; }
    }
    if (part == 0 && vec < n) {
      sh.sgn[k_slot][vec] = big < 0.0 ? -1.0 : 1.0;
      sh.nrm[k_slot][vec] = lam[vec] * scale;
      sh.ord[k_slot][close ? sh.twist[vec] : n - 1 - vec] = vec;      // (in ascending order)
    }
  }
  __syncthreads();
}

// Eigen-decomposition of the symmetric matrix entry(i, j): into slot k as above, the vectors to the start of lds (stride n + 2:
// vectors side by side in different banks).  A row without
// off-diagonal entries (zero-padded dimensions) is left out of the eigenproblem: its diagonal entry is an eigenvalue, its
// unit vector the eigenvector.  Several such rows would have equal eigenvalues and send the whole matrix through the QR
// steps: fits with a quarter of the coordinates zero, 8 heads, d 16 / 64 / 128 take 78 / 145 / 378 us, with them 121 /
// 723 / 2504.
template <int RJ, class Entry>
__device__ __forceinline__ void decompose_symmetric(Entry entry, double* scr, int n, int k, FitShared& sh, double* lds) {
  double* v = lds;
  constexpr int RH = RJ / 2, TW = TRI_WAVES, NQ = 8 * RJ;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  double a[NQ][RH];
  // The entries by way of LDS: all waves fetch, eight rows each in flight (by the four waves that hold the matrix, entry by entry: 25 k
  // cycles at n = 128)
  for (int r0 = wave; r0 < n; r0 += 8 * (FIT_NT / 64)) {
    double e[8][RH];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < RH; ++h) e[i][h] = entry(min(r0 + (FIT_NT / 64) * i, n - 1), min(lane + 64 * h, n - 1));
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < RH; ++h) {
        const int r = r0 + (FIT_NT / 64) * i, c = lane + 64 * h;
        if (r < n && c < n) lds[(size_t)r * n + c] = e[i][h];
      }
  }
  // rows and columns row_of(0 .. m - 1) of it
  auto load = [&](int m, auto row_of) {
    if (wave >= TW) return;
#pragma unroll
    for (int h = 0; h < RH; ++h) {
      const double* at = lds + row_of(min(lane + 64 * h, m - 1));
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const double e = at[row_of(min(wave + TW * q, m - 1)) * n];
        a[q][h] = wave + TW * q < m && lane + 64 * h < m ? e : 0.0;
      }
    }
  };
  if (t < n) {
    sh.row[t] = t;
    sh.twist[t] = 0;
  }
  __syncthreads();
  load(n, [](int i) { return i; });
  if (wave < TW) {                                   // rows with an off-diagonal entry
#pragma unroll
    for (int h = 0; h < RH; ++h) {
      unsigned bits = 0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const unsigned b = ((unsigned)__double2hiint(a[q][h]) << 1) | (unsigned)__double2loint(a[q][h]);
        bits |= wave + TW * q == lane + 64 * h ? 0u : b;
      }
      if (bits != 0u) sh.twist[lane + 64 * h] = 1;
    }
  }
  __syncthreads();
  unsigned long long off[RJ / 2];
  int coupled = 0;
#pragma unroll
  for (int h = 0; h < RJ / 2; ++h) {
    off[h] = __ballot(lane + 64 * h < n && sh.twist[lane + 64 * h] != 0);
    coupled += __popcll(off[h]);
  }
  if (coupled < n) {
    if (t < n) {
      int before = __popcll(off[RJ / 2 - 1] & ((1ull << lane) - 1));
      if (t < 64) before = __popcll(off[0] & ((1ull << lane) - 1));
      else before += __popcll(off[0]);
      sh.row[sh.twist[t] ? before : coupled + t - before] = t;
    }
    __syncthreads();
    if (coupled > 0) load(coupled, [&](int i) { return sh.row[i]; });
    __syncthreads();
  }
  if (coupled > 0) eig_tridiagonal<RJ>(a, coupled, v, n + 2, scr, k, sh, lds);
  if (coupled < n) {
    for (int e = t; e < n * n; e += FIT_NT) {
      const int j = e / n, i = e % n;
      if (j >= coupled || i >= coupled) v[(size_t)j * (n + 2) + sh.row[i]] = i == j ? 1.0 : 0.0;
    }
    if (t >= coupled && t < n) {
      sh.nrm[k][t] = entry(sh.row[t], sh.row[t]);
      sh.sgn[k][t] = 1.0;
    }
    __syncthreads();
    if (t < n) sh.ord[k][descending_place(sh.nrm[k], n, t)] = t;
    __syncthreads();
  }
}

__device__ void write_header(float* th, double logD, double lbar, int flags, int variant) {
  th[0] = (float)logD;
  th[1] = (float)lbar;
  th[2] = (float)flags;
  th[3] = (float)variant;
  th[4] = th[5] = th[6] = th[7] = 0.f;
}

// grid (groups), block FIT_NT.  stats: per group [M1 d*d, mu4 d][M2 d*d, mu5 d]; ws: per group 5 d*d doubles.
// RJ: d <= 32 RJ (of eig_tridiagonal, which four waves enter with RJ / 2 rows per lane and 8 RJ columns each).
template <int RJ>
__global__ void __launch_bounds__(FIT_NT) k_fit_device(int variant, int d, const double* stats, double ridge, double* ws,
                                                       float* theta, int* status, size_t theta_floats) {
  extern __shared__ __align__(16) unsigned char fit_lds[];
  __shared__ FitShared sh;
  const int t = threadIdx.x, grp = blockIdx.x, n = d, nn = d * d;
  const size_t per = (size_t)nn + d;
  const double* M1 = stats + (size_t)grp * 2 * per;
  const double* mu4 = M1 + nn;
  const double* M2 = M1 + per;
  const double* mu5 = M2 + nn;
  float* th = theta + (size_t)grp * theta_floats;
  float* A = th + 8;
  float* B1 = A + d;
  float* B2 = B1 + nn;
  float* C1 = B2 + nn;
  float* C2 = C1 + nn;
  double* w = ws + (size_t)grp * 5 * nn;
  double* lds = (double*)fit_lds;
  const double nan = __builtin_nan("");

  // traces and mu4 . mu5 (every wave sums them for itself: d <= 128 terms)
  double tr1 = 0.0, tr2 = 0.0, dot = 0.0;
  auto traces = [&]() {
    for (int l = t & 63; l < d; l += 64) {
      tr1 += M1[(size_t)l * d + l];
      tr2 += M2[(size_t)l * d + l];
      dot += mu4[l] * mu5[l];
    }
    tr1 = sum64(tr1);
    tr2 = sum64(tr2);
    dot = sum64(dot);
  };

  if (variant <= 2) {                                   // PosRF, GERF, SADERF: A = a I, diagonal B and C
    traces();
    // psi_l = (M2_ll / M1_ll)^(1/4) for SADERF, 1 otherwise
    bool bad = false;
    double s = variant == 2 ? 2.0 * dot : tr1 + tr2 + 2.0 * dot, sx = tr1, sy = tr2;
    if (variant == 2) {
      sx = sy = 0.0;
      for (int l = 0; l < d; ++l) {
        const double m1 = M1[(size_t)l * d + l], m2 = M2[(size_t)l * d + l];
        if (!(m1 > 0.0) || !(m2 > 0.0)) { bad = true; break; }
        const double p2 = sqrt(m2 / m1);
        sx += p2 * m1; sy += m2 / p2;
      }
      s += sx + sy;
    }
    if (bad) {
      if (t == 0) status[grp] = 3;
      return;
    }
    const double a = variant == 0 ? 0.0 : a_star(s / d);
    const double b = sqrt(1.0 - 4.0 * a);
    for (int e = t; e < 4 * nn; e += FIT_NT) B1[e] = 0.f;
    __syncthreads();
    if (t < d) {
      const double psi = variant == 2 ? sqrt(sqrt(M2[(size_t)t * d + t] / M1[(size_t)t * d + t])) : 1.0;
      A[t] = (float)a;
      B1[(size_t)t * d + t] = (float)(b * psi);
      B2[(size_t)t * d + t] = (float)(b / psi);
      C1[(size_t)t * d + t] = (float)(-0.5 * psi * psi);
      C2[(size_t)t * d + t] = (float)(-0.5 / (psi * psi));
    }
    if (t == 0) {
      const double lbar = variant == 0 ? nan
                                       : d * log((1.0 - 4.0 * a) / sqrt(1.0 - 8.0 * a)) + (2.0 - 8.0 * a) / (1.0 - 8.0 * a) * s - sx - sy;
      write_header(th, 0.25 * d * log(1.0 - 4.0 * a), lbar, variant == 2 ? 0 : 3, variant);
      status[grp] = 0;
    }
    return;
  }

  const int lane = t & 63, wave = t >> 6;
  if (variant == 4) {                                   // SDERF: one eigendecomposition of N
    decompose_symmetric<RJ>([=](int r, int c) {
      const size_t e = (size_t)r * d + c;
      return M1[e] + mu4[r] * mu5[c] + mu5[r] * mu4[c] + M2[e];
    }, w, n, 0, sh, lds);
    // row scales: sqrt(1 - 4a), with the sign of the eigenvector; the eigenvalues' terms of log D and of the objective
    if (t < d) {
      const int src = sh.ord[0][t];
      const double lam = fmax(sh.nrm[0][src], 0.0), a = a_star(lam);
      A[t] = (float)a;
      sh.red_row[src] = sqrt(1.0 - 4.0 * a) * sh.sgn[0][src];
      sh.nrm[1][t] = 0.25 * log(1.0 - 4.0 * a);
      sh.nrm[2][t] = log(1.0 - 4.0 * a) - 0.5 * log(1.0 - 8.0 * a) + (1.0 + 1.0 / (1.0 - 8.0 * a)) * lam;
    }
    __syncthreads();
    for (int l = wave; l < d; l += FIT_NT / 64) {       // B = (I - 4A)^(1/2) Q3^T: row l is the scaled eigenvector l
      const int src = sh.ord[0][l];
      const double sc = sh.red_row[src];
      for (int c = lane; c < d; c += 64) {
        const float bv = (float)(sc * lds[(size_t)src * (d + 2) + c]);
        const size_t e = (size_t)l * d + c;
        B1[e] = bv;
        B2[e] = bv;
        C1[e] = C2[e] = l == c ? -0.5f : 0.f;
      }
    }
    if (wave == 0) {
      traces();
      double logD = 0.0, lbar = 0.0;
      for (int l = lane; l < d; l += 64) { logD += sh.nrm[1][l]; lbar += sh.nrm[2][l]; }
      logD = sum64(logD);
      lbar = sum64(lbar) - tr1 - tr2;
      if (lane == 0) {
        write_header(th, logD, lbar, 3, variant);
        status[grp] = 0;
      }
    }
    return;
  }

  traces();
  // ADERF: eig M1, eig M2, SVD of Z = L1^(1/2) Q1^T Q2 L2^(1/2)
  double* V1 = w;
  double* V2 = w + nn;
  double* Z = w + 2 * (size_t)nn;      // column-major
  double* b1 = w + 3 * (size_t)nn;     // row-major
  double* b2 = w + 4 * (size_t)nn;
  // (Z, b1 and b2 are not yet in use: scratch)
  for (int m = 0; m < 2; ++m) {
    const double* M = m ? M2 : M1;
    decompose_symmetric<RJ>([=](int r, int c) { return M[(size_t)r * d + c] + (r == c ? ridge : 0.0); }, Z, n, m, sh, lds);
    for (int e = t; e < nn; e += FIT_NT) (m ? V2 : V1)[e] = lds[(size_t)(e / d) * (d + 2) + e % d];
    __syncthreads();
  }
  {
    const double l1max = sh.nrm[0][sh.ord[0][0]], l1min = sh.nrm[0][sh.ord[0][d - 1]];
    const double l2max = sh.nrm[1][sh.ord[1][0]], l2min = sh.nrm[1][sh.ord[1][d - 1]];
    if (!(l1min > 1e-12 * l1max) || !(l2min > 1e-12 * l2max)) {
      if (t == 0) status[grp] = 3;
      return;
    }
  }
  for (int e = t; e < nn; e += FIT_NT) {
    const int c = e / d, r = e % d;                     // Z[r][c] at Z[c * d + r]
    const int s1 = sh.ord[0][r], s2 = sh.ord[1][c];
    double acc = 0.0;
    for (int k = 0; k < d; ++k) acc += V1[(size_t)s1 * d + k] * V2[(size_t)s2 * d + k];
    Z[e] = sqrt(sh.nrm[0][s1]) * sh.sgn[0][s1] * acc * sh.sgn[1][s2] * sqrt(sh.nrm[1][s2]);
  }
  __syncthreads();
  decompose_columns(Z, n, 2, sh, lds);
  if (t == 0) {
    double trs = 0.0;
    for (int l = 0; l < d; ++l) trs += sh.nrm[2][l];
    sh.red[0] = trs;
  }
  __syncthreads();
  const double trs = sh.red[0], sigmin = sh.nrm[2][sh.ord[2][d - 1]];
  if (!(sigmin > 0.0)) {
    if (t == 0) status[grp] = 3;
    return;
  }
  const double mu3 = dot / d;
  const double a = a_star(2.0 * trs / d + 2.0 * mu3);
  const double b = sqrt(1.0 - 4.0 * a);
  // B1 = b S^(1/2) U^T L1^(-1/2) Q1^T,  B2 = b S^(-1/2) U^T L1^(1/2) Q1^T
  for (int e = t; e < nn; e += FIT_NT) {
    const int r = e / d, c = e % d, s3 = sh.ord[2][r];
    const double sig = sh.nrm[2][s3];
    double t1 = 0.0, t2 = 0.0;
    for (int k = 0; k < d; ++k) {
      const int s1 = sh.ord[0][k];
      const double uq = Z[(size_t)s3 * d + k] / sig * sh.sgn[0][s1] * V1[(size_t)s1 * d + c];
      const double rl = sqrt(sh.nrm[0][s1]);
      t1 += uq / rl;
      t2 += uq * rl;
    }
    b1[e] = b * sqrt(sig) * t1;
    b2[e] = b / sqrt(sig) * t2;
    B1[e] = (float)b1[e];
    B2[e] = (float)b2[e];
  }
  __syncthreads();
  for (int e = t; e < nn; e += FIT_NT) {                // C^(k) = -B^(k)T B^(k) / (2 (1 - 4a))
    const int r = e / d, c = e % d;
    double t1 = 0.0, t2 = 0.0;
    for (int k = 0; k < d; ++k) {
      t1 += b1[(size_t)k * d + r] * b1[(size_t)k * d + c];
      t2 += b2[(size_t)k * d + r] * b2[(size_t)k * d + c];
    }
    C1[e] = (float)(-t1 / (2.0 * (1.0 - 4.0 * a)));
    C2[e] = (float)(-t2 / (2.0 * (1.0 - 4.0 * a)));
  }
  if (t < d) A[t] = (float)a;
  if (t == 0) {
    const double lbar = d * (log(1.0 - 4.0 * a) - 0.5 * log(1.0 - 8.0 * a) + 2.0 / (1.0 - 8.0 * a) * (trs / d + mu3) + 2.0 * mu3);
    write_header(th, 0.25 * d * log(1.0 - 4.0 * a), lbar, 0, variant);
    status[grp] = 0;
  }
}

}  // namespace

size_t fit_device_workspace_doubles(int d, int groups) { return (size_t)groups * 5 * d * d; }

int launch_fit_device(int variant, int d, int groups, const double* stats, double ridge, double* ws, float* theta,
                      int* status, size_t theta_floats, hipStream_t st) {
  if (d < 1 || d > FIT_DMAX) return 2;
  // what the tridiagonal form keeps there; more than the matrix of the one-sided iteration
  static_assert(64 * 65 <= tri_lds_doubles(64) && 128 * 129 <= tri_lds_doubles(128), "");
  const size_t lds = tri_lds_doubles(d <= 64 ? 64 : 128) * sizeof(double);
  auto kernel = d <= 64 ? k_fit_device<2> : k_fit_device<4>;
  if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  hipLaunchKernelGGL(kernel, dim3(groups), dim3(FIT_NT), lds, st, variant, d, stats, ridge, ws, theta, status, theta_floats);
  if (hipGetLastError() != hipSuccess) return 5;
  return 0;
}

}  // namespace fs
