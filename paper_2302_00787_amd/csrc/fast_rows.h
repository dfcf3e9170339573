// Row side of the non-causal bf16 kernels (d = dv = 64, M = 256): a workgroup holds ALL 256 features of one (b,h) as
// MFMA operand images in LDS, and every wave takes its own 16 NTT rows through all of them.
//
// What bounds such a kernel is the matrix pipe together with the exponentials: per 16 rows 32 MFMAs of projection and 40
// of the contraction with the state, 16 cycles each, of which about 8 leave room for other vector work (128 exp2 and
// 32 converts per 16 rows).  With the features split over the waves (64 each, the operands in registers) every wave of a
// workgroup needs every row and holds a quarter of every output: rows staged in LDS, two barriers per 64 rows, partial
// tiles through LDS as bf16 and a second pass over them on the matrix pipe.  Here a wave needs nobody: rows come from
// memory as operands, features go from the accumulators of the projection straight into the contraction, outputs are
// complete in fp32, and there is no barrier after the images are in place.  The price is LDS traffic, 88 KB of
// operands per wave and step of 16 NTT rows; four row tiles per wave keep it at about 60 % of the LDS rate beside a full
// matrix pipe, one tile would need 2.4 times the rate.  Measured (non-causal calls, us, features split -> rows split):
// B8 H8 L4096 74.5 -> 64.4, 32 x 16384 117.7 -> 103.3, 1 x 262144 86.8 -> 72.3, 256 x 1000 69.8 -> 55.8, 16 x 300
// 21.4 -> 19.5; one workgroup per sequence: 768 x 197 67.0 -> 61.6, 512 x 1024 98 -> 85.
#pragma once
#include <algorithm>

#include "fast_pc.h"

namespace fs {
namespace rows {

using namespace fast;

// Parts into which each of BH sequences of `units` steps is cut for kernels with one workgroup per CU: as many as fit into one,
// two, three or four passes over the chip, whichever takes the fewest steps (the last pass takes as long as a full one;
// `fixed`: steps' worth of a workgroup's constants, images and results; at most `most` parts).  One workgroup per CU
// rounded up instead leaves a second pass nearly empty: non-causal calls (us) 48 x 1024 44.2 -> 31.0, 24 x 2048 43.8 -> 31.2,
// 12 x 4096 45.9 -> 32.5; gradients 48 x 1024 111.7 -> 69.8, 24 x 2048 103.4 -> 71.8.
inline int parts_per_sequence(int BH, int units, int most, float fixed) {
  int best = 1;
  float least = 1e30f;
  for (int pass = 1; pass <= 4; ++pass) {
    const int n = std::max(1, std::min(most, 256 * pass / BH));
    const float steps = (float)((n * BH + 255) / 256) * ((float)((units + n - 1) / n) + fixed);
    if (steps < least) { least = steps; best = n; }
  }
  return best;
}

// Workgroups go to the eight XCDs in turn, each with an L2 of its own: the workgroup's place in an order in which an
// XCD's workgroups are neighbours, so that those of one sequence fetch its state and constants through one L2.
__device__ __forceinline__ int xcd_contiguous(int id, int n) {
  const int x = id & 7;
  return x * (n >> 3) + min(x, n & 7) + (id >> 3);
}

// Feature f = 32 fb + 16 mt + i, tile ft = 2 fb + mt.
struct __attribute__((aligned(16))) SmemOps {
  uint16_t w[M / 16][KS][64][8];     // W~ as A operand: row = feature 16 ft + c, k = 32 ks + 8 g + e
  uint16_t t[M / 32][NVT][64][8];    // state^T as A operand: row v = 16 vt + c, k <-> feature 32 fb + 16 (e/4) + 4 g + e%4;
                                     // rows 64 .. 79 all hold column 64, so that every lane gets the normaliser of its token
  float bias[M];                     // 2 (bias - largest bias)
};

// ---- global memory -> LDS without registers (buffer_load_dwordx4 ... lds) -----------------------------------------
// Lane l's 16 bytes at base + voff go to LDS address `lds` + 16 l (`lds` wave-uniform); offsets past `bytes` are not
// read.  Written as assembly because the compiler, which cannot tell the images of this file apart, would otherwise
// put a wait for every such load in front of every LDS read.  There is no destination register; the code that reads
// the LDS waits with dma_wait (the compiler's own waits only become more conservative by loads it does not count).
struct DmaBase { u32x4 rsrc; };
__device__ __forceinline__ DmaBase dma_base(const void* base, int bytes) {
  const uint64_t p = (uint64_t)base;
  DmaBase d;
  d.rsrc = u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)p), (uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) & 0xffffu,
                 (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
  return d;
}
__device__ __forceinline__ void dma16(const DmaBase& d, uint32_t voff, const void* lds) {
  const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)lds);
  // (m0 holds the LDS address and nothing else in these files; five wait states between a descriptor written by
  // v_readfirstlane and the load that reads it, which the compiler does not count inside assembly)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(voff), "s"(d.rsrc) : "memory");
}
// Waits until at most N vector memory operations issued since are outstanding.
template <int N>
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// Image of W~ (DMA), for all threads of the workgroup; the caller waits and puts a barrier behind it.
template <int NTH>
__device__ __forceinline__ void load_w_image(SmemOps& sm, const uint16_t* Wbf) {
  constexpr int NP = (M / 16) * KS * 64;
  const DmaBase src = dma_base(Wbf, M * D * 2);
#pragma unroll
  for (int i = 0; i < NP / NTH; ++i) {
    const int p = threadIdx.x + NTH * i, l = p & 63, ks = (p >> 6) % KS, ft = p / (64 * KS);
    dma16(src, 2 * ((16 * ft + (l & 15)) * D + 32 * ks + 8 * (l >> 4)), &sm.w[0][0][0][0] + 8 * (p & ~63));
  }
}
// The same and the biases.
template <int NTH>
__device__ __forceinline__ void load_w_image(SmemOps& sm, const uint16_t* Wbf, const float* bias, float amax) {
  load_w_image<NTH>(sm, Wbf);
  if (threadIdx.x < M) sm.bias[threadIdx.x] = 2.f * (bias[threadIdx.x] - amax);
}

// Image of a state that k_fast_total left in memory: piece (fb, vt, lane), 16 bytes, in the place of the first four of
// the eight numbers it holds.
template <int NTH>
__device__ __forceinline__ void load_t_image(SmemOps& sm, const float* T) {
  constexpr int NP = (M / 32) * NVT * 64;
  const DmaBase src = dma_base(T, M * DVP * 4);
#pragma unroll
  for (int i = 0; i < NP / NTH; ++i) {
    const int p = threadIdx.x + NTH * i, l = p & 63, vt = (p >> 6) % NVT, fb = p / (64 * NVT);
    dma16(src, 4 * (2 * fb * NVT + vt) * 256 + 16 * (vt == NVT - 1 ? l & 48 : l), &sm.t[0][0][0][0] + 8 * (p & ~63));
  }
}

// The same from the registers of four waves that hold 64 features each (fast_state.h).
__device__ __forceinline__ void put_t_image(SmemOps& sm, const f32x4 (&T)[4][NVT], int w, int lane) {
  const int c = lane & 15;
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
    for (int vt = 0; vt < NVT - 1; ++vt) *(bf16x8*)(&sm.t[2 * w + mb][vt][lane][0]) = pack8(T[2 * mb][vt], T[2 * mb + 1][vt]);
    // column 64 (lanes c = 0 of the last tile) to all sixteen rows
    const bf16x8 n = pack8(T[2 * mb][NVT - 1], T[2 * mb + 1][NVT - 1]);
    if (c == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) *(bf16x8*)(&sm.t[2 * w + mb][NVT - 1][lane + i][0]) = n;
    }
  }
}

// 16 NTT rows as MFMA operand (lane <-> row 16 t + c, k = 32 ks + 8 g + e); rows from `nv` on read as zero.  `chunk` and
// `nv` must be wave-uniform.
template <int NTT>
__device__ __forceinline__ void load_row_ops(bf16x8 (&x)[NTT][KS], const uint16_t* chunk, long long sl, int nv, int lane) {
  const int g = lane >> 4, c = lane & 15;
  const __amdgpu_buffer_rsrc_t rs = pc::chunk_rsrc(chunk, 2 * (int)sl, min(nv, 16 * NTT), 2 * D);
#pragma unroll
  for (int t = 0; t < NTT; ++t)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      x[t][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, 2 * ((16 * t + c) * (int)sl + 32 * ks + 8 * g), 0, 0));
}

// The same rows on their way to a wave's own LDS buffer ([row tile][k-step][lane][8]), and from there.
template <int NTT>
__device__ __forceinline__ void dma_rows(uint16_t* buf, const uint16_t* chunk, long long sl, int nv, int lane) {
  const int g = lane >> 4, c = lane & 15, rows = min(nv, 16 * NTT);
  const DmaBase src = dma_base(chunk, rows > 0 ? (rows - 1) * 2 * (int)sl + 2 * D : 0);
#pragma unroll
  for (int t = 0; t < NTT; ++t)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dma16(src, 2 * ((16 * t + c) * (int)sl + 32 * ks + 8 * g), buf + 512 * (KS * t + ks));
}
template <int NTT>
__device__ __forceinline__ void read_rows(bf16x8 (&x)[NTT][KS], const uint16_t* buf, int lane) {
#pragma unroll
  for (int t = 0; t < NTT; ++t)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[t][ks] = *(const bf16x8*)(buf + 512 * (KS * t + ks) + 8 * lane);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the buffer may be filled again
}

// Exponents of the 32 features of block fb: W~ x + bias (BIAS), or + what is added to the exponents of the lane's row.
template <int NTT, bool BIAS>
__device__ __forceinline__ void project(f32x4 (&acc)[2][NTT], const SmemOps& sm, int fb, const bf16x8 (&x)[NTT][KS], const f32x4* add,
                                        int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const bf16x8 w0 = *(const bf16x8*)(&sm.w[2 * fb + mt][0][lane][0]), w1 = *(const bf16x8*)(&sm.w[2 * fb + mt][1][lane][0]);
    f32x4 b;
    if (BIAS) b = *(const f32x4*)(&sm.bias[32 * fb + 16 * mt + 4 * g]);
#pragma unroll
    for (int t = 0; t < NTT; ++t) acc[mt][t] = mfma(w0, x[t][0], BIAS ? b : add[t]);
#pragma unroll
    for (int t = 0; t < NTT; ++t) acc[mt][t] = mfma(w1, x[t][1], acc[mt][t]);
  }
}

// y[vt][t] = (state^T x features^T): rows = columns 16 vt + 4 g + r of the state, lane <-> row 16 t + c of the chunk;
// y[NVT - 1][t][0] is the row's normaliser in every lane.  SHIFT: add[t] is added to the exponents of the lane's row.
// KEEP: the features stay with the caller, keep[fb][t] (k <-> feature 32 fb + 16 (e/4) + 4 g + e%4 of the lane's row).
// A wave issues in order, so the exponentials of block fb + 1 are interleaved with the contraction of block fb, one
// matrix instruction to three of the others (left to the compiler they come in runs: encoder call 64.4 against 63.4 us).
template <int NTT, bool SHIFT, bool KEEP = false>
__device__ __forceinline__ void contract_rows(f32x4 (&y)[NVT][NTT], const SmemOps& sm, const bf16x8 (&x)[NTT][KS],
                                              const float (&add)[NTT], int lane, bf16x8 (*keep)[NTT] = nullptr) {
  f32x4 acc[2][NTT];
  bf16x8 p[NTT];
  auto features = [&](bf16x8 (&f)[NTT]) {
#pragma unroll
    for (int t = 0; t < NTT; ++t)
      f[t] = SHIFT ? pack8(exp2v(acc[0][t] + add[t]), exp2v(acc[1][t] + add[t])) : pack8(exp2v(acc[0][t]), exp2v(acc[1][t]));
  };
  project<NTT, true>(acc, sm, 0, x, nullptr, lane);
  features(p);
  project<NTT, true>(acc, sm, 1, x, nullptr, lane);
#pragma unroll
  for (int vt = 0; vt < NVT; ++vt)
#pragma unroll
    for (int t = 0; t < NTT; ++t) y[vt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int fb = 0; fb < M / 32; ++fb) {
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 pn[NTT];
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) {
      const bf16x8 s = *(const bf16x8*)(&sm.t[fb][vt][lane][0]);
#pragma unroll
      for (int t = 0; t < NTT; ++t) y[vt][t] = mfma(s, p[t], y[vt][t]);
    }
    if (fb + 1 < M / 32) {
      features(pn);
#pragma unroll
      for (int i = 0; i < NVT * NTT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (fb + 2 < M / 32) project<NTT, true>(acc, sm, fb + 2, x, nullptr, lane);
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      if (KEEP) keep[fb][t] = p[t];
      p[t] = pn[t];
    }
  }
}

// The largest Cauchy-Schwarz bound at which a query row may go without its shift (a factor per row cancels in the
// normalisation), given the largest magnitude `tmax` in the state that its features meet: a sum over the 256 features
// is at most 2^(bound + 8) tmax, kept under 2^125 here, so that no row which is finite with its shift overflows without.
// 2^80 at most, as far as a feature itself is concerned.  (The state of ordinary data reaches 2^20: every row up to
// 2^80.  All rows shifted instead: B8 H8 L4096 59.6 -> 62.4 us, 64 x 12 x 197 59.5 -> 60.3.)
__device__ __forceinline__ float noshift_bound(float tmax) { return fminf(80.f, 117.f - __builtin_amdgcn_logf(tmax)); }

// The largest magnitude in a state that k_fast_total left in memory: one per wave of that kernel, in the unused half of
// its piece.
__device__ __forceinline__ float state_max(const float* T) {
  constexpr int NPART = (M / 32) * NVT;
  const int i = min((int)(threadIdx.x & 63), NPART - 1);
  return wave_max(T[(size_t)((2 * (i / NVT) + 1) * NVT + i % NVT) * 256]);
}
static_assert((M / 32) * NVT <= 64, "one per lane");

// The queries' per-row shifts: zero for all rows of the wave (and `false` returned) when no row's bound exceeds
// `noshift`, else -row_shift of the lane's row.
template <int NTT>
__device__ __forceinline__ bool query_shifts(float (&add)[NTT], const bf16x8 (&x)[NTT][KS], float wmax, float noshift, int nv, int lane) {
  const int g = lane >> 4, c = lane & 15;
  float n2[NTT];
  bool large = false;
#pragma unroll
  for (int t = 0; t < NTT; ++t) {
    n2[t] = tile_row_norms(x[t][0], x[t][1], lane);
    add[t] = 0.f;
    large |= g == (c >> 2) && 16 * t + c < nv && !(wmax * __builtin_amdgcn_sqrtf(n2[t]) <= noshift);
  }
  if (__ballot(large) == 0) return false;
#pragma unroll
  for (int t = 0; t < NTT; ++t) add[t] = -row_shift(__shfl(n2[t], 16 * (c >> 2) + c), wmax);
  return true;
}

// Rows [row_beg, row_end) of the queries of one (b,h), taken by NWV waves in turn: Y = (P T) normalised by its last column.
// Rows whose bounds are all at most `noshift` go without their shifts.
// `buf`: the wave's LDS buffer of 16 NTT rows when the rows of the next step travel during this one's work (PREF; the
// caller has issued dma_rows for the first step), else unused; `first`: else the operands of the first step, or nullptr.  Returns
// the number of rows this wave finished with a zero normaliser.
template <int NTT, int NWV, bool PREF>
__device__ __forceinline__ int apply_rows(const FastArgs& a, const SmemOps& sm, uint16_t* buf, const bf16x8 (*first)[KS], float wmax,
                                          float noshift, int bh, int row_beg, int row_end) {
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* Qb = (const uint16_t*)a.Q.ptr + b * a.Q.sb + h * a.Q.sh;
  const long long ybase = b * a.Y.sb + h * a.Y.sh;
  constexpr int RT = 16 * NTT;
  int nzero = 0;
  for (int row0 = row_beg + RT * w; row0 < row_end; row0 += RT * NWV) {
    bf16x8 x[NTT][KS];
    if (PREF) {
      // the rows were requested ahead of the 4 NTT stores of the step before
      if (row0 == row_beg + RT * w) dma_wait<0>();
      else dma_wait<4 * NTT>();
      read_rows(x, buf, lane);
      const int next = row0 + RT * NWV;
      if (next < row_end) dma_rows<NTT>(buf, Qb + (long long)next * a.Q.sl, a.Q.sl, row_end - next, lane);
    } else if (first != nullptr && row0 == row_beg + RT * w) {
#pragma unroll
      for (int t = 0; t < NTT; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x[t][ks] = first[t][ks];
    } else {
      load_row_ops(x, Qb + (long long)row0 * a.Q.sl, a.Q.sl, row_end - row0, lane);
    }
    const int nv = row_end - row0;
    f32x4 y[NVT][NTT];
    float add[NTT];
    if (query_shifts(add, x, wmax, noshift, nv, lane)) contract_rows<NTT, true>(y, sm, x, add, lane);
    else contract_rows<NTT, false>(y, sm, x, add, lane);
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      const float den = y[NVT - 1][t][0];
      const float inv = den > 0.f ? __builtin_amdgcn_rcpf(den) : 0.f;
      nzero += count_zero_tokens((unsigned)__ballot(!(den > 0.f)) & 0xffffu, t, nv);
#pragma unroll
      for (int vt = 0; vt < 4; ++vt) y[vt][t] *= inv;
    }
    if (a.Y.dtype == 1) {
      const __amdgpu_buffer_rsrc_t ry = pc::chunk_rsrc((const uint16_t*)a.Y.ptr + ybase + (long long)row0 * a.Y.sl, 2 * (int)a.Y.sl,
                                                       min(nv, RT), 2 * D);
#pragma unroll
      for (int t = 0; t < NTT; ++t)
#pragma unroll
        for (int vt = 0; vt < 4; ++vt)
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, __builtin_convertvector(y[vt][t], bf16x4)), ry,
                                                2 * ((16 * t + c) * (int)a.Y.sl + 16 * vt + 4 * g), 0, 0);
    } else {
      const __amdgpu_buffer_rsrc_t ry = pc::chunk_rsrc((const float*)a.Y.ptr + ybase + (long long)row0 * a.Y.sl, 4 * (int)a.Y.sl,
                                                       min(nv, RT), 4 * D);
#pragma unroll
      for (int t = 0; t < NTT; ++t)
#pragma unroll
        for (int vt = 0; vt < 4; ++vt)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y[vt][t]), ry,
                                                 4 * ((16 * t + c) * (int)a.Y.sl + 16 * vt + 4 * g), 0, 0);
    }
  }
  return nzero;
}

}  // namespace rows
}  // namespace fs
