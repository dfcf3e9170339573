// Key-side state pass of the bf16 path (d = dv = 64, M = 256), shared by the forward kernels (kernels_bf16.hip) and
// the backward kernel that takes a whole sequence per workgroup (kernels_bf16_bwd.hip).
#pragma once
#include "fast_pc.h"

namespace fs {

using namespace fast;

// ---------------------------------------------------------------------------------------------------
// Key-side state of a range of rows: T = sum_j S'_j [V_j 1]^T / 2^dk, S' = features without the bias (Section 2.1,
// S^T C with C = [V 1]), for a workgroup of 256 threads (two per CU).
//
// Four waves of 64 features; per 64-token chunk every wave builds its feature tiles feature-major (A = token rows,
// B = W~; the per-token part of the exponent is the accumulator's initial value, read from LDS as a 16-byte vector)
// and adds S^T [V 1] to its state slice in registers.  Key and value rows stay row-major in LDS as they are in
// memory (global -> registers -> LDS, no arithmetic on the way): the value operand is a transposing LDS read, the
// squared row norms (row term -|y|^2/2 and the bound for the running shift) are the diagonal of Y Y^T on the MFMA
// pipe, computed by wave w for token tile w ONE CHUNK AHEAD, so that a single barrier per chunk orders everything:
// iteration c computes the constants of chunk c+1 (its key rows arrived in iteration c-1: three key buffers),
// contracts chunk c, and stores the value rows of chunk c+1 and the key rows of chunk c+2.  The largest bound of a
// chunk is gathered with an LDS float maximum, so the chunk starts with one broadcast read instead of a reduction.
// A wave executes in order, so every LDS read of a chunk is issued at the top of the iteration, ahead of the MFMA
// and exp2 streams that consume them.  What bounds the loop is the sum of both streams: 74 MFMAs of 16 cycles and about
// 1050 cycles of vector work per wave and chunk, of which little overlaps between the two waves of a SIMD (4750 cycles
// per chunk for both, measured).  B8 H8 L4096: state and reduction 40 -> 29 us with the interleaving, the loads ahead of
// the constants and one state per two groups of waves (k_fast_state2).
// ---------------------------------------------------------------------------------------------------
struct SmemState {
  uint16_t k[3][TC][LDR];                                   // key rows of three consecutive chunks
  __attribute__((aligned(16))) uint16_t v[2][TC][LDV];      // value rows (columns 64.. are constant: 1, 0, ..)
  __attribute__((aligned(16))) float kadd[2][TC];           // per key token: row term (-inf past the end)
  float kmax[4];                                            // largest row_shift + row term of a chunk, at chunk index % 3
};

// The state of the key rows [row_beg, row_end) of one (b,h), left in the registers of the workgroup's four waves
// (wave w: features 64w .. 64w+63 x 80 columns) on the shift dk.  Ends behind a barrier: the caller may reuse the LDS.
// STATE_BOUND: nothing but dk, the largest bound of the rows (the shift such a state would have): no projections, no
// values, T untouched.
// STATE_QUERIES: the query-side twin R = sum_i P_i G1_i^T of the backward pass: Q's rows with their own shifts and the
// biases, a.V = the G1 rows of 80 numbers; dk = 0.
// A workgroup of 512 threads calls it with two row ranges, one per group of four waves, each group with an LDS struct of
// its own and both with the same `niter`, the number of chunks of the longer range (the barriers are the workgroup's).
enum { STATE_KEYS, STATE_BOUND, STATE_QUERIES };
template <int MODE = STATE_KEYS>
__device__ __forceinline__ void state_rows(const FastArgs& a, SmemState& sm, int bh, int row_beg, int row_end, int niter,
                                           f32x4 (&T)[4][NVT], float& dk) {
  constexpr bool BOUND_ONLY = MODE == STATE_BOUND, QUERIES = MODE == STATE_QUERIES;
  constexpr int side = QUERIES ? 0 : 1;
  const TensorDev& X = QUERIES ? a.Q : a.K;
  const int b = bh / a.H, h = bh % a.H;
  const int tid = threadIdx.x & (NT - 1), lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const int pg = group_of(a.pgroups, b, h, a.H);
  const float* th = a.theta + (size_t)group_of(a.groups, b, h, a.H) * (FS_THETA_HEADER_ + (size_t)D + 4 * (size_t)D * D);
  const uint16_t* Kb = (const uint16_t*)X.ptr + b * X.sb + h * X.sh + (long long)row_beg * X.sl;
  const uint16_t* Vb = (const uint16_t*)a.V.ptr + b * a.V.sb + h * a.V.sh + (long long)row_beg * a.V.sl;
  const float* rkb = a.rk + (size_t)bh * a.L + row_beg;
  const int nrows = row_end - row_beg;

  // staging: thread -> rows tid/8 and tid/8 + 32 of a chunk, bytes 16 (tid%8); rows past the end read as zero
  // (a fresh descriptor per chunk: uniform base = the chunk's first row, 32-bit offsets and extent inside the chunk)
  const int srow = tid >> 3, spc = tid & 7;
  u32x4 kr[2], vr[QUERIES ? 3 : 2];
  auto load_k = [&](int r0) {
    const __amdgpu_buffer_rsrc_t rk_ = pc::chunk_rsrc(Kb + (long long)r0 * X.sl, 2 * (int)X.sl, min(nrows - r0, TC), 2 * D);
#pragma unroll
    for (int i = 0; i < 2; ++i) kr[i] = __builtin_amdgcn_raw_buffer_load_b128(rk_, 2 * ((srow + 32 * i) * (int)X.sl + spc * 8), 0, 0);
  };
  auto load_v = [&](int r0) {
    if (BOUND_ONLY) return;
    const __amdgpu_buffer_rsrc_t rv_ = pc::chunk_rsrc(Vb + (long long)r0 * a.V.sl, 2 * (int)a.V.sl, min(nrows - r0, TC), QUERIES ? 2 * DVP : 2 * D);
    if (QUERIES) {             // G1 rows: 160 bytes one after the other, a chunk is 640 pieces in a row
#pragma unroll
      for (int i = 0; i < (QUERIES ? 3 : 2); ++i) vr[i] = __builtin_amdgcn_raw_buffer_load_b128(rv_, 16 * (tid + NT * i), 0, 0);
      return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) vr[i] = __builtin_amdgcn_raw_buffer_load_b128(rv_, 2 * ((srow + 32 * i) * (int)a.V.sl + spc * 8), 0, 0);
  };
  auto store_k = [&](int kb) {
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4*)(&sm.k[kb][srow + 32 * i][spc * 8]) = kr[i];
  };
  auto store_v = [&](int vb) {
    if (BOUND_ONLY) return;
    if (QUERIES) {
#pragma unroll
      for (int i = 0; i < (QUERIES ? 3 : 2); ++i)
        if (tid + NT * i < TC * (LDV / 8)) *(u32x4*)(&sm.v[vb][0][0] + 8 * (tid + NT * i)) = vr[i];
      return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4*)(&sm.v[vb][srow + 32 * i][spc * 8]) = vr[i];
  };
  // the first two chunks' key rows and the first chunk's value rows are requested ahead of everything else: the constants
  // arrive meanwhile (one memory latency at the start of the kernel instead of three in a row)
  load_k(0);
  load_v(0);
  const u32x4 k0[2] = {kr[0], kr[1]};
  load_k(TC);
  WSlice wk;
  if (!BOUND_ONLY) {
    load_wslice(wk, a.Wbf + ((size_t)pg * 2 + side) * M * D, w);
    if (!QUERIES) init_value_pad(sm.v[0], 2 * TC, NT, tid);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) T[mt][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float bcol[4] = {0.f, 0.f, 0.f, 0.f};           // (queries) 2 (bias - largest bias) of feature 64 w + 16 mt + c
  if (QUERIES) {
    const float* bias = a.bias + ((size_t)pg * 2) * M;
    const float amax = max256(bias);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) bcol[mt] = 2.f * (bias[64 * w + 16 * mt + c] - amax);
  }
  const float wmax = max256(a.wnorm + ((size_t)pg * 2 + side) * M);
  const bool isoC = QUERIES || (((int)th[2]) & 1);
  if (tid < 3) sm.kmax[tid] = -INFINITY;
  dk = QUERIES ? 0.f : -INFINITY;

  // Per-token constants of token tile w of a chunk (first row r0 of the slot) from the squared norms n2 of its rows
  // (valid in the lanes (g, c) = (c / 4, c)): row terms to kadd[cb], the largest bound into kmax[mb].
  // (`rkv`: the token's row term from memory, for parameter sets with a dense C2: requested by the caller ahead of time)
  auto row_term_of = [&](int r0) {
    float v = 0.f;
    if (!isoC && g == (c >> 2) && r0 + 16 * w + c < nrows) v = rkb[r0 + 16 * w + c];
    return v;
  };
  auto constants = [&](float n2, float rkv, int cb, int mb, int r0) {
    if (g == (c >> 2)) {
      const int t = 16 * w + c;
      const bool valid = r0 + t < nrows;
      if (QUERIES) {
        sm.kadd[cb][t] = valid ? -row_shift(n2, wmax) : -INFINITY;
        return;
      }
      float rt = -0.5f * kLog2e * a.scale * a.scale * n2;
      if (!isoC) rt = valid ? rkv : 0.f;
      // rows past the end get -inf: their features are exactly zero whatever the key shift is
      sm.kadd[cb][t] = valid ? rt : -INFINITY;
      if (valid) lds_fmax(&sm.kmax[mb], row_shift(n2, wmax) + rt);
    }
  };
  auto tile_op = [&](int kb, int jt, int ks) { return *(const bf16x8*)(&sm.k[kb][16 * jt + c][32 * ks + 8 * g]); };

  store_k(1);
  kr[0] = k0[0]; kr[1] = k0[1];
  store_k(0);
  store_v(0);
  __syncthreads();
  constants(tile_row_norms(tile_op(0, w, 0), tile_op(0, w, 1), lane), row_term_of(0), 0, 0, 0);
  load_v(TC);
  load_k(2 * TC);
  __syncthreads();

  // The second half of a chunk's state update is left for the next iteration, where its matrix instructions cover the
  // LDS reads behind the barrier; the exponentials of a token pair are interleaved with the matrix instructions beside
  // them (a wave issues in order: left to the compiler they came in runs of 32 and more).
  // (Ahead of the first chunk a flag says that there is none, opaque to the compiler, which would peel that chunk off, with registers
  // for both; where registers are short, with the queries' three pieces of a value row, the operands are zero instead: k_bwd_rstate
  // 50.7 us on 32 x 16384 tokens, 58.7 with the flag.)
  const bf16x8 zero8 = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  bf16x8 st1[4] = {zero8, zero8, zero8, zero8}, vop1[NVT] = {zero8, zero8, zero8, zero8, zero8};
  int pending = QUERIES;
  auto update1 = [&]() {
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) T[mt][vt] = mfma(st1[mt], vop1[vt], T[mt][vt]);
  };
  int kcur = 0, knext = 1, kfree = 2;
  for (int r0 = 0, ci = 0; ci < niter; r0 += TC, ++ci) {
    const int cb = ci & 1;
    if constexpr (BOUND_ONLY) {
      // the constants of the next chunk and the running maximum only
      const float dnew = sm.kmax[kcur];
      const bf16x8 xn0 = tile_op(knext, w, 0), xn1 = tile_op(knext, w, 1);
      const float rk_next = row_term_of(r0 + TC);
      dk = fmaxf(dk, dnew);
      const float n2 = tile_row_norms(xn0, xn1, lane);
      if (tid == 0) sm.kmax[kfree] = -INFINITY;
      constants(n2, rk_next, cb ^ 1, knext, r0 + TC);
      store_k(kfree);
      load_k(r0 + 3 * TC);
      __syncthreads();
      const int t = kcur; kcur = knext; knext = kfree; kfree = t;
      continue;
    }
    float n2 = 0.f;
    const float rk_next = row_term_of(r0 + TC);      // (dense C2) requested here, used at the end of the iteration
    if (r0 < nrows) {          // (always, but for the last chunk of the shorter of two ranges)
      // ---- every LDS read of the projections, up front
      const float dnew = sm.kmax[kcur];
      bf16x8 x[4][KS];
      f32x4 kadd4[4];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        kadd4[jt] = *(const f32x4*)(&sm.kadd[cb][16 * jt + 4 * g]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x[jt][ks] = tile_op(kcur, jt, ks);
      }
      const bf16x8 xn0 = tile_op(knext, w, 0), xn1 = tile_op(knext, w, 1);     // token tile w of the next chunk
      __builtin_amdgcn_sched_barrier(0);
      if (!QUERIES) asm volatile("" : "+s"(pending));
      if (pending) update1();
      pending = 1;
      __builtin_amdgcn_sched_barrier(0);
      // ---- running key shift: the state is rebased when the chunk's largest bound exceeds the current shift
      if (!QUERIES && dnew > dk) {
        const float f = fast_exp2(dk - dnew);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int vt = 0; vt < NVT; ++vt) T[mt][vt] *= f;
        dk = dnew;
      }
      f32x4 acc[2][4][2];            // [pair][feature tile][tile of the pair]
      auto project = [&](int jp) {
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            acc[jp][mt][jj] = mfma(x[2 * jp + jj][0], wk.w[mt][0], kadd4[2 * jp + jj] + (QUERIES ? bcol[mt] : -dk));
#pragma unroll
            for (int ks = 1; ks < KS; ++ks) acc[jp][mt][jj] = mfma(x[2 * jp + jj][ks], wk.w[mt][ks], acc[jp][mt][jj]);
          }
      };
      bf16x8 st0[4], vop0[NVT];
      project(0);
      n2 = tile_row_norms(xn0, xn1, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) vop0[vt] = load_vop_tr(sm.v[cb], 0, vt, lane);
      project(1);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) st0[mt] = pack8(exp2v(acc[0][mt][0]), exp2v(acc[0][mt][1]));
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) vop1[vt] = load_vop_tr(sm.v[cb], 1, vt, lane);
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) T[mt][vt] = mfma(st0[mt], vop0[vt], T[mt][vt]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) st1[mt] = pack8(exp2v(acc[1][mt][0]), exp2v(acc[1][mt][1]));
#pragma unroll
      for (int i = 0; i < 20; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 3, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tid == 0) sm.kmax[kfree] = -INFINITY;    // last read in the previous iteration, gathered again in the next one
    constants(n2, rk_next, cb ^ 1, knext, r0 + TC);
    store_v(cb ^ 1);
    store_k(kfree);
    load_v(r0 + 2 * TC);
    load_k(r0 + 3 * TC);
    __syncthreads();
    const int t = kcur; kcur = knext; knext = kfree; kfree = t;
  }
  if (!QUERIES) asm volatile("" : "+s"(pending));
  if (!BOUND_ONLY && pending) update1();
}

// The state of the rows [row_beg, row_end) by two groups of four waves, whose states meet in LDS: one state per CU and launch goes
// to memory instead of two, and one is read by the reduction behind it (B8 H8 L4096: 21 MB each way instead of 42, which at
// 5 TB/s is what the two kernels spent a third of their time on).  Each group takes half of the chunks; group 0 finishes
// feature tiles 0 and 1 of every wave, group 1 tiles 2 and 3.  For 512 threads and kState2Lds bytes of LDS.
__device__ __forceinline__ int chunks_of(int rows) { return (rows + TC - 1) / TC; }

union SmemState2 {
  SmemState s[2];
  f32x4 x[2][NW][2][NVT][64];      // [sender][wave of the group][its two tiles][value tile][lane]
};
constexpr size_t kState2Lds = sizeof(SmemState2) + 16;
static_assert(kState2Lds <= 160 * 1024, "one workgroup per CU");

template <int MODE>
__device__ __forceinline__ void state_two_groups(const FastArgs& a, unsigned char* smem_raw, int bh, int row_beg, int row_end,
                                                 bool image, float* out, float* shift_out) {
  SmemState2& sm = *reinterpret_cast<SmemState2*>(smem_raw);
  float* dks = (float*)(smem_raw + sizeof(SmemState2));
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
  const int half = (chunks_of(row_end - row_beg) + 1) / 2, mid = min(row_end, row_beg + half * TC);
  f32x4 T[4][NVT];
  float dk;
  state_rows<MODE>(a, sm.s[grp], bh, grp ? mid : row_beg, grp ? row_end : mid, half, T, dk);
  // (state_rows ends behind a barrier: its LDS is free)
  if ((threadIdx.x & (NT - 1)) == 0) dks[grp] = dk;
  auto put = [&](int t0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) sm.x[grp][w][i][vt][lane] = T[t0 + i][vt];
  };
  if (grp) put(0);
  else put(2);
  __syncthreads();
  const float dm = fmaxf(dks[0], dks[1]), other = dks[grp ^ 1];
  // (a group without rows has a zero state and a shift of -inf)
  const float f = dk == dm ? 1.f : fast_exp2(dk - dm), fo = other == dm ? 1.f : fast_exp2(other - dm);
  auto finish = [&](int t0) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) {
        const f32x4 v = T[t0 + i][vt] * f + sm.x[grp ^ 1][w][i][vt][lane] * fo;
        if (image) {
          *(f32x4*)(out + (size_t)((w * 4 + t0 + i) * NVT + vt) * 256 + 4 * lane) = v;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) out[(size_t)(64 * w + 16 * (t0 + i) + 4 * (lane >> 4) + r) * DVP + 16 * vt + (lane & 15)] = v[r];
        }
      }
  };
  if (grp) finish(2);
  else finish(0);
  if (threadIdx.x == 0) *shift_out = dm;
}

}  // namespace fs
