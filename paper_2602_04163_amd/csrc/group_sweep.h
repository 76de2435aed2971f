// Steps 3-4 of the pass: the group / column sweep of BPDQ with lazy block updates
// (paper Sec. 3.2, 3.3; Eq. 3-9; App. B).
//
// Mapping.  Every formula of the method is row-wise; the only sequential axis is the column
// index inside a group.  One row of a group lives in 16 lanes (one DPP row): column j sits in
// lane j % 16, register slot j / 16, so the live columns stay spread over all 16 lanes while
// the sweep advances.  A wavefront carries 4 rows, a work-group 16.  The local factor
// U_loc (g x g) is staged once per work-group in LDS, permuted so that a lane's slots are
// contiguous, with the diagonal and lower part zeroed (no masks in the inner loop).
//
// What is computed.  For a row with group-start working weights t and bit rows b_i, all the
// quantities the method needs are right-solves with U_loc:
//     tau = t U_loc^-1,   P_0 = 1 U_loc^-1,   P_i = b_i U_loc^-1.
// The same forward recurrence as the error propagation of Eq. 3-4 gives them
// (x_l = v_l / U_ll;  v_{l+1:} -= x_l U_{l,l+1:}).  The sweep is that recurrence on the working weights alone, one
// column per step (column_step); the plane solves need the finished codes and no decision needs them, so they
// follow it by blocks of 16 columns (solve_planes; a single plane of a large group advances with it).  Then
//   * the fit of Eq. 6 is the (k+1) x (k+1) system G c = r with G_ab = P_a.P_b, r_a = P_a.tau
//     (since U_loc^-T B_r = [P_0 .. P_k]^T), accumulated and solved in fp64;
//   * the corrected propagation coordinates of Eq. 9 are E' = tau - sum_a c_a P_a
//     (App. B.3: E' U_loc = T - What_new), so What_old / Delta E are never materialised;
//   * the score of an iterate is ||E'||^2.
// Decisions (8-bit RTN code, nearest level) are taken in fp32 in a fixed operation order.
#pragma once
#include <type_traits>
#include <utility>

#include "mfma_kmajor.h"

namespace bpdq {

constexpr int kRowsPerWG = 16;
constexpr int kSweepThreads = 256;
// Two work-groups per CU (a sweeping one and one in the tail role) need the kernel within 256
// registers per lane; the state of a g = 256 group does not fit that.
template <int G>
constexpr int kSweepWavesPerSimd = (G <= 128) ? 2 : 1;
// The lazy block update rides along with the sweep (extra work-groups of the group launch) only
// where a sweeping and an updating work-group fit on one CU; at g = 256 it is a launch of its own.
template <int G>
constexpr bool kTailInSweep = (G <= 128);

// ------------------------------------------------------------------ lane helpers -----------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  // every lane reads a valid lane of its own row, so the "old" operand is never used: passing x
  // itself spares the compiler a zero-initialisation per DPP move
  const int xi = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(xi, xi, CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  // bound_ctrl: without it the compiler writes a zero into each half first
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Butterfly over the 16 lanes of a row: xor 1, xor 2 (quad permutes), then half-row mirror and
// row mirror, which act as xor 4 / xor 8 once quads are uniform.  Every lane ends with the same
// bits (each stage adds the same two operands in both partners).
template <typename OP>
__device__ __forceinline__ float row_reduce_f(float v, OP op) {
  v = op(v, dpp_f<0xB1>(v));
  v = op(v, dpp_f<0x4E>(v));
  v = op(v, dpp_f<0x141>(v));
  v = op(v, dpp_f<0x140>(v));
  return v;
}
__device__ __forceinline__ double row_sum_d(double v) {
  v += dpp_d<0xB1>(v);
  v += dpp_d<0x4E>(v);
  v += dpp_d<0x141>(v);
  v += dpp_d<0x140>(v);
  return v;
}

// ------------------------------------------------------------------ per-row state ----------
typedef float f4 __attribute__((ext_vector_type(4)));

template <int K, int G>
struct RowState {
  static constexpr int CPL = G / 16;
  float t[CPL];       // group-start working weights (frozen for the group)
  float tau[CPL];     // t U_loc^-1
  float p0[CPL];      // 1 U_loc^-1 (the same for every row)
  float inv[CPL];     // 1 / U_ll of my columns
  float wg[CPL];      // working copy during a sweep; a finished column keeps the weight that it was decided on
  f4 P[CPL];          // component i: running right-hand side of plane i, then P_i = b_i U_loc^-1 (solve_planes)
  int code[CPL];      // plane bits of my columns, bit (i-1) = B_i
};

// LDS layout of the local factor.  Row l only ever meets columns j > l, and column j lives in
// slot j / 16 of lane j % 16, so row l keeps just the S = CPL - l / 16 slots m >= M = l / 16 of
// every lane.  The slots are cut into chunks of 4, then 2, then 1 (three left over are read as a
// chunk of 4 with a zero: one read instead of two); a chunk of width w that starts at slot M + o holds
//   sU[row_offset(l) + 16 o + lane * w + e] = -U[l][16 (M + o + e) + lane]    (0 where j <= l)
// so one ds_read_b128 / b64 / b32 of the 16 lanes of a row covers 16 w contiguous floats (no bank
// conflicts) at an immediate offset, and the lower part reads as zero (no masks in the inner loop).
// 38 KB at g = 128, 136 KB at g = 256.
//
// The image of every group is laid out once per layer in the workspace, by extra work-groups of the
// launch that copies W (pack_factor), together with 1 / U_ll and P_0 = 1 U_loc^-1, which are the
// same for all rows: a group launch streams the image into LDS with LDS-DMA while it gathers its
// target.  Fetching and rearranging U_loc in every work-group had cost 12 k of a launch's 186 k cycles
// (k = 2, g = 128, 5 iterations; 154 k without them) and the P_0 recurrence a quarter of the initial pass.
template <int G>
struct SuLayout {
  static constexpr int CPL = G / 16;
  // widest chunk: 4 floats (ds_read_b128); 2 at g = 256, where the wider reads push the
  // fully unrolled sweep over the register file
  static constexpr int kMaxVec = (G >= 256) ? 2 : 4;
  __host__ __device__ static constexpr int live(int M) {          // slots kept per lane, with the pad
    return CPL - M + ((kMaxVec == 4 && (CPL - M) % 4 == 3) ? 1 : 0);
  }
  __host__ __device__ static constexpr int row_offset(int l) {
    int off = 0;
    for (int M = 0; M < l / 16; ++M) off += 256 * live(M);
    return off + 16 * (l % 16) * live(l / 16);
  }
  __host__ __device__ static constexpr int floats() { return row_offset(G); }
  // a group's record in the workspace: image | 1 / U_ll [G] | P_0 [G], whole KB
  __host__ __device__ static constexpr int record_floats() { return (floats() + 2 * G + 255) / 256 * 256; }
  // reads of a row that keeps the slots m >= M
  __host__ __device__ static constexpr int chunks(int M) { return (CPL - M + kMaxVec - 1) / kMaxVec; }
  // width of the chunk that holds live slot o (0-based among the live slots) of a row with S
  // live slots, and the live slot that chunk starts at
  __host__ __device__ static constexpr int chunk_width(int S, int o) {
    const int g0 = o / kMaxVec * kMaxVec, r = S - g0;
    if (r >= kMaxVec || r == 3) return kMaxVec;     // a full chunk, or three and a pad
    return r;                                       // 2 or 1
  }
  __host__ __device__ static constexpr int chunk_start(int, int o) { return o / kMaxVec * kMaxVec; }
  // float index (relative to the row) of live slot o for lane `lane`; o = S: the pad after three left over
  __host__ __device__ static constexpr int slot_index(int S, int o, int lane) {
    const int w = chunk_width(S, o), c0 = chunk_start(S, o);
    return 16 * c0 + lane * w + (o - c0);
  }
};

// the slots [FROM, CPL) of one row that keeps [M, CPL) for this lane; p = sU + row_offset(l)
template <int G, int M, int FROM = M>
__device__ __forceinline__ void load_u_row(const float* __restrict__ p, int lane16,
                                           float (&u)[G / 16]) {
  using Lay = SuLayout<G>;
  constexpr int CPL = G / 16, S = CPL - M;
  typedef float vec4 __attribute__((ext_vector_type(4)));
  typedef float vec2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int o = 0; o < S; ++o) {
    if (Lay::chunk_start(S, o) != o || o + Lay::chunk_width(S, o) <= FROM - M) continue;
    const int w = Lay::chunk_width(S, o);
    if (w == 4 && o + 2 <= FROM - M) {             // the upper half of a chunk
      const vec2 v = *reinterpret_cast<const vec2*>(p + 16 * o + lane16 * 4 + 2);
#pragma unroll
      for (int e = 0; e < 2; ++e)
        if (o + 2 + e < S) u[M + o + 2 + e] = v[e];
    } else if (w == 4) {
      const vec4 v = *reinterpret_cast<const vec4*>(p + 16 * o + lane16 * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (o + e < S) u[M + o + e] = v[e];
    } else if (w == 2) {
      const vec2 v = *reinterpret_cast<const vec2*>(p + 16 * o + lane16 * 2);
      u[M + o] = v[0]; u[M + o + 1] = v[1];
    } else {
      u[M + o] = p[16 * o + lane16];
    }
  }
}

constexpr int kMaxIters = 63;             // largest refine_iters
// LDS floats of the staged image, whole KB
template <int G>
constexpr int kStageFloats = (SuLayout<G>::floats() + 255) / 256 * 256;

// x of another lane of this 16-lane row as the DPP operand of the arithmetic it feeds (bound_ctrl set and no
// "old" value: the compiler folds the move into a VOP2 instruction that uses it once).
template <int CTRL>
__device__ __forceinline__ int dpp_operand(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}
template <int O>
__device__ __forceinline__ float from_lane(float x) {
  return __builtin_bit_cast(float, dpp_operand<0x150 + O>(__builtin_bit_cast(int, x)));
}
// unsigned minimum with the partner of butterfly stage R (xor 1, xor 2, half mirror, mirror)
template <int R>
__device__ __forceinline__ unsigned min_stage(unsigned x) {
  constexpr int kCtrl[4] = {0xB1, 0x4E, 0x141, 0x140};
  const unsigned o = (unsigned)dpp_operand<kCtrl[R]>((int)x);
  return o < x ? o : x;
}
// A signed distance as an unsigned number that orders by magnitude, then positive before negative
__device__ __forceinline__ unsigned distance_key(float d) {
  const unsigned x = __builtin_bit_cast(unsigned, d);
  return __builtin_amdgcn_alignbit(x, x, 31);
}

// Empty asm statements with a value as in/out operand fix the place of the instruction that
// produces it: volatile asm statements keep their order.
#define BPDQ_PIN(x) asm volatile("" : "+v"(x))

// Rows of the local factor on their way from LDS: a step lasts 55 cycles, less than a read of LDS takes, so rows are requested
// kAhead steps before the one that uses them (at g = 256, where a step is longer and a row takes twice the registers, one).
// A ring of kAhead + 2 rows: the update of the next column's slot is on the critical path and done at once; the slots beyond it
// are updated inside the next step, where their multiply-adds fill the wait states of that step's serial chain.
template <int G>
constexpr int kAhead = G > 128 ? 1 : 3;
template <int G>
struct RowRing {
  float e;                              // broadcast error coordinate of the column before
  float x;                              // its coordinate of the plane's solve, where that advances with the sweep
  float u[kAhead<G> + 2][G / 16];
};
template <int G, int L>
__device__ __forceinline__ void request_row(RowRing<G>& ring, const float* __restrict__ sU, int lane16) {
  if constexpr (L + 1 < G) load_u_row<G, L / 16>(sU + SuLayout<G>::row_offset(L), lane16, ring.u[L % (kAhead<G> + 2)]);
}
// LDS reads in flight behind row L once row L + kAhead is requested
template <int G>
constexpr int reads_behind(int L) {
  int n = 0;
  for (int r = L + 1; r <= L + kAhead<G> && r + 1 < G; ++r) n += SuLayout<G>::chunks(r / 16);
  return n;
}
template <bool SOLVE, int K, int G, int L, int FIRST, int F0, int F1>
__device__ __forceinline__ void far_updates(RowState<K, G>& st, const RowRing<G>& ring) {
  if constexpr (F0 < F1) {
    const float u = ring.u[L % (kAhead<G> + 2)][FIRST + F0];
    st.wg[FIRST + F0] = fmaf(ring.e, u, st.wg[FIRST + F0]);
    BPDQ_PIN(st.wg[FIRST + F0]);
    if constexpr (SOLVE) {
      st.P[FIRST + F0][0] = fmaf(ring.x, u, st.P[FIRST + F0][0]);
      BPDQ_PIN(st.P[FIRST + F0][0]);
    }
    far_updates<SOLVE, K, G, L, FIRST, F0 + 1, F1>(st, ring);
  }
}

// One column of the sweep: nearest level (Eq. 7-8), error coordinate (Eq. 3), compensation of the later
// columns of the group (Eq. 4).
//
// A step is bound by vector issue (a SIMD holds one or two wavefronts, and every instruction of one
// takes four cycles), so what counts is how few instructions it has and that the serial chain of the
// decision never waits:
//   * Lane c of a row holds the level of code c % 2^K (`lv`), so one subtraction gives all distances.  What the
//     later columns need is the signed distance to the nearest level and not its code: distances are turned into keys that
//     order by magnitude and keep the sign (distance_key), K butterfly stages give the smallest.  The codes are found after
//     the sweep, for 16 columns at a time, from the weights that it leaves in place (the factor's row is zero on and
//     left of its diagonal), and the plane solves, which no decision of the sweep needs, follow it (solve_planes).
//   * Two levels at the same distance on either side of the weight: the key takes the lower level, a scan over the codes
//     with a strict `<` the lower code.  That is the same level where levels ascend with their codes; elsewhere
//     sweep() looks for such ties.
//   * Broadcasts are DPP operands of the arithmetic that needs them.
//   * A DPP operand must be two instructions old: the far updates of the previous column are dealt to those places.
// 14 instructions per column at 2 planes, 73 cycles in a launch of one wavefront per SIMD (their serial chain alone takes 52); with
// the code found by a second butterfly in the step and the solves advancing with it, 42 instructions and 176 cycles.
// Sweep and solves together, a group of 128 columns, 2 planes: 22.5 k -> 18.6 k cycles; whole layers, the same bits:
// 3584 x 3584, 2 planes, 5 iterations 2531 -> 2212 us; 18944 x 3584, 3 planes 10.4 -> 8.96 ms; 256 x 256 (groups of 64, 3
// iterations) 113.5 -> 90.3 us.
// One plane in groups of 128 and 256 (kSolveInSweep): the plane's solve advances with the sweep, 4 instructions and a
// multiply-add per slot, with the row that is there.  Behind the sweep it reads the factor again and fills a quarter of the
// matrix products' rows.  Whole layers, 5 iterations, solve behind / in the sweep, us: groups of 256, 3584 x 2048 1372 / 1170,
// 18944 x 1024 2940 / 2428, 70 x 2048 1282 / 1076; groups of 128, 986 / 954, 1514 / 1405, 802 / 764; on the other side, groups of 64,
// 1006 / 1061, 1428 / 1460, 808 / 860, of 32 1309 / 1392, 1707 / 1817, 1117 / 1180 (chains that the few slots do not fill).
template <int K, int G>
constexpr bool kSolveInSweep = K == 1 && G >= 128;
template <bool SOLVE, int K, int G, int L>
__device__ __forceinline__ void column_step(RowState<K, G>& st, const float* __restrict__ sU, float lv, int lane16,
                                            RowRing<G>& ring) {
  constexpr int CPL = G / 16, M = L / 16, O = L % 16, MN = (L + 1) / 16;
  // far updates of column L - 1: the slots beyond column L's
  constexpr int NF = (L == 0) ? 0 : CPL - M - 1;
  request_row<G, L + kAhead<G>>(ring, sU, lane16);
  __builtin_amdgcn_s_waitcnt(0xc07f | (reads_behind<G>(L) << 8));        // lgkmcnt: this column's row is here
  __builtin_amdgcn_sched_barrier(0);     // the requests stay ahead of this column's arithmetic
  constexpr auto at = [](int f) { return f < NF ? f : NF; };
  // The two ends of the chain are strings: between two values that a pin fixes the compiler would put wait states.
  // wg[M] has to be two instructions old for its broadcast, which the compiler does not look after in a string: a read
  // and a wait lie in between, or two waits.
  unsigned key;
  if constexpr (L + kAhead<G> + 1 >= G) asm volatile("s_nop 0");
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("v_sub_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n\t"
               "v_alignbit_b32 %0, %0, %0, 31" : "=&v"(key) : "v"(st.wg[M]), "v"(lv), "n"(O));      // distance_key
  far_updates<SOLVE, K, G, L - 1, M + 1, 0, at(2)>(st, ring);
  const unsigned own = key;
  key = min_stage<0>(key);
  if constexpr (K > 1) {
    BPDQ_PIN(key);
    far_updates<SOLVE, K, G, L - 1, M + 1, at(2), at(4)>(st, ring);
    key = min_stage<1>(key);
  }
  if constexpr (K > 2) {
    BPDQ_PIN(key);
    far_updates<SOLVE, K, G, L - 1, M + 1, at(4), at(6)>(st, ring);
    key = min_stage<2>(key);
  }
  if constexpr (K > 3) {
    BPDQ_PIN(key);
    far_updates<SOLVE, K, G, L - 1, M + 1, at(6), at(8)>(st, ring);
    key = min_stage<3>(key);
  }
  far_updates<SOLVE, K, G, L - 1, M + 1, at(2 * K), NF>(st, ring);
  // back to the distance, its error coordinate, and the slot of column L + 1 at once; the others in the next step
  float e;
  asm volatile("v_alignbit_b32 %0, %2, %2, 1\n\t"
               "v_mul_f32_dpp %0, %3, %0 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
               "v_fmac_f32 %1, %0, %4"
               : "=&v"(e), "+v"(st.wg[MN]) : "v"(key), "v"(st.inv[M]), "v"(ring.u[L % (kAhead<G> + 2)][MN]), "n"(O));
  ring.e = e;
  if constexpr (SOLVE) {
    const float b = (unsigned)dpp_operand<0x150>((int)own) != key ? 1.f : 0.f;     // level 0 is not the nearest
    ring.x = (from_lane<O>(st.P[M][0]) + b) * from_lane<O>(st.inv[M]);
    st.P[MN][0] = fmaf(ring.x, ring.u[L % (kAhead<G> + 2)][MN], st.P[MN][0]);
  }
  __builtin_amdgcn_sched_barrier(0);     // later steps' reads stay behind this step
}
template <bool SOLVE, int K, int G, int... Ls>
__device__ __forceinline__ void run_columns(RowState<K, G>& st, const float* sU, float lv, int lane16,
                                            std::integer_sequence<int, Ls...>) {
  RowRing<G> ring;
  request_row<G, 0>(ring, sU, lane16);
  if constexpr (kAhead<G> > 1) {
    request_row<G, 1>(ring, sU, lane16);
    request_row<G, 2>(ring, sU, lane16);
  }
  __builtin_amdgcn_sched_barrier(0);
  (column_step<SOLVE, K, G, Ls>(st, sU, lv, lane16, ring), ...);
}

// v(code) = ((c0 + b1 c1) + b2 c2) + ...  in fp32 (Eq. 7)
template <int K>
__device__ __forceinline__ void level_table(const float (&c)[K + 1], float (&lv)[1 << K]) {
#pragma unroll
  for (int code = 0; code < (1 << K); ++code) {
    float v = c[0];
#pragma unroll
    for (int i = 0; i < K; ++i)
      if ((code >> i) & 1) v = v + c[i + 1];
    lv[code] = v;
  }
}
// The levels a sweep decides on.  A level that is not finite never beats code 0 in a scan with a strict `<`: it takes part
// as another code 0, so that all distances of a NaN weight, and of an infinite C_0, are one bit pattern
// (NaNs of different origin are not).
template <int K>
__device__ __forceinline__ void sweep_levels(const float (&c)[K + 1], float (&lv)[1 << K]) {
  level_table<K>(c, lv);
#pragma unroll
  for (int q = 1; q < (1 << K); ++q) lv[q] = __builtin_isfinite(lv[q]) ? lv[q] : c[0];
}

// Nearest level of w by squared distance, the lowest code of several: the definition of a decision.
template <int K>
__device__ __forceinline__ float scan_levels(float w, const float (&lv)[1 << K], int& code) {
  float d0 = w - lv[0], best = d0 * d0;
  code = 0;
#pragma unroll
  for (int q = 1; q < (1 << K); ++q) {
    const float d = w - lv[q], s = d * d;
    const bool lt = s < best;
    best = lt ? s : best;
    d0 = lt ? d : d0;
    code = lt ? q : code;
  }
  return d0;
}

// The sweep by that definition, column by column, in a loop: for the rare wavefront whose sweep by keys met a tie that
// the definition decides the other way (a few times the duration of the unrolled sweep).
template <int K, int G, int M = 0>
__device__ __forceinline__ void sweep_by_scan(RowState<K, G>& st, const float* __restrict__ sU, const float (&lv)[1 << K],
                                              int lane16) {
  using Lay = SuLayout<G>;
  constexpr int CPL = G / 16;
  BPDQ_PIN(lane16);           // opaque, as in solve_block
#pragma unroll 1
  for (int o = 0; o < 16; ++o) {
    int code;
    const float e = scan_levels<K>(__shfl(st.wg[M], o, 16), lv, code) * __shfl(st.inv[M], o, 16);
    st.code[M] = (lane16 == o) ? code : st.code[M];
    const float* row = sU + Lay::row_offset(16 * M) + 16 * o * Lay::live(M);
#pragma unroll
    for (int m = M; m < CPL; ++m) st.wg[m] = fmaf(e, row[Lay::slot_index(CPL - M, m - M, lane16)], st.wg[m]);
  }
  if constexpr (M + 1 < CPL) sweep_by_scan<K, G, M + 1>(st, sU, lv, lane16);
}

// One sweep over the group's columns with coefficients c: leaves the codes, and in wg the weights they were decided on.  With
// SOLVE also the plane's solve, true then; false if it has to follow.
template <bool SOLVE, int K, int G>
__device__ __forceinline__ bool sweep(RowState<K, G>& st, const float* __restrict__ sU, const float (&c)[K + 1], int lane16) {
  constexpr int CPL = G / 16;
  float lv = c[0];
#pragma unroll
  for (int i = 0; i < K; ++i) lv = ((lane16 >> i) & 1) ? lv + c[i + 1] : lv;
  lv = __builtin_isfinite(lv) ? lv : c[0];
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    st.wg[m] = st.t[m];
    if constexpr (SOLVE) st.P[m][0] = 0.f;
  }
  run_columns<SOLVE, K, G>(st, sU, lv, lane16, std::make_integer_sequence<int, G - 1>{});     // the last column has none behind it

  // The codes, by the smallest magnitude; its order is that of the squares unless those leave the range of fp32.  Where levels
  // descend somewhere (ties, see column_step), lie so close that squares of distances between them underflow, or so
  // far out that they overflow, each decision is compared with the definition.  So it is where a weight is not finite:
  // the zeros left of the factor's diagonal make NaNs of the columns that were finished before it.
  float lvl[1 << K], sum = 0.f;
  sweep_levels<K>(c, lvl);
  bool odd = false;
#pragma unroll
  for (int q = 1; q < (1 << K); ++q) {
    const float gap = lvl[q] - lvl[q - 1];
    odd |= !(gap >= 0x1p-60f || gap == 0.f);
  }
#pragma unroll
  for (int m = 0; m < CPL; ++m) sum += fabsf(st.wg[m]);
  odd |= !(sum + fabsf(lvl[0]) + fabsf(lvl[(1 << K) - 1]) < 0x1p60f);
  if (!__any(odd)) {
#pragma unroll
    for (int m = 0; m < CPL; ++m) {
      const float w = st.wg[m];
      float best = fabsf(w - lvl[0]);
      int code = 0;
#pragma unroll
      for (int q = 1; q < (1 << K); ++q) {
        const float d = fabsf(w - lvl[q]);
        code = d < best ? q : code;
        best = d < best ? d : best;
      }
      st.code[m] = code;
    }
    return SOLVE;
  }
  bool other = false;
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    const float d0 = scan_levels<K>(st.wg[m], lvl, st.code[m]);
    unsigned key = distance_key(st.wg[m] - lvl[0]);
#pragma unroll
    for (int q = 1; q < (1 << K); ++q) {
      const unsigned k = distance_key(st.wg[m] - lvl[q]);
      key = k < key ? k : key;
    }
    other |= key != distance_key(d0) || st.wg[m] != st.wg[m];
  }
  if (__any(other)) {
#pragma unroll
    for (int m = 0; m < CPL; ++m) st.wg[m] = st.t[m];
    sweep_by_scan<K, G>(st, sU, lvl, lane16);
    return false;
  }
  return SOLVE;
}

// Right-solves with U_loc of rows that are known: slots [0, NP) of st.P run from the plane bits, and, where NT, slot NP from
// what st.P holds there (the target).  The forward recurrence x_l = v_l / U_ll, v_j -= x_l U_lj with its products in
// ascending l, every one a fused multiply-add in fp32, so where a product is formed does not change a bit:
//   * inside a block of 16 columns, and from a block to the next, on the vector units, x_l as a DPP operand;
//   * from a block to all later ones on the matrix cores: v_mfma_f32_16x16x4_f32 gives the same bits as a chain of four
//     fused multiply-adds in ascending k, rounded to nearest each (measured, and compared with an emulation by the tests).  Row a = 4 q + i of its A operand is slot i of row q of the wavefront, so register i
//     of lane (q, c) of the result is that slot's right-hand side of column c, which is where the recurrence wants it.  A
//     block's coordinates reach that operand layout through LDS.
// The matrix cores take fp32 products through the vector units' multipliers: nothing of the wavefront issues beside
// one, and one costs 31 cycles in a run of them on different tiles (40 alone, 52 behind one of the same tile), so a block's
// products come as one run, tiles innermost.  Four slots wide they do the work of 16 broadcast multiply-adds of 5 cycles
// a slot; at 2 planes half of that is used: 124 cycles a tile against 166.
constexpr int kSolveFloats = 256;             // LDS of a wavefront: [column of the block][row][slot]
template <int G, int M>
__device__ __forceinline__ void load_block_rows(const float* __restrict__ sU, int lane16, float (&own)[16], float (&next)[16]) {
  using Lay = SuLayout<G>;
  typedef float vec2 __attribute__((ext_vector_type(2)));
  constexpr int S = G / 16 - M, w = Lay::chunk_width(S, 0);
#pragma unroll
  for (int o = 0; o < 16; ++o) {
    const float* p = sU + Lay::row_offset(16 * M + o);
    if constexpr (S > 1) {
      const vec2 v = *reinterpret_cast<const vec2*>(p + w * lane16);
      own[o] = v[0];
      next[o] = v[1];
    } else {
      own[o] = p[lane16];
    }
  }
}
// The multiply-add with a broadcast operand, v += z(lane O of the row) * u, is not formed by the compiler (a move and a
// multiply-add instead): assembly.  z must have been written two instructions before, which the compiler does not look after
// there: a string holds what writes z, or begins with the wait; and several columns, because the compiler puts a wait
// state between two strings that share a register.
#define BPDQ_FMAC(v, z, u, o) "v_fmac_f32_dpp %[v" #v "], %[z" #z "], %[u" #u "] row_newbcast:%[o]+" #o " row_mask:0xf bank_mask:0xf\n\t"
#define BPDQ_Z(i) "v_add_f32 %[z" #i "], %[b" #i "], %[v" #i "]\n\t"
#define BPDQ_S(i) "v_mul_f32 %[z" #i "], %[z" #i "], %[w]\n\t"
#define BPDQ_STEP1(e) BPDQ_Z(0) BPDQ_S(0) "s_nop 1\n\t" BPDQ_FMAC(0, 0, e, e)
#define BPDQ_STEP2(e) BPDQ_Z(0) BPDQ_Z(1) BPDQ_S(0) BPDQ_S(1) "s_nop 0\n\t" BPDQ_FMAC(0, 0, e, e) BPDQ_FMAC(1, 1, e, e)
#define BPDQ_STEP3(e) BPDQ_Z(0) BPDQ_Z(1) BPDQ_Z(2) BPDQ_S(0) BPDQ_S(1) BPDQ_S(2) BPDQ_FMAC(0, 0, e, e) BPDQ_FMAC(1, 1, e, e) \
  BPDQ_FMAC(2, 2, e, e)
#define BPDQ_STEP4(e) BPDQ_Z(0) BPDQ_Z(1) BPDQ_Z(2) BPDQ_Z(3) BPDQ_S(0) BPDQ_S(1) BPDQ_S(2) BPDQ_S(3) BPDQ_FMAC(0, 0, e, e) \
  BPDQ_FMAC(1, 1, e, e) BPDQ_FMAC(2, 2, e, e) BPDQ_FMAC(3, 3, e, e)
#define BPDQ_FIVE(S) S(0) S(1) S(2) S(3) S(4)
#define BPDQ_U5 [u0] "v"(u[O]), [u1] "v"(u[O + 1]), [u2] "v"(u[O + 2]), [u3] "v"(u[O + 3]), [u4] "v"(u[O + 4]), [w] "v"(inv), [o] "n"(O)
// columns O .. O + 4 of a block: z = (b + v) / U_ll where the column is, then the rest of the block
template <int N, int O>
__device__ __forceinline__ void solve_five(float (&v)[4], const float (&b)[4], float inv, const float (&u)[16]) {
  float z0, z1, z2, z3;
  if constexpr (N == 1)
    asm volatile(BPDQ_FIVE(BPDQ_STEP1) : [v0] "+v"(v[0]), [z0] "=&v"(z0) : [b0] "v"(b[0]), BPDQ_U5);
  else if constexpr (N == 2)
    asm volatile(BPDQ_FIVE(BPDQ_STEP2) : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [z0] "=&v"(z0), [z1] "=&v"(z1)
                 : [b0] "v"(b[0]), [b1] "v"(b[1]), BPDQ_U5);
  else if constexpr (N == 3)
    asm volatile(BPDQ_FIVE(BPDQ_STEP3)
                 : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2]), [z0] "=&v"(z0), [z1] "=&v"(z1), [z2] "=&v"(z2)
                 : [b0] "v"(b[0]), [b1] "v"(b[1]), [b2] "v"(b[2]), BPDQ_U5);
  else
    asm volatile(BPDQ_FIVE(BPDQ_STEP4)
                 : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2]), [v3] "+v"(v[3]), [z0] "=&v"(z0), [z1] "=&v"(z1),
                   [z2] "=&v"(z2), [z3] "=&v"(z3)
                 : [b0] "v"(b[0]), [b1] "v"(b[1]), [b2] "v"(b[2]), [b3] "v"(b[3]), BPDQ_U5);
}
#define BPDQ_NEXT1(e) BPDQ_FMAC(0, 0, e, e) "s_nop 0\n\t"
#define BPDQ_NEXT2(e) BPDQ_FMAC(0, 0, e, e) BPDQ_FMAC(1, 1, e, e)
#define BPDQ_NEXT3(e) BPDQ_NEXT2(e) BPDQ_FMAC(2, 2, e, e)
#define BPDQ_NEXT4(e) BPDQ_NEXT3(e) BPDQ_FMAC(3, 3, e, e)
#define BPDQ_EIGHT(S) "s_nop 1\n\t" S(0) S(1) S(2) S(3) S(4) S(5) S(6) S(7)
#define BPDQ_U8 [u0] "v"(u[O]), [u1] "v"(u[O + 1]), [u2] "v"(u[O + 2]), [u3] "v"(u[O + 3]), [u4] "v"(u[O + 4]), \
  [u5] "v"(u[O + 5]), [u6] "v"(u[O + 6]), [u7] "v"(u[O + 7]), [o] "n"(O)
// columns O .. O + 7 of a finished block to the next block
template <int N, int O>
__device__ __forceinline__ void solve_next(float (&v)[4], const float (&z)[4], const float (&u)[16]) {
  if constexpr (N == 1)
    asm volatile(BPDQ_EIGHT(BPDQ_NEXT1) : [v0] "+v"(v[0]) : [z0] "v"(z[0]), BPDQ_U8);
  else if constexpr (N == 2)
    asm volatile(BPDQ_EIGHT(BPDQ_NEXT2) : [v0] "+v"(v[0]), [v1] "+v"(v[1]) : [z0] "v"(z[0]), [z1] "v"(z[1]), BPDQ_U8);
  else if constexpr (N == 3)
    asm volatile(BPDQ_EIGHT(BPDQ_NEXT3) : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2])
                 : [z0] "v"(z[0]), [z1] "v"(z[1]), [z2] "v"(z[2]), BPDQ_U8);
  else
    asm volatile(BPDQ_EIGHT(BPDQ_NEXT4) : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2]), [v3] "+v"(v[3])
                 : [z0] "v"(z[0]), [z1] "v"(z[1]), [z2] "v"(z[2]), [z3] "v"(z[3]), BPDQ_U8);
}
template <int NP, int NT, int K, int G, int M>
__device__ __forceinline__ void solve_block(RowState<K, G>& st, const float* __restrict__ sU, float* sX, int lane,
                                            float (&v)[4], float (&own)[16], float (&next)[16]) {
  using Lay = SuLayout<G>;
  constexpr int CPL = G / 16, N = NP + NT;
  int lane16 = lane & 15, q = lane >> 4;
  if constexpr (G > 128) {      // opaque again: registers are short
    BPDQ_PIN(lane16);
    BPDQ_PIN(q);
  }
  float b[4], z[4];
#pragma unroll
  for (int i = 0; i < N; ++i) b[i] = (i < NP) ? (float)((st.code[M] >> i) & 1) : -0.f;    // -0 + v is v, its sign too
  solve_five<N, 0>(v, b, st.inv[M], own);
  solve_five<N, 5>(v, b, st.inv[M], own);
  solve_five<N, 10>(v, b, st.inv[M], own);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    z[i] = (b[i] + v[i]) * st.inv[M];
    st.P[M][i] = z[i];
  }
  if constexpr (M + 1 < CPL) {
    constexpr bool kFar = M + 2 < CPL, kAll = G <= 128;
    float nown[16], nnext[16], a[4], f[kAll ? 4 : 2][CPL], w[4];
    auto request = [&](int kk) {                                   // the factor's rows 4 kk .. 4 kk + 3 of the block
      load_u_row<G, M, M + 2>(sU + Lay::row_offset(16 * M) + 16 * (4 * kk + q) * Lay::live(M), lane16, f[kAll ? kk : kk & 1]);
    };
    if constexpr (kFar) {
      *reinterpret_cast<f4*>(sX + 16 * lane16 + 4 * q) = st.P[M];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // one wavefront's LDS accesses keep their order
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        a[kk] = sX[64 * kk + lane];
        if (kAll || kk == 0) request(kk);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = st.P[M + 1][i];
    solve_next<N, 0>(w, z, next);
    solve_next<N, 8>(w, z, next);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kAll || !kFar) load_block_rows<G, M + 1>(sU, lane16, nown, nnext);
    if constexpr (kFar) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if constexpr (!kAll) {
          if (kk < 3) request(kk + 1);
          else load_block_rows<G, M + 1>(sU, lane16, nown, nnext);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = M + 2; n < CPL; ++n)
          st.P[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], f[kAll ? kk : kk & 1][n], st.P[n], 0, 0, 0);
      }
      // The strings of the next block may be given registers of slots that nobody reads: eleven wait states behind a
      // product that writes them.  (The vector units are not free sooner.)
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 10");
    }
    __builtin_amdgcn_sched_barrier(0);
    solve_block<NP, NT, K, G, M + 1>(st, sU, sX, lane, w, nown, nnext);
  }
}
template <int NP, int NT, int K, int G>
__device__ __forceinline__ void solve_planes(RowState<K, G>& st, const float* __restrict__ sU, float* sX) {
  int lane = threadIdx.x & 63;
  BPDQ_PIN(lane);               // opaque, or the addresses that follow from it stay in registers over all sweeps
#pragma unroll
  for (int m = 0; m < G / 16; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (NT == 0 || i != NP) st.P[m][i] = 0.f;
  float own[16], next[16], v[4];
  load_block_rows<G, 0>(sU, lane & 15, own, next);
#pragma unroll
  for (int i = 0; i < NP + NT; ++i) v[i] = st.P[0][i];
  solve_block<NP, NT, K, G, 0>(st, sU, sX, lane, v, own, next);
}
// One column of the recurrence on the target alone, in wg.
// (Four planes fill the rows of the matrix products; a pass of those for the target alone fills a quarter of them, and without
// refinement made 18944 x 1024 in groups of 128 slower than column steps that hold target and planes: 671 us, 715 with the pass,
// 675 with these steps; with one iteration 1152, 1082, 1046.)
template <int K, int G, int L>
__device__ __forceinline__ void target_step(RowState<K, G>& st, const float* __restrict__ sU, int lane16, RowRing<G>& ring) {
  constexpr int CPL = G / 16, M = L / 16, O = L % 16, MN = (L + 1) / 16;
  request_row<G, L + kAhead<G>>(ring, sU, lane16);
  __builtin_amdgcn_s_waitcnt(0xc07f | (reads_behind<G>(L) << 8));        // lgkmcnt: this column's row is here
  __builtin_amdgcn_sched_barrier(0);
  float z = st.wg[M] * st.inv[M];
  BPDQ_PIN(z);
  far_updates<false, K, G, L - 1, M + 1, 0, (L == 0) ? 0 : CPL - M - 1>(st, ring);
  ring.e = from_lane<O>(z);
  st.wg[MN] = fmaf(ring.e, ring.u[L % (kAhead<G> + 2)][MN], st.wg[MN]);
  __builtin_amdgcn_sched_barrier(0);
}
template <int K, int G, int... Ls>
__device__ __forceinline__ void run_target(RowState<K, G>& st, const float* sU, int lane16, std::integer_sequence<int, Ls...>) {
  RowRing<G> ring;
  request_row<G, 0>(ring, sU, lane16);
  if constexpr (kAhead<G> > 1) {
    request_row<G, 1>(ring, sU, lane16);
    request_row<G, 2>(ring, sU, lane16);
  }
  __builtin_amdgcn_sched_barrier(0);
  (target_step<K, G, Ls>(st, sU, lane16, ring), ...);
}

// tau = t U_loc^-1 and the planes of the first codes: in one pass where a slot is left for tau
template <int K, int G>
__device__ __forceinline__ void solve_target(RowState<K, G>& st, const float* __restrict__ sU, float* sX) {
  if constexpr (K < 4) {
#pragma unroll
    for (int m = 0; m < G / 16; ++m) st.P[m][K] = st.t[m];
    solve_planes<K, 1, K, G>(st, sU, sX);
#pragma unroll
    for (int m = 0; m < G / 16; ++m) st.tau[m] = st.P[m][K];
  } else {
#pragma unroll
    for (int m = 0; m < G / 16; ++m) st.wg[m] = st.t[m];
    run_target<K, G>(st, sU, threadIdx.x & 15, std::make_integer_sequence<int, G - 1>{});
#pragma unroll
    for (int m = 0; m < G / 16; ++m) st.tau[m] = st.wg[m] * st.inv[m];
    solve_planes<K, 0, K, G>(st, sU, sX);
  }
}

// Group records of a layer (SuLayout), by work-groups of 256 threads, kPackWGs<G> to a group: one per 16 rows of the
// image (they keep the same slots, so an element's place is a few operations) and one for 1 / U_ll and P_0.
// Each is one or a few round trips to memory and a short chain.  With the whole image to a work-group, whose places
// took a loop per element, the launch took 20 us at g = 128: 16 x 256, 1 plane, fixed grid 46.1 us, 40.0 before there
// were records, 28.9 now; larger layers hide it beside the copy.
template <int G>
constexpr int kPackWGs = G / 16 + 1;

// Rows [16 M, 16 M + 16) of the rearranged block, zeros on and below the diagonal of the kept slots.
template <int G>
__device__ __forceinline__ void pack_image(const float* __restrict__ U, int ldu, int s0, int M, float* __restrict__ rec) {
  using Lay = SuLayout<G>;
  constexpr int kPer = 16 * G / 256;
  const int S = Lay::CPL - M, live = Lay::live(M), l0 = 16 * M;
  float* rows = rec + Lay::row_offset(l0);
  float v[kPer];
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int e = threadIdx.x + t * 256;
    v[t] = U[(long)(s0 + l0 + e / G) * ldu + s0 + e % G];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int e = threadIdx.x + t * 256;
    const int l = e / G, j = e % G, m = j >> 4;         // row l0 + l
    if (m < M) continue;
    float* row = rows + 16 * l * live;
    row[Lay::slot_index(S, m - M, j & 15)] = (j > l0 + l) ? -v[t] : 0.f;
    if (m == M && live > S) row[Lay::slot_index(S, S, j & 15)] = 0.f;
  }
}

// 1 / U_ll and, where `ones` (a fit follows), P_0 by the forward recurrence of column_step: one wavefront, lane
// j % 64 holding columns j, the next rows on their way while the present ones are worked on.
template <int G>
__device__ __forceinline__ void pack_p0(const float* __restrict__ U, int ldu, int s0, bool ones, float* __restrict__ rec) {
  constexpr int NS = (G + 63) / 64, kRows = (G > 128) ? 16 : 32;
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  float* out_inv = rec + SuLayout<G>::floats();
  float p[NS], iv[NS], u[2][kRows][NS];
  auto fetch = [&](int l0, float (&w)[kRows][NS]) {
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int j = lane + 64 * s;
        w[r][s] = U[(long)(s0 + l0 + r) * ldu + s0 + (j < G ? j : 0)];
      }
  };
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int j = lane + 64 * s;
    iv[s] = U[(long)(s0 + (j < G ? j : 0)) * ldu + s0 + (j < G ? j : 0)];
    p[s] = 1.0f;
  }
  if (ones) fetch(0, u[0]);
  __builtin_amdgcn_sched_barrier(0);       // all on their way before the first is used
#pragma unroll
  for (int s = 0; s < NS; ++s) iv[s] = 1.0f / iv[s];
  if (ones) {
#pragma unroll
    for (int l0 = 0; l0 < G; l0 += kRows) {
      if (l0 + kRows < G) fetch(l0 + kRows, u[(l0 / kRows + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int l = l0 + r, sl = l / 64;
        const float xl = p[sl] * iv[sl];
        const float x = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, xl), l % 64));
#pragma unroll
        for (int s = 0; s < NS; ++s) p[s] = fmaf(-x, (lane + 64 * s > l) ? u[(l0 / kRows) & 1][r][s] : 0.f, p[s]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int j = lane + 64 * s;
    if (j >= G) continue;
    out_inv[j] = iv[s];
    if (ones) out_inv[G + j] = p[s] * iv[s];
  }
}

// Request a group's image into LDS (at byte address 0 of the dynamic LDS), 1 KB per instruction, dealt
// to the four wavefronts; stage_wait() before the barrier that publishes it.  (Assembly, because the
// compiler would wait for all of it before the first LDS access; M0 is used for nothing else here, and has
// to be one wait state old when the load reads it, which the compiler does not see to in assembly: the s_nop.)
template <int G>
__device__ __forceinline__ void stage_request(const float* __restrict__ rec, float* sU) {
  typedef __attribute__((address_space(3))) float lds_float;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kKb = (SuLayout<G>::floats() + 255) / 256;
  const unsigned lds0 = (unsigned)(size_t)(lds_float*)sU;
  for (int c = wave; c < kKb; c += kSweepThreads / 64)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds0 + 1024u * c), "v"(1024u * c + 16u * lane), "s"(rec)
                 : "memory");
}
__device__ __forceinline__ void stage_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int K, int G>
__device__ __forceinline__ void load_record_rows(RowState<K, G>& st, const float* __restrict__ rec, int lane16) {
  const float* p = rec + SuLayout<G>::floats();
#pragma unroll
  for (int m = 0; m < G / 16; ++m) {
    st.inv[m] = p[16 * m + lane16];
    st.p0[m] = p[G + 16 * m + lane16];
  }
}

// Storage precision of the coefficients: fp32, or IEEE half (nearest even, from the precision they come in)
// when the layer is stored with 16-bit coefficients (Table 1), so that everything computed from them
// belongs to the stored values.  (A branch, uniform over the launch: as a select both would be computed
// for every fit, and the rounding of a double to half is a long piece of integer code.)
template <int N, typename T>
__device__ __forceinline__ void store_precision(const T (&c)[N], int coef_fp16, float (&c32)[N]) {
  if (coef_fp16) {
    asm volatile("");
#pragma unroll
    for (int a = 0; a < N; ++a) c32[a] = (float)(_Float16)c[a];
  } else {
#pragma unroll
    for (int a = 0; a < N; ++a) c32[a] = (float)c[a];
  }
}

// Coefficient fit (Eq. 6) from the solved vectors; returns c (fp32) and the row's ||E'||^2.
template <int K, int G>
__device__ __forceinline__ double fit_and_score(const RowState<K, G>& st, double alpha, int coef_fp16,
                                                float (&c32)[K + 1], float (&Ep)[G / 16]) {
  constexpr int CPL = G / 16, N = K + 1;
  double Gm[N][N], r[N];
#pragma unroll
  for (int a = 0; a < N; ++a) {
#pragma unroll
    for (int b = a; b < N; ++b) {
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < CPL; ++m) {
        const float va = (a == 0) ? st.p0[m] : st.P[m][a - 1 < 0 ? 0 : a - 1];
        const float vb = (b == 0) ? st.p0[m] : st.P[m][b - 1 < 0 ? 0 : b - 1];
        s += (double)va * (double)vb;
      }
      Gm[a][b] = row_sum_d(s);
    }
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < CPL; ++m) {
      const float va = (a == 0) ? st.p0[m] : st.P[m][a - 1 < 0 ? 0 : a - 1];
      s += (double)va * (double)st.tau[m];
    }
    r[a] = row_sum_d(s);
  }
  double tr = 0.0;
#pragma unroll
  for (int a = 0; a < N; ++a) tr += Gm[a][a];
  const double mu = alpha * tr / (double)N;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    Gm[a][a] += mu;
#pragma unroll
    for (int b = 0; b < a; ++b) Gm[a][b] = Gm[b][a];
  }
  // Gaussian elimination without pivoting (G is symmetric positive definite after the ridge)
#pragma unroll
  for (int p = 0; p < N; ++p) {
    const double ip = 1.0 / Gm[p][p];
#pragma unroll
    for (int a = p + 1; a < N; ++a) {
      const double f = Gm[a][p] * ip;
#pragma unroll
      for (int b = p + 1; b < N; ++b) Gm[a][b] -= f * Gm[p][b];
      r[a] -= f * r[p];
    }
  }
  double c[N];
#pragma unroll
  for (int a = N - 1; a >= 0; --a) {
    double s = r[a];
#pragma unroll
    for (int b = a + 1; b < N; ++b) s -= Gm[a][b] * c[b];
    c[a] = s / Gm[a][a];
  }
  store_precision(c, coef_fp16, c32);
  double sc = 0.0;
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    float e = fmaf(-c32[0], st.p0[m], st.tau[m]);
#pragma unroll
    for (int i = 0; i < K; ++i) e = fmaf(-c32[i + 1], st.P[m][i], e);
    Ep[m] = e;
    sc += (double)e * (double)e;
  }
  return row_sum_d(sc);
}

// ------------------------------------------------------------------ pending updates --------
// Error compensation of the columns not yet quantized (Eq. 4) is applied lazily, block by block
// (App. B.3, tail form), and never on the critical path between two groups:
//   * every committed E* is kept K-major in Eall[column][row] (leading dimension lde);
//   * the group that starts at column s0 reads its target left-looking:
//       t = W'[rows, s0:s0+g] - Eall[kp0:s0, rows]^T U[kp0:s0, s0:s0+g]
//     where kp0 is the start of the previous block: W' itself holds the updates of all blocks
//     before that one;
//   * the update of block q-1 to the columns beyond block q is a GEMM that extra work-groups of
//     the first group launch of block q perform (the "tail role"): it only needs E* committed
//     before the launch and touches no column the launch's sweep reads, so it overlaps the
//     latency-bound sweep instead of waiting between two of them;
//   * two levels: that per-block update (depth B) only reaches to the end of the NEXT super-block
//     (about 1024 columns per super-block); the columns beyond receive one deep update per finished
//     super-block (depth ~1024: an eighth of the traffic on W' per flop, and long enough to
//     amortise a tile's prologue), dealt in column chunks to the group launches of the following
//     super-block.  The two updates of one launch never touch the same columns (see the host loop).
//     Only the order of summation differs from one update per block.
struct TailTask {
  const float* Et;     // Eall + k0 * lde
  int Kd;              // depth of the update (finished columns)
  int k0;              // first finished column (row of U)
  int c_begin, c_end;  // columns [c_begin, c_end) of W' to update
  int tiles_n;         // column tiles; 0 = nothing to do
};
struct TailArgs {
  TailTask far, near;  // deep update of a finished super-block / update of the previous block
  float* Wp;           // working copy W'
  int first_wg;        // work-groups below this index sweep
  int far_wgs;         // tail work-groups [first_wg, first_wg + far_wgs) take `far`, the rest `near`
};

// Layers that share one input share U and go through the sweep stacked by rows; the best
// iterate of a group is chosen per layer (segment).  Boundaries in work-groups of 16 rows.
constexpr int kMaxSegments = 8;
struct SegArgs {
  int n_seg;
  int wg_end[kMaxSegments];   // ascending; wg_end[n_seg - 1] = number of sweeping work-groups
};

// W'[:, c_begin:c_end] -= Et^T U[k0:k0+Kd, c_begin:c_end], one 128 x 128 tile per work-group
__device__ __forceinline__ void tail_role(const TailArgs& ta, const float* __restrict__ U, int ldu,
                                          int lde, int ldw, int d_out) {
  int t = blockIdx.x - ta.first_wg;
  const bool is_far = t < ta.far_wgs;          // uniform over the work-group
  if (!is_far) t -= ta.far_wgs;
  const TailTask& task = is_far ? ta.far : ta.near;
  const int tm = t / task.tiles_n, tn = t % task.tiles_n;
  TailGemm::Acc acc;
  TailGemm::zero(acc);
  TailGemm::run<0>(task.Et, lde, tm * TailGemm::kTileM, lde, U + (long)task.k0 * ldu, ldu,
                   task.c_begin + tn * TailGemm::kTileN, task.c_end, 0, task.Kd, acc);
  const int r0 = tm * TailGemm::kTileM, c0 = task.c_begin + tn * TailGemm::kTileN;
  float* Wp = ta.Wp;
  const int c_end = task.c_end;
  // in-place read-modify-write of this lane's 64 results: all loads first, then the stores.  A tile that
  // lies inside the matrix takes them unguarded (guards become a branch per element); at the edges
  // masked elements read a valid address and are not stored.
  float old[TailGemm::kAccPerLane];
  if (r0 + TailGemm::kTileM <= d_out && c0 + TailGemm::kTileN <= c_end) {
    float* w = Wp + (long)r0 * ldw + c0;
    int n = 0;
    TailGemm::for_each(acc, [&](int row, int col, float) { old[n++] = w[(long)row * ldw + col]; });
    __builtin_amdgcn_sched_barrier(0);
    n = 0;
    TailGemm::for_each(acc, [&](int row, int col, float v) { w[(long)row * ldw + col] = old[n++] - v; });
    return;
  }
  int n = 0;
  TailGemm::for_each(acc, [&](int row, int col, float) {
    const int r = r0 + row, c = c0 + col;
    old[n++] = Wp[(r < d_out && c < c_end) ? (long)r * ldw + c : 0L];
  });
  n = 0;
  TailGemm::for_each(acc, [&](int row, int col, float v) {
    const int r = r0 + row, c = c0 + col;
    if (r < d_out && c < c_end) Wp[(long)r * ldw + c] = old[n] - v;
    ++n;
  });
}

// sT[r][c] = sum_{k < Kp} Eall[kp0 + k][row0 + r] * U[kp0 + k][s0 + c]   (16 rows x G columns)
// with v_mfma_f32_16x16x4_f32: the column blocks of 16 are dealt to the four wavefronts; operands
// go straight from global memory to registers (lane l: A[l % 16][l / 16], B[l / 16][l % 16]),
// the result (register r of lane l = D[4 (l / 16) + r][l % 16]) to LDS.  Kp % 32 == 0.
template <int G>
struct PendingTile {
  static constexpr int kStride = G + 4;
  static constexpr int kFloats = kRowsPerWG * kStride;
};
// LDS behind the image: the pending tile, later the row scores of every iterate
template <int G>
constexpr int kScratchFloats = PendingTile<G>::kFloats > 2 * (kMaxIters + 1) * kRowsPerWG ? PendingTile<G>::kFloats
                                                                                 : 2 * (kMaxIters + 1) * kRowsPerWG;
template <int G>
__device__ __forceinline__ void pending_update_tile(const float* __restrict__ Eall, int lde,
                                                    const float* __restrict__ U, int ldu, int kp0,
                                                    int Kp, int row0, int s0, float* sT) {
  constexpr int NB = G / 16, BPW = (NB + 3) / 4;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, kq = lane >> 4;
  f4 acc[BPW];
#pragma unroll
  for (int b = 0; b < BPW; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
  const float* ap = Eall + (long)(kp0 + kq) * lde + row0 + i;
  const float* bp = U + (long)(kp0 + kq) * ldu + s0 + 16 * wave * BPW + i;
  const bool active = wave * BPW < NB;          // g = 32: two blocks, wavefronts 2 and 3 idle
  if (active) {
    // Every MFMA step (4 columns of E*) of a batch is requested before the first is used, so a batch costs
    // one round trip to memory: 128 columns at once (the whole of a one-group block), then 64, then 32.
    // Kp % 32 == 0 (g >= 32 divides it).
    auto batch = [&](auto steps, int k) {
      constexpr int kSteps = decltype(steps)::value;
      float a[kSteps], bv[kSteps][BPW];
#pragma unroll
      for (int u = 0; u < kSteps; ++u) {
        a[u] = ap[(long)(k + 4 * u) * lde];
#pragma unroll
        for (int b = 0; b < BPW; ++b) bv[u][b] = bp[(long)(k + 4 * u) * ldu + 16 * b];
      }
      __builtin_amdgcn_sched_barrier(0);   // or the scheduler sinks every load to its product again
#pragma unroll
      for (int u = 0; u < kSteps; ++u)
#pragma unroll
        for (int b = 0; b < BPW; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], bv[u][b], acc[b], 0, 0, 0);
    };
    int k = 0;
    if constexpr (BPW <= 2)
      for (; k + 128 <= Kp; k += 128) batch(std::integral_constant<int, 32>{}, k);
    for (; k + 64 <= Kp; k += 64) batch(std::integral_constant<int, 16>{}, k);
    for (; k < Kp; k += 32) batch(std::integral_constant<int, 8>{}, k);
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sT[(4 * kq + r) * PendingTile<G>::kStride + 16 * (wave * BPW + b) + i] = acc[b][r];
  }
}

// Group-start working weights of this lane's columns: W' minus the pending updates.
template <int K, int G>
__device__ __forceinline__ void load_group_target(RowState<K, G>& st, const float* __restrict__ Wp,
                                                  int ldw, int rr, int s0, int lane16,
                                                  const float* __restrict__ Eall, int lde,
                                                  const float* __restrict__ U, int ldu, int kp0,
                                                  float* sT) {
  constexpr int CPL = G / 16;
  const float* wrow = Wp + (long)rr * ldw + s0;
#pragma unroll
  for (int m = 0; m < CPL; ++m) st.t[m] = wrow[16 * m + lane16];
  if (kp0 < s0) {                                   // uniform over the launch
    pending_update_tile<G>(Eall, lde, U, ldu, kp0, s0 - kp0, blockIdx.x * kRowsPerWG, s0, sT);
    __syncthreads();
    const float* trow = sT + (threadIdx.x >> 4) * PendingTile<G>::kStride;
#pragma unroll
    for (int m = 0; m < CPL; ++m) st.t[m] -= trow[16 * m + lane16];
  }
}

// Per-iterate scratch in the workspace, laid out by lane: codes uint32 [T+1][d_out][16][words], slot m of a
// lane in bits 4 (m % 8) of word m / 8; coefficients [T+1][d_out][K+1]; E' [T+1][d_out][16][G/16].  One
// to four wide stores per lane and iterate instead of one per slot and value.
template <int G>
constexpr int kCodeWords = (G > 128) ? 2 : 1;

template <int K, int G>
__device__ __forceinline__ void store_candidate(const RowState<K, G>& st, const float (&c32)[K + 1],
                                                const float (&Ep)[G / 16], double rowscore, int it,
                                                int row, bool valid, int d_out, uint32_t* codes,
                                                float* coef, float* E, double* sScore, int lane16) {
  constexpr int CPL = G / 16, NW = kCodeWords<G>;
  typedef float evec __attribute__((ext_vector_type(CPL < 4 ? 2 : 4)));
  constexpr int W = CPL < 4 ? 2 : 4;
  if (valid) {
    const long base = ((long)it * d_out + row) * 16 + lane16;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      uint32_t packed = 0u;
#pragma unroll
      for (int m = 8 * w; m < CPL && m < 8 * w + 8; ++m) packed |= (uint32_t)st.code[m] << (4 * (m - 8 * w));
      codes[base * NW + w] = packed;
    }
#pragma unroll
    for (int m = 0; m < CPL; m += W) {
      evec v;
#pragma unroll
      for (int e = 0; e < W; ++e) v[e] = Ep[m + e];
      *reinterpret_cast<evec*>(E + base * CPL + m) = v;
    }
    if (lane16 <= K) {
      float v = c32[0];
#pragma unroll
      for (int i = 1; i <= K; ++i) {
        v = (lane16 == i) ? c32[i] : v;
        BPDQ_PIN(v);        // or c32 goes through scratch memory, and its load waits for the stores above
      }
      coef[((long)it * d_out + row) * (K + 1) + lane16] = v;
    }
  }
  if (lane16 == 0) sScore[it * kRowsPerWG + (threadIdx.x >> 4)] = valid ? rowscore : 0.0;
}

// Scores of the work-group's 16 rows, summed in row order, for iterates 0 .. T.  Once per launch: a
// barrier per iterate would make every wavefront wait for its stores (1.4 k cycles an iterate).
__device__ __forceinline__ void store_scores(const double* sScore, int T, int n_wg, double* __restrict__ score) {
  __syncthreads();
  const int it = threadIdx.x;
  if (it <= T) {
    double s = 0.0;
    for (int q = 0; q < kRowsPerWG; ++q) s += sScore[it * kRowsPerWG + q];
    score[(long)it * n_wg + blockIdx.x] = s;
  }
}

// One group of g columns for 16 rows per work-group: initialisation, fit, T refinement
// iterations; every iterate's (codes, coefficients, E', score) is kept for the selection.
template <int K, int G>
__global__ __launch_bounds__(kSweepThreads, kSweepWavesPerSimd<G>) void bpdq_group_kernel(
    const float* __restrict__ Wp, int ldw, int d_out, const float* __restrict__ U, int ldu,
    const float* __restrict__ rec, int s0, int T, float alpha, int coef_fp16, uint32_t* __restrict__ cand_codes,
    float* __restrict__ cand_coef,
    float* __restrict__ cand_E, double* __restrict__ cand_score, int n_wg,
    const float* __restrict__ Eall, int lde, int kp0, TailArgs ta) {
  if constexpr (kTailInSweep<G>) {
    if ((int)blockIdx.x >= ta.first_wg) {
      tail_role(ta, U, ldu, lde, ldw, d_out);
      return;
    }
  }
  // the sweep is the critical path of the launch: where a sweeping and an updating wavefront share
  // a SIMD, the sweeping one issues first
  __builtin_amdgcn_s_setprio(3);
  constexpr int CPL = G / 16;
  extern __shared__ float lds[];
  float* sU = lds;                            // packed local factor, see SuLayout
  float* sT = lds + kStageFloats<G>;          // pending-update tile, then the row scores of every iterate
  double* sScore = reinterpret_cast<double*>(sT);
  const int tid = threadIdx.x;
  const int lane16 = tid & 15;
  float* sX = sT + kScratchFloats<G> + (tid >> 6) * kSolveFloats;     // this wavefront's, see solve_planes
  stage_request<G>(rec, sU);

  const int row = blockIdx.x * kRowsPerWG + (tid >> 4);
  const bool valid = row < d_out;
  const int rr = valid ? row : d_out - 1;
  RowState<K, G> st;
  load_record_rows<K, G>(st, rec, lane16);
  load_group_target<K, G>(st, Wp, ldw, rr, s0, lane16, Eall, lde, U, ldu, kp0, sT);
  stage_wait();
  __syncthreads();

  // ---- bit-plane initialisation (Sec. 3.2, Eq. 5): 8-bit affine RTN, keep the k MSB planes
  float lo = st.t[0], hi = st.t[0];
#pragma unroll
  for (int m = 1; m < CPL; ++m) {
    lo = fminf(lo, st.t[m]);
    hi = fmaxf(hi, st.t[m]);
  }
  lo = row_reduce_f(lo, [](float a, float b) { return fminf(a, b); });
  hi = row_reduce_f(hi, [](float a, float b) { return fmaxf(a, b); });
  const float sc = (hi - lo) / 255.0f;
  const bool flat = (hi == lo);
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    const float q = (st.t[m] - lo) / (flat ? 1.0f : sc);
    float z = rintf(q);                       // round half to even
    z = fminf(fmaxf(z, 0.f), 255.f);
    st.code[m] = flat ? 0 : ((int)z >> (8 - K));
  }
  float c32[K + 1], Ep[CPL];
  solve_target<K, G>(st, sU, sX);

  double rs = fit_and_score<K, G>(st, (double)alpha, coef_fp16, c32, Ep);
  store_candidate<K, G>(st, c32, Ep, rs, 0, row, valid, d_out, cand_codes, cand_coef, cand_E, sScore, lane16);

  // ---- refinement iterations (Sec. 3.3)
  for (int it = 1; it <= T; ++it) {
    if (sweep<kSolveInSweep<K, G>, K, G>(st, sU, c32, lane16)) {
#pragma unroll
      for (int m = 0; m < CPL; ++m) st.P[m][0] = ((float)(st.code[m] & 1) + st.P[m][0]) * st.inv[m];
    } else {
      solve_planes<K, 0, K, G>(st, sU, sX);
    }
    rs = fit_and_score<K, G>(st, (double)alpha, coef_fp16, c32, Ep);
    store_candidate<K, G>(st, c32, Ep, rs, it, row, valid, d_out, cand_codes, cand_coef, cand_E, sScore, lane16);
  }
  store_scores(sScore, T, n_wg, cand_score);
}

// Fixed-uniform-grid comparator (App. A, "Fixed Grid"): the same column sweep with the levels
// frozen to lo + s * {0 .. 2^k - 1}, s = (hi - lo) / (2^k - 1), written as bit-plane coefficients
// (lo, s, 2s, 4s, ...) -- the special case of Prop. 1.  One pass, no fit, no iteration: this is
// GPTQ on the asymmetric min/max grid.  The result is stored as iterate 0.
template <int K, int G>
__global__ __launch_bounds__(kSweepThreads, kSweepWavesPerSimd<G>) void uniform_group_kernel(
    const float* __restrict__ Wp, int ldw, int d_out, const float* __restrict__ U, int ldu,
    const float* __restrict__ rec, int s0, int coef_fp16, uint32_t* __restrict__ cand_codes, float* __restrict__ cand_coef,
    float* __restrict__ cand_E, double* __restrict__ cand_score, int n_wg,
    const float* __restrict__ Eall, int lde, int kp0, TailArgs ta) {
  if constexpr (kTailInSweep<G>) {
    if ((int)blockIdx.x >= ta.first_wg) {
      tail_role(ta, U, ldu, lde, ldw, d_out);
      return;
    }
  }
  // the sweep is the critical path of the launch: where a sweeping and an updating wavefront share
  // a SIMD, the sweeping one issues first
  __builtin_amdgcn_s_setprio(3);
  constexpr int CPL = G / 16;
  extern __shared__ float lds[];
  float* sU = lds;
  float* sT = lds + kStageFloats<G>;
  double* sScore = reinterpret_cast<double*>(sT);
  const int tid = threadIdx.x;
  const int lane16 = tid & 15;
  stage_request<G>(rec, sU);

  const int row = blockIdx.x * kRowsPerWG + (tid >> 4);
  const bool valid = row < d_out;
  const int rr = valid ? row : d_out - 1;
  RowState<K, G> st;
  load_record_rows<K, G>(st, rec, lane16);
  load_group_target<K, G>(st, Wp, ldw, rr, s0, lane16, Eall, lde, U, ldu, kp0, sT);
  stage_wait();
  __syncthreads();
  float lo = st.t[0], hi = st.t[0];
#pragma unroll
  for (int m = 1; m < CPL; ++m) {
    lo = fminf(lo, st.t[m]);
    hi = fmaxf(hi, st.t[m]);
  }
  lo = row_reduce_f(lo, [](float a, float b) { return fminf(a, b); });
  hi = row_reduce_f(hi, [](float a, float b) { return fmaxf(a, b); });
  float step = (hi - lo) / (float)((1 << K) - 1);
  if (step == 0.f) step = 1.0f;                 // flat row: every weight takes code 0
  float grid[K + 1], c32[K + 1], Ep[CPL];
  grid[0] = lo;
#pragma unroll
  for (int i = 0; i < K; ++i) grid[i + 1] = step * (float)(1 << i);
  store_precision(grid, coef_fp16, c32);
  sweep<false, K, G>(st, sU, c32, lane16);
  float lvl[1 << K];
  sweep_levels<K>(c32, lvl);
  double sc = 0.0;
#pragma unroll
  for (int m = 0; m < CPL; ++m) {
    float q = lvl[0];
#pragma unroll
    for (int c = 1; c < (1 << K); ++c) q = (st.code[m] == c) ? lvl[c] : q;
    Ep[m] = (st.wg[m] - q) * st.inv[m];
    sc += (double)Ep[m] * (double)Ep[m];
  }
  sc = row_sum_d(sc);
  store_candidate<K, G>(st, c32, Ep, sc, 0, row, valid, d_out, cand_codes, cand_coef, cand_E, sScore, lane16);
  store_scores(sScore, 0, n_wg, cand_score);
}

// Selection + commit of one group, 32 rows (two row blocks of the sweep, with its lane mapping) per work-group.
// Every work-group first sums the row-block scores of each iterate over its own layer (segment)
// in one fixed order and takes the earliest minimum (Sec. 3.3: keep the iterate with the smallest
// ||E_group||_F^2), so all work-groups of a layer agree bit for bit; the first row block of a
// segment publishes grp_iter / grp_err (arrays of n_grp entries per segment).  Then the kept
// iterate is written out: packed planes (wave ballots), coefficients, What, and E* transposed
// into the K-major error buffer Eblk[(s0 - b0) + j][row] (leading dimension lde).
// Bound by the dependent trips to memory (scores, then the kept iterate) on small layers, by traffic on large ones:
// 32 rows write whole lines of 128 bytes of Eblk and read the scores half as often as 16 rows do, eight wavefronts take one
// iterate each up to T = 7, and What goes out by 16 bytes a lane.  A launch at T = 5, 16 rows and 4-byte stores / this:
// 18944 rows, 3 planes 15.9 / 13.3 us (31 MB), 3584 rows, 2 planes 5.5 / 5.3.
constexpr int kCommitBlocks = 2, kCommitRows = kCommitBlocks * kRowsPerWG, kCommitThreads = 16 * kCommitRows;
template <int K, int G>
__global__ __launch_bounds__(kCommitThreads) void commit_group_kernel(
    const uint32_t* __restrict__ cand_codes, const float* __restrict__ cand_coef,
    const float* __restrict__ cand_E, const double* __restrict__ cand_score, int n_wg, int T,
    SegArgs seg, double* __restrict__ grp_err, int* __restrict__ grp_iter, int d_out, int d_in,
    int s0, int b0,
    uint32_t* __restrict__ planes, float* __restrict__ coefs, float* __restrict__ W_hat,
    float* __restrict__ Eblk, int lde) {
  constexpr int CPL = G / 16, kFlight = 8;
  __shared__ double tot[64];
  __shared__ float sE[G][kCommitRows + 1];
  __shared__ __attribute__((aligned(4))) unsigned char sCode[kCommitRows][G + 4];
  __shared__ float sLevel[kCommitRows][(1 << K) + 1];
  const int tid = threadIdx.x, lane16 = tid & 15;
  int it = 0, si_done = -1;
#pragma unroll 1
  for (int h = 0; h < kCommitBlocks; ++h) {
    // the segment of this row block (blocks past the last row belong to the last one; they write nothing)
    const int blk = blockIdx.x * kCommitBlocks + h;
    int wg_lo = 0, wg_hi = seg.wg_end[0], si = 0;
#pragma unroll
    for (int q = 1; q < kMaxSegments; ++q)
      if (q < seg.n_seg && blk >= seg.wg_end[q - 1]) {
        wg_lo = seg.wg_end[q - 1];
        wg_hi = seg.wg_end[q];
        si = q;
      }
    if (si == si_done) break;                            // uniform: the block before has it
    if (h > 0) __syncthreads();                          // tot has been read
    // iterate q is summed by wavefront q % 8: strided partial sums per lane, then a fixed
    // xor butterfly over the 64 lanes
    for (int q = tid >> 6; q <= T; q += kCommitThreads / 64) {
      double s = 0.0;
      // kFlight scores of a lane in flight, added in the order of the row blocks (one at a time a layer of 18944
      // rows waited 19 times per iterate; a score past the end adds zero)
      for (int w = wg_lo + (tid & 63); w < wg_hi; w += 64 * kFlight) {
        double v[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) v[u] = cand_score[(long)q * n_wg + (w + 64 * u < wg_hi ? w + 64 * u : w)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kFlight; ++u) s += (w + 64 * u < wg_hi) ? v[u] : 0.0;
      }
#pragma unroll
      for (int m = 32; m > 8; m >>= 1) s += __shfl_xor(s, m, 64);
      // within 16 lanes by rotations: of values that repeat every 16, 8, 4 and 2 lanes by then, those 8, 4, 2 and 1
      // lanes away are the butterfly's pairs (and a sum of two has no order)
      s += dpp_d<0x128>(s);
      s += dpp_d<0x124>(s);
      s += dpp_d<0x122>(s);
      s += dpp_d<0x121>(s);
      if ((tid & 63) == 0) tot[q] = s;
    }
    __syncthreads();
    int kept = 0;
    double best = tot[0];
#pragma unroll 4
    for (int q = 1; q <= T; ++q) {
      const double v = tot[q];
      kept = v < best ? q : kept;
      best = v < best ? v : best;
    }
    if (blk == wg_lo && tid == 0) {
      grp_iter[(long)si * (d_in / G)] = kept;
      grp_err[(long)si * (d_in / G)] = best;
    }
    if ((tid >> 8) >= h) it = kept;                      // 256 threads to a row block
    si_done = si;
  }

  const int row0 = blockIdx.x * kCommitRows;
  const int rloc = tid >> 4;
  const int row = row0 + rloc;
  const bool valid = row < d_out;
  const int rr = valid ? row : d_out - 1;
  const int n_grp = d_in / G, gi = s0 / G, n_word = d_in / 32;
  const long cbase = ((long)it * d_out + rr) * 16 + lane16;
  float c[K + 1], lv[1 << K];
#pragma unroll
  for (int i = 0; i <= K; ++i) c[i] = cand_coef[((long)it * d_out + rr) * (K + 1) + i];
  level_table<K>(c, lv);
  int code[CPL];
  float ev[CPL];
#pragma unroll
  for (int w = 0; w < kCodeWords<G>; ++w) {
    const uint32_t packed = cand_codes[cbase * kCodeWords<G> + w];
#pragma unroll
    for (int m = 8 * w; m < CPL && m < 8 * w + 8; ++m) code[m] = (int)((packed >> (4 * (m - 8 * w))) & 15u);
  }
  typedef float evec __attribute__((ext_vector_type(CPL < 4 ? 2 : 4)));
  constexpr int EW = CPL < 4 ? 2 : 4;
#pragma unroll
  for (int m = 0; m < CPL; m += EW) {
    const evec v = *reinterpret_cast<const evec*>(cand_E + cbase * CPL + m);
#pragma unroll
    for (int e = 0; e < EW; ++e) ev[m + e] = v[e];
  }
#pragma unroll
  for (int m = 0; m < CPL; ++m) sE[16 * m + lane16][rloc] = valid ? ev[m] : 0.f;
  // planes: a wave ballot holds bit (16 q + lane16) for row q of the wave
  const int shift = 16 * ((tid & 63) >> 4);
#pragma unroll
  for (int i = 0; i < K; ++i) {
#pragma unroll
    for (int w = 0; w < G / 32; ++w) {
      const unsigned long long lo = __ballot((code[2 * w] >> i) & 1);
      const unsigned long long hi = __ballot((code[2 * w + 1] >> i) & 1);
      const uint32_t word = (uint32_t)((lo >> shift) & 0xffffu) | ((uint32_t)((hi >> shift) & 0xffffu) << 16);
      if (valid && lane16 == 0) planes[((long)i * d_out + row) * n_word + s0 / 32 + w] = word;
    }
  }
  if (W_hat) {
#pragma unroll
    for (int m = 0; m < CPL; ++m) sCode[rloc][16 * m + lane16] = (unsigned char)code[m];
    float v = lv[0];
#pragma unroll
    for (int q = 1; q < (1 << K); ++q) v = (lane16 == q) ? lv[q] : v;
    if (lane16 < (1 << K)) sLevel[rloc][lane16] = v;
  }
  if (valid && lane16 <= K) {
    float v = c[0];
#pragma unroll
    for (int i = 1; i <= K; ++i) v = (lane16 == i) ? c[i] : v;
    coefs[((long)lane16 * d_out + row) * n_grp + gi] = v;
  }
  __syncthreads();
  for (int idx = tid; idx < G * kCommitRows / 4; idx += kCommitThreads) {
    const int j = idx / (kCommitRows / 4), r = 4 * (idx % (kCommitRows / 4));
    *reinterpret_cast<float4*>(Eblk + (long)(s0 - b0 + j) * lde + row0 + r) =
        make_float4(sE[j][r], sE[j][r + 1], sE[j][r + 2], sE[j][r + 3]);
  }
  if (W_hat) {
    typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));      // (W_hat need not be aligned to 16 bytes)
    for (int idx = tid; idx < G * kCommitRows / 4; idx += kCommitThreads) {
      const int r = idx / (G / 4), x = 4 * (idx % (G / 4));
      if (row0 + r >= d_out) break;                      // (later ones are further rows)
      const uint32_t four = *reinterpret_cast<const uint32_t*>(&sCode[r][x]);
      f4_any v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = sLevel[r][(four >> (8 * e)) & 15u];
      *reinterpret_cast<f4_any*>(W_hat + (long)(row0 + r) * d_in + s0 + x) = v;
    }
  }
}

// ------------------------------------------------------------------ host side --------------
struct QuantLayout {
  size_t wp_off, eall_off, codes_off, coef_off, e_off, score_off, rec_off, total;
  int rec_floats;       // floats of a group's record (SuLayout::record_floats)
  int B, lde, n_wg;
};

static inline QuantLayout quant_layout(int d_out, int d_in, const bpdq_params& p) {
  QuantLayout L;
  const int g = p.group, T = p.refine_iters, K = p.bits;
  L.B = p.block > g ? p.block : g;
  L.lde = (int)bpdq_align_up((size_t)d_out, 64);
  L.n_wg = bpdq_ceil_div(d_out, kRowsPerWG);
  size_t off = 0;
  L.wp_off = off;    off += bpdq_align_up((size_t)d_out * d_in * sizeof(float), 256);
  L.eall_off = off;  off += bpdq_align_up((size_t)d_in * L.lde * sizeof(float), 256);
  L.codes_off = off; off += bpdq_align_up((size_t)(T + 1) * d_out * 16 * (g > 128 ? 2 : 1) * sizeof(uint32_t), 256);
  L.coef_off = off;  off += bpdq_align_up((size_t)(T + 1) * d_out * (K + 1) * sizeof(float), 256);
  L.e_off = off;     off += bpdq_align_up((size_t)(T + 1) * d_out * g * sizeof(float), 256);
  L.score_off = off; off += bpdq_align_up((size_t)(T + 1) * L.n_wg * sizeof(double), 256);
  L.rec_floats = g == 32 ? SuLayout<32>::record_floats() : g == 64 ? SuLayout<64>::record_floats()
                 : g == 128 ? SuLayout<128>::record_floats() : SuLayout<256>::record_floats();
  L.rec_off = off;   off += (size_t)(d_in / g) * L.rec_floats * sizeof(float);
  L.total = off;
  return L;
}

// the tail role as a kernel of its own (defined with the host loop)
int launch_tail_update(hipStream_t stream, TailArgs ta, const float* U, int ldu, int lde, int ldw,
                       int d_out, int n_tiles);

template <int G>
constexpr size_t sweep_lds_bytes() {
  const size_t a = (kStageFloats<G> + kScratchFloats<G> + 4 * kSolveFloats) * sizeof(float);
  return a < TailGemm::kLdsBytes ? TailGemm::kLdsBytes : a;
}

// launch of the fixed-grid comparator's sweep kernel
struct UniformSweepArgs {
  hipStream_t stream;
  int grid;
  const float* Wp;
  int d_in, d_out;
  const float* U;
  const float* rec;
  int s0, coef_fp16;
  uint32_t* c_codes;
  float* c_coef;
  float* c_E;
  double* c_score;
  int n_wg;
  const float* Eall;
  int lde, kp0;
  TailArgs ta;
};

template <int K, int G>
static inline int launch_uniform_sweep(const UniformSweepArgs& a) {
  const size_t lds = sweep_lds_bytes<G>();
  BPDQ_HIP_TRY((bpdq_lds_limit<&uniform_group_kernel<K, G>>(lds)));
  hipLaunchKernelGGL((uniform_group_kernel<K, G>), dim3(a.grid), dim3(kSweepThreads), lds, a.stream,
                     a.Wp, a.d_in, a.d_out, a.U, a.d_in, a.rec, a.s0, a.coef_fp16, a.c_codes, a.c_coef, a.c_E,
                     a.c_score, a.n_wg, a.Eall, a.lde, a.kp0, a.ta);
  BPDQ_LAUNCH_CHECK();
  return 0;
}
// group size 256: defined in group_sweep_k{K}_g256u.hip (the two g = 256 kernels of a plane count
// are the longest compilations of the build; apart they run in parallel)
template <int K>
int launch_uniform_sweep_256(const UniformSweepArgs& a);

// One group: the sweep kernel (with the pending updates read left-looking from column kp0 on, and
// the tail role `ta` for the previous block, see above), then selection + commit.
template <int K, int G>
static inline int launch_group(hipStream_t stream, const float* Wp, int d_out, int d_in, const float* U,
                        int s0, int kp0, TailArgs ta, const SegArgs& seg, const bpdq_params& p,
                        const QuantLayout& L, char* base, uint32_t* planes, float* coefs,
                        float* W_hat, double* grp_err, int* grp_iter) {
  uint32_t* c_codes = reinterpret_cast<uint32_t*>(base + L.codes_off);
  float* c_coef = reinterpret_cast<float*>(base + L.coef_off);
  float* c_E = reinterpret_cast<float*>(base + L.e_off);
  double* c_score = reinterpret_cast<double*>(base + L.score_off);
  float* Eall = reinterpret_cast<float*>(base + L.eall_off);
  const size_t lds = sweep_lds_bytes<G>();
  const int gi = s0 / G;
  const float* rec = reinterpret_cast<const float*>(base + L.rec_off) + (long)gi * L.rec_floats;
  const bool uniform = (p.grid == BPDQ_GRID_UNIFORM);
  const int T = uniform ? 0 : p.refine_iters;
  ta.first_wg = L.n_wg;
  const int row_tiles = bpdq_ceil_div(L.lde, TailGemm::kTileM);
  ta.far_wgs = row_tiles * ta.far.tiles_n;
  int n_tail = row_tiles * (ta.far.tiles_n + ta.near.tiles_n);
  if (!kTailInSweep<G> && n_tail > 0) {
    const int rc = launch_tail_update(stream, ta, U, d_in, L.lde, d_in, d_out, n_tail);
    if (rc) return rc;
    n_tail = 0;
  }
  const int grid = L.n_wg + n_tail;
  if (uniform) {
    const UniformSweepArgs a{stream, grid, Wp, d_in, d_out, U, rec, s0, p.coef_fp16, c_codes, c_coef, c_E,
                             c_score, L.n_wg, Eall, L.lde, kp0, ta};
    int rc;
    if constexpr (G >= 256) rc = launch_uniform_sweep_256<K>(a);   // a translation unit of its own
    else rc = launch_uniform_sweep<K, G>(a);
    if (rc) return rc;
  } else {
    BPDQ_HIP_TRY((bpdq_lds_limit<&bpdq_group_kernel<K, G>>(lds)));
    hipLaunchKernelGGL((bpdq_group_kernel<K, G>), dim3(grid), dim3(kSweepThreads), lds, stream,
                       Wp, d_in, d_out, U, d_in, rec, s0, T, p.alpha, p.coef_fp16, c_codes, c_coef, c_E, c_score,
                       L.n_wg, Eall, L.lde, kp0, ta);
  }
  BPDQ_LAUNCH_CHECK();
  hipLaunchKernelGGL((commit_group_kernel<K, G>), dim3(L.lde / kCommitRows), dim3(kCommitThreads), 0, stream,
                     c_codes, c_coef, c_E, c_score, L.n_wg, T, seg, grp_err + gi, grp_iter + gi, d_out,
                     d_in, s0, 0, planes, coefs, W_hat, Eall, L.lde);
  BPDQ_LAUNCH_CHECK();
  return 0;
}

typedef int (*GroupLauncher)(hipStream_t, const float*, int, int, const float*, int, int, TailArgs,
                             const SegArgs&, const bpdq_params&, const QuantLayout&, char*, uint32_t*,
                             float*, float*, double*, int*);

// The group kernels are large, fully unrolled kernels: one translation unit per plane count
// instantiates group sizes 32 / 64 / 128, and two more per plane count (1..3) group size 256
// (variable grid, fixed grid), which keeps the build parallel.  Four planes at g = 256 -- a
// combination the paper does not use -- would by itself double the build time and is left out.
GroupLauncher pick_group_k1(int g);
GroupLauncher pick_group_k2(int g);
GroupLauncher pick_group_k3(int g);
GroupLauncher pick_group_k4(int g);
GroupLauncher group256_k1();
GroupLauncher group256_k2();
GroupLauncher group256_k3();

template <int K>
static inline GroupLauncher pick_group_g(int g) {
  switch (g) {
    case 32: return launch_group<K, 32>;
    case 64: return launch_group<K, 64>;
    case 128: return launch_group<K, 128>;
  }
  return nullptr;
}
}  // namespace bpdq
