// Step 2 of the pass: damping and U = chol(H^-1), H^-1 = U^T U with U upper triangular
// (paper Sec. 3.1, "Quantization Error Compensation").
//
// Route: with Ht = H + lambda I, factor Ht = R R^T with R UPPER triangular (a Cholesky
// factorisation that runs from the last column to the first).  Then
// Ht^-1 = R^-T R^-1 = (R^-1)^T (R^-1), so U = R^-1: one factorisation plus one triangular
// inverse (2/3 d^3 flops) and Ht^-1 is never formed.  Everything runs in fp64 inside the
// workspace; the result is rounded to fp32 once, on output.
//
// Two ways to do it.  From 65 to 12288 columns the factor and its inverse in one sweep over pairs of 64-column panels from
// the right (prepare_by_pairs): while a pair is factored by a few work-groups, the others of the same launch update what
// the next pairs need only later and build the rows of the inverse behind it (3584 columns: 1939 -> 1245 us; 8192: 9996
// -> 8095).  Otherwise, and with a workspace of only the size that this needs, the factor first and then the inverse:
//   factor : right-looking over 64-column panels from the right, two panels per launch: every
//            panel work-group factors the two diagonal blocks for itself (in LDS, by panels of
//            16 columns) and solves its 64 rows of R12 R22^T = A12.  The trailing update
//            A11 -= R12 R12^T (fp64 MFMA) is two-level: after each panel pair only inside the
//            current 512-column outer block (64 x 64 tiles), and once per outer block, with
//            K = 512, on everything to its left (128 x 128 tiles fed by LDS-DMA from 4096
//            columns on).
//   invert : divide and conquer over block ranges, [R11 R12; 0 R22]^-1 =
//            [U11, -U11 R12 U22; 0, U22]; every tree level is two launches (128 x 128 tiles
//            where a level has enough of them, 64 x 64 otherwise).
// Both tile sizes stream their operands by LDS-DMA; widths that are odd (trailing updates) or not a
// multiple of 64 (inversion) take 64 x 64 tiles staged through registers.
#include <type_traits>

#include "common.h"

namespace bpdq {

constexpr int NB = 64;    // panel / tile size (fp64)

// ---------------------------------------------------------------- damping ------------------
// One work-group: dead flags, mean of the (fixed) diagonal, lambda.  scal[0] = lambda.
__global__ __launch_bounds__(1024) void prep_diag_kernel(const float* __restrict__ H, int d,
                                                         float damp, unsigned char* __restrict__ dead,
                                                         double* __restrict__ scal, int* info) {
  __shared__ double red[1024];
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 1024) {
    float h = H[(long)i * d + i];
    const bool dd = (h == 0.f);
    if (dead) dead[i] = dd ? 1 : 0;
    s += dd ? 1.0 : (double)h;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    scal[0] = (double)damp * (red[0] / (double)d);
    *info = 0;
  }
}

// A (fp64, d x d) <- upper triangle of H with the diagonal fixed and damped, one 64 x 64 block per
// work-group; blocks below the diagonal are neither written nor ever read.  Bound by HBM (no division per
// element, half of the stores: 24 -> 17 us at d = 3584, 181 -> 72 us at 8192).
// ld > d: A is padded with the identity to ld x ld.  U: zeros below the diagonal blocks go there at once (U may be H: the
// blocks below the diagonal are not read).
__global__ __launch_bounds__(256) void prep_load_kernel(const float* H, int d,
                                                        const double* __restrict__ scal,
                                                        double* __restrict__ A, int ld, float* U) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj < bi) {
    if (!U) return;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int i = bi * NB + (threadIdx.x >> 6) + 4 * t, j = bj * NB + (threadIdx.x & 63);
      if (i < d && j < d) U[(long)i * d + j] = 0.f;
    }
    return;
  }
  const double lam = scal[0];
  const int j = bj * NB + (threadIdx.x & 63), i0 = bi * NB + (threadIdx.x >> 6);
  float h[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = i0 + 4 * t;
    h[t] = H[(i < d && j < d) ? (long)i * d + j : 0L];
  }
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = i0 + 4 * t;
    if (i >= ld || j >= ld) continue;
    double v = (j >= i) ? (double)h[t] : 0.0;
    if (i == j) v = (h[t] == 0.f ? 1.0 : v) + lam;
    if (i >= d || j >= d) v = (i == j) ? 1.0 : 0.0;
    A[(long)i * ld + j] = v;
  }
}

// ---------------------------------------------------------------- factor -------------------
// 1 / x in fp64: hardware estimate (about 2^-27 relative) + one Newton step (about 2^-52): the
// pivot reciprocal sits on the critical path of every column step, where every dependent fp64
// operation costs tens of cycles; an error of an ulp or two in it is far below the fp32 rounding
// of H and of the result.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// 1 / sqrt(x) in fp64: hardware estimate and one third-order step, an ulp or two
__device__ __forceinline__ double fast_rsqrt(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * r, r, 1.0);
  return fma(r, e * fma(0.375, e, 0.5), r);
}

// A 64 x 64 tile of doubles moves between global memory and LDS through registers, 16 elements
// per thread of 256 (element e = tid + 256 t -> row e / 64, column e % 64).  All 16 loads of a
// thread are issued before the first is used: a rolled loop would wait for memory 16 times.
// ok(i, j): is the element read (else 0);  idx(i, j): its offset from `base`, which must itself
// be a valid address (masked elements read base[0] and discard it).
// (Work-groups of 512 threads are two teams of 256 on tiles of their own: team_tid and team_wave.)
__device__ __forceinline__ int team_tid() { return threadIdx.x & 255; }
__device__ __forceinline__ int team_wave() { return (threadIdx.x >> 6) & 3; }
__device__ __forceinline__ int team_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 8); }

template <typename OK, typename IDX>
__device__ __forceinline__ void fetch_tile64(const double* __restrict__ base, OK ok, IDX idx,
                                             double (&v)[16]) {
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int e = team_tid() + 256 * t;
    const int i = e >> 6, j = e & 63;
    const bool in = ok(i, j);
    const double x = base[in ? idx(i, j) : 0L];
    v[t] = in ? x : 0.0;
  }
}
template <typename ROW>
__device__ __forceinline__ void put_tile64(ROW* s, const double (&v)[16]) {
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int e = team_tid() + 256 * t;
    s[e >> 6][e & 63] = v[t];
  }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// value of lane J of this lane's 16-lane row, in every lane of the row (one v_mov_b64_dpp)
template <int J>
__device__ __forceinline__ double row_bcast(double x) {
  return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + J, 0xF, 0xF, true);
}

typedef double Inv16[16][16];

// Elimination of column J of a 16 x 16 symmetric block and of its companion W (at first the identity).
// Lane i % 16 = row i holds the block's row in a[0..15]; all four 16-lane rows hold the same block, and
// row q of them the columns 4 ks + q of W in w[ks].  With t_i = A_iJ / A_JJ the rows above J lose t_i
// times row J; only the reciprocal's chain (about six dependent fp64 operations) is serial, the
// broadcasts of row J do not wait for it.
// A pivot that is not positive is replaced by 1; row i keeps its own as it came (raw_own), so that the caller can tell.
// The broadcast is an operand of the multiply-add (v_fmac_f64_dpp, which the compiler does not form: a move and a
// multiply-add each were 30 instructions a column, now about 22; every one takes a wavefront alone about eight cycles).
// A DPP operand must be two instructions old, and the compiler does not look into assembly: the entry the next
// column's pivot is read from is followed by the wait, every other one by more than two instructions.
template <int J, bool WAIT>
__device__ __forceinline__ void fmac_bcast(double& x, double t) {      // x -= t (x of lane J of the 16-lane row)
  if constexpr (WAIT)
    asm volatile("v_fmac_f64_dpp %0, %0, -%1 row_newbcast:%2 row_mask:0xf bank_mask:0xf\n\ts_nop 1" : "+v"(x) : "v"(t), "n"(J));
  else
    asm volatile("v_fmac_f64_dpp %0, %0, -%1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(x) : "v"(t), "n"(J));
}
template <int J>
__device__ __forceinline__ void eliminate16(double (&a)[16], double (&w)[4], double& raw_own, int i) {
  if constexpr (J == 15) {                  // the loaded and selected values stand two instructions before their first use
    asm volatile("s_nop 1"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]), "+v"(a[8]),
                   "+v"(a[9]), "+v"(a[10]), "+v"(a[11]), "+v"(a[12]), "+v"(a[13]), "+v"(a[14]));
    asm volatile("s_nop 1" : "+v"(a[15]), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]));
  }
  const double piv_raw = row_bcast<J>(a[J]);
  if (i == J) raw_own = piv_raw;
  const double r = fast_rcp(piv_raw);       // the test of the pivot runs beside the reciprocal's chain
  const double t = a[J] * (piv_raw > 0.0 ? r : 1.0);
  const double tm = (i < J) ? t : 0.0;
  if constexpr (J > 0) fmac_bcast<J, true>(a[J - 1], t);
#pragma unroll
  for (int e = J - 2; e >= 0; --e) fmac_bcast<J, false>(a[e], t);
#pragma unroll
  for (int ks = J / 4; ks < 4; ++ks) fmac_bcast<J, false>(w[ks], tm);  // columns left of J are still zero in row J
  if constexpr (J > 0) eliminate16<J - 1>(a, w, raw_own, i);
}

// a[e] *= (value of `s` in lane e of the 16-lane row), e = E .. 0
template <int E>
__device__ __forceinline__ void scale_columns16(double (&a)[16], double s) {
  a[E] *= row_bcast<E>(s);
  if constexpr (E > 0) scale_columns16<E - 1>(a, s);
}

// Reversed Cholesky of one 64 x 64 block held in LDS: D = R R^T, R upper, columns taken from the
// last to the first, in panels of 16 columns.
//   in : sD, the upper triangle of the block (identity padding where the block is ragged)
//   out: sD = R on and above the diagonal (undefined below it), sRinv[J] = (R_JJ)^-1 of the four
//        16 x 16 diagonal blocks (zero below the diagonal)
// The 16 x 16 diagonal block of a panel is eliminated in registers by every wavefront for itself, one
// 16-lane row of the wavefront holding the block (row broadcasts are single DPP moves), together with its
// inverse.  The inverse comes out in the operand layout of the fp64 matrix instruction, so the rest of the
// panel, X = A R_JJ^-T, and the update of the columns to its left, -= X X^T, are matrix products on the
// upper 16 x 16 tiles.  Per panel: one chain of 16 columns of about 120 cycles each and two barriers.
// (One wavefront with lane = row of the whole panel, its pivot columns going through LDS, took 430
// cycles a column, and the inverses a pass of their own: a panel pair 52 -> 40 us at d = 3584.)
// A non-positive pivot is reported as column p0 + j + 1 (by the work-group with `report`) and
// replaced by 1.  All 256 threads call this; it begins and ends with a barrier.
//
// `idle`: of a 512-thread work-group one team factors (active), the other keeps the barriers company and does work of
// its own between them, idle(integral_constant<int, n>), n = 0 .. 7: the odd ones are the short intervals.
struct NoWork {
  template <typename N>
  __device__ __forceinline__ void operator()(N) const {}
};
template <typename IDLE = NoWork>
__device__ __forceinline__ void factor64_blocked(double (*sD)[NB + 1], Inv16* sRinv, int* info, int p0, bool report,
                                                 bool active = true, IDLE idle = IDLE{}) {
  if (!active) {
    auto wait = [&](auto n) {
      __syncthreads();
      idle(n);
    };
    wait(std::integral_constant<int, 0>{}); wait(std::integral_constant<int, 1>{});
    wait(std::integral_constant<int, 2>{}); wait(std::integral_constant<int, 3>{});
    wait(std::integral_constant<int, 4>{}); wait(std::integral_constant<int, 5>{});
    wait(std::integral_constant<int, 6>{}); wait(std::integral_constant<int, 7>{});
    __syncthreads();
    return;
  }
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(team_wave());
  const int m = lane & 15, q = lane >> 4;
  int off[16];                              // element (m, e) of a diagonal block, from its upper triangle
#pragma unroll
  for (int e = 0; e < 16; ++e) off[e] = (m < e) ? m * (NB + 1) + e : e * (NB + 1) + m;
#pragma unroll 1
  for (int J = NB / 16 - 1; J >= 0; --J) {
    const int c0 = 16 * J;
    __syncthreads();                        // the block, with every earlier panel's update, is in LDS
    double a[16], wi[4], raw = 1.0, at[4];
#pragma unroll
    for (int e = 0; e < 16; ++e) a[e] = (&sD[c0][c0])[off[e]];
    if (w < J) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) at[ks] = sD[16 * w + m][c0 + 4 * ks + q];     // A operand of row tile w
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) wi[ks] = (m == 4 * ks + q) ? 1.0 : 0.0;
    eliminate16<15>(a, wi, raw, m);
    const bool bad = !(raw > 0.0);          // the pivot of row j = m
    const unsigned bad_rows = (unsigned)__builtin_amdgcn_ballot_w64(bad) & 0xffffu;
    const double inv_d = fast_rsqrt(bad ? 1.0 : raw);      // 1 / R_jj
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) wi[ks] *= inv_d;                                // R_JJ^-1 [m][4 ks + q]
    if (w == 3) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) sRinv[J][m][4 * ks + q] = wi[ks];
    }
    if (bad_rows && report && w == 0 && lane == 0)         // the first one met: the rest stands on replaced pivots
      atomicCAS(info, 0, p0 + c0 + 32 - __builtin_clz(bad_rows));
    if (w < J) {                            // X = A R_JJ^-T, row tile w
      f64x4 x[2] = {(f64x4){0.0, 0.0, 0.0, 0.0}, (f64x4){0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) x[ks & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(at[ks], wi[ks], x[ks & 1], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sD[16 * w + 4 * r + q][c0 + m] = x[0][r] + x[1][r];
    }
    __syncthreads();
    // (after the barrier: every wavefront has read the diagonal block)
    if (w == 3 && q == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const double sc = (m <= e) ? a[e] : 0.0;
        a[e] = sc;
      }
      scale_columns16<15>(a, inv_d);
#pragma unroll
      for (int e = 0; e < 16; ++e) sD[c0 + m][c0 + e] = a[e];
    }
    // the tiles to the left, the next panel's first; a wavefront's two are in flight together
    auto tile_of = [&](int t, int& ti, int& tk) {
      tk = J - 1;
      while (tk > 0 && t > tk) { t -= tk + 1; --tk; }
      ti = tk - t;
    };
    const int n_tiles = J * (J + 1) / 2;
    if (w < n_tiles) {
      const bool two = w + 4 < n_tiles;
      int ti[2], tk[2];
      tile_of(w, ti[0], tk[0]);
      tile_of(two ? w + 4 : w, ti[1], tk[1]);
      double xi[2][4], xk[2][4], old[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          xi[u][ks] = sD[16 * ti[u] + m][c0 + 4 * ks + q];
          xk[u][ks] = sD[16 * tk[u] + m][c0 + 4 * ks + q];
          old[u][ks] = sD[16 * ti[u] + 4 * ks + q][16 * tk[u] + m];
        }
      __builtin_amdgcn_sched_barrier(0);
      f64x4 acc[2][2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[u][h] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        acc[0][ks & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[0][ks], xk[0][ks], acc[0][ks & 1], 0, 0, 0);
      if (two)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          acc[1][ks & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[1][ks], xk[1][ks], acc[1][ks & 1], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (u == 0 || two) {
#pragma unroll
          for (int r = 0; r < 4; ++r) sD[16 * ti[u] + 4 * r + q][16 * tk[u] + m] = old[u][r] - (acc[u][0][r] + acc[u][1][r]);
        }
    }
  }
  __syncthreads();
}

// X R^T = A for a 64 x 64 tile, in place, by blocks of 16 columns from the right (R upper, sRinv =
// inverses of its 16 x 16 diagonal blocks), all on the fp64 matrix cores (v_mfma_f64_16x16x4_f64):
//   (1) X_J = A_J R_JJ^-T;
//   (2) the blocks to its left receive  A_J' -= X_J R[J', J]^T.
// Wavefront w of the team takes rows 16 w .. 16 w + 15 through all four blocks; a row block never
// meets another one's data, so there is no barrier inside and no dependent substitution chain (a
// column-by-column substitution took 7 us a solve instead of 2).  The caller puts a barrier behind it.
// What is not solved yet stays in registers (acc, the layout of the result), the operands of a step are requested
// before its first product.

// LDS serves a wavefront in order, so what one lane wrote another lane of it may read without a barrier; but the compiler,
// which looks at one lane's addresses only, has to be kept from moving the reads over the writes.
__device__ __forceinline__ void in_wave_order() { asm volatile("" ::: "memory"); }

template <int J>
__device__ __forceinline__ void trsm_block_step(f64x4 (&acc)[4], double (*sX)[NB + 1], const double (*sR)[NB + 1], const Inv16* sRinv) {
  const int lane = threadIdx.x & 63, i0 = 16 * team_wave();
  const int lm = lane & 15, lq = lane >> 4;
  double a[4], ri[4], rb[J > 0 ? J : 1][4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    ri[ks] = sRinv[J][lm][4 * ks + lq];
#pragma unroll
    for (int Jp = 0; Jp < J; ++Jp) rb[Jp][ks] = sR[16 * Jp + lm][16 * J + 4 * ks + lq];
  }
  if constexpr (J < 3) {
#pragma unroll
    for (int r = 0; r < 4; ++r) sX[i0 + 4 * r + lq][16 * J + lm] = acc[J][r];
  }
  in_wave_order();
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) a[ks] = sX[i0 + lm][16 * J + 4 * ks + lq];
  f64x4 x[2] = {(f64x4){0.0, 0.0, 0.0, 0.0}, (f64x4){0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)                                                    // A[m][k] = A_J, B[k][n] = Rinv[n][k]
    x[ks & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], ri[ks], x[ks & 1], 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) sX[i0 + 4 * r + lq][16 * J + lm] = x[0][r] + x[1][r];  // D[4r + l/16][l%16]
  in_wave_order();
  if constexpr (J > 0) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[ks] = -sX[i0 + lm][16 * J + 4 * ks + lq];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int Jp = J - 1; Jp >= 0; --Jp)                                           // B[k][n] = R[J'n][Jk]
        acc[Jp] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], rb[Jp][ks], acc[Jp], 0, 0, 0);
  }
}
__device__ __forceinline__ void trsm_load(f64x4 (&acc)[4], const double (*sX)[NB + 1]) {
  const int lane = threadIdx.x & 63, i0 = 16 * team_wave();
#pragma unroll
  for (int Jp = 0; Jp < 3; ++Jp)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[Jp][r] = sX[i0 + 4 * r + (lane >> 4)][16 * Jp + (lane & 15)];
}
__device__ __forceinline__ void trsm64_blocked(double (*sX)[NB + 1], const double (*sR)[NB + 1], const Inv16* sRinv) {
  f64x4 acc[4];
  trsm_load(acc, sX);
  trsm_block_step<3>(acc, sX, sR, sRinv);
  trsm_block_step<2>(acc, sX, sR, sRinv);
  trsm_block_step<1>(acc, sX, sR, sRinv);
  trsm_block_step<0>(acc, sX, sR, sRinv);
}

// 64 x 64 tile at (r0, c0) of A, `nr` x `nc` of it inside (identity padding where `diag`, else zeros), 16
// elements per thread of a team in the order of put_tile: pairs of columns (16-byte loads) where `vec`, which
// needs a full tile and an even d.  Below the diagonal of A there are zeros or nothing of meaning.
__device__ __forceinline__ void fetch_tile(const double* __restrict__ A, int d, int r0, int c0, int nr, int nc,
                                           bool diag, bool vec, double (&v)[16]) {
  if (vec) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = team_tid() + 256 * t;
      const double2 x = *reinterpret_cast<const double2*>(A + (long)(r0 + (e >> 5)) * d + c0 + 2 * (e & 31));
      v[2 * t] = x.x;
      v[2 * t + 1] = x.y;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int e = team_tid() + 256 * t;
      const int i = e >> 6, j = e & 63;
      const bool in = i < nr && j < nc;
      const double x = A[in ? (long)(r0 + i) * d + c0 + j : 0L];
      v[t] = in ? x : ((diag && i == j) ? 1.0 : 0.0);
    }
  }
}
template <typename ROW>
__device__ __forceinline__ void put_tile(ROW* s, bool vec, const double (&v)[16]) {
  if (vec) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int e = team_tid() + 256 * t;
      s[e >> 5][2 * (e & 31)] = v[2 * t];
      s[e >> 5][2 * (e & 31) + 1] = v[2 * t + 1];
    }
  } else {
    put_tile64(s, v);
  }
}

// Panel step of the reversed Cholesky for ONE 64-column panel, one work-group (256 threads) per
// 64 rows of the panel.
//   (1) every work-group factors the 64 x 64 diagonal block for itself (factor64_blocked);
//   (2) rows [64 b, 64 b + 64) of the panel above the block: X R^T = A12 (trsm64_blocked).
// Work-group 0 also writes R of the diagonal block to Rdiag (NB x NB, row-major, zero below the
// diagonal, identity-padded), clears the block's pair flag and reports a non-positive pivot.
// Launch with max(p, 1) work-groups, p = number of 64-row blocks above the diagonal block.
__global__ __launch_bounds__(256) void panel_factor_kernel(double* __restrict__ A, int d, int p0,
                                                           int nb, int n_above,
                                                           double* __restrict__ Rdiag,
                                                           int* __restrict__ pair_flag, int* info) {
  __shared__ double sR[NB][NB + 1];     // R (upper) of the diagonal block
  __shared__ double sA[NB][NB + 1];     // panel tile of this work-group
  __shared__ Inv16 sRinv[NB / 16];
  const int tid = threadIdx.x;

  {
    double v[16];
    fetch_tile(A, d, p0, p0, nb, nb, true, false, v);
    put_tile(sR, false, v);
  }
  // panel tile (coalesced), used after the factorisation
  const int r0 = blockIdx.x * NB;
  if (n_above > 0) {
    double v[16];
    fetch_tile64(A, [&](int i, int j) { return r0 + i < p0 && j < nb; },
                 [&](int i, int j) { return (long)(r0 + i) * d + p0 + j; }, v);
    put_tile64(sA, v);
  }
  factor64_blocked(sR, sRinv, info, p0, blockIdx.x == 0);
  // R of the diagonal block goes to its own buffer: the block itself must stay untouched, because
  // work-groups of this launch that start later still have to read it
  if (blockIdx.x == 0) {
    for (int e = tid; e < NB * NB; e += 256) Rdiag[e] = sR[e / NB][e % NB];
    if (tid == 0) *pair_flag = 0;
  }
  if (n_above == 0) return;
  trsm64_blocked(sA, sR, sRinv);
  __syncthreads();
  for (int e = tid; e < NB * NB; e += 256) {
    const int i = e / NB, j = e % NB;
    if (r0 + i < p0 && j < nb) A[(long)(r0 + i) * d + p0 + j] = sA[i][j];
  }
}

// V = R^-1 of one 64 x 64 upper triangular block in LDS, by 16 x 16 blocks: the diagonal ones by back
// substitution (wavefront = block, lane = column), then one block diagonal after the other on the fp64
// matrix cores, V_IJ = -V_II sum_{I < K <= J} R_IK V_KJ; the sum leaves the matrix instruction in the
// layout in which the second product reads it.  All 256 threads; begins and ends with a barrier.
// (A thread per column with a dot product per element took 40 us of the launch.)
__device__ __forceinline__ void invert64(const double (*sR)[NB + 1], double (*sV)[NB + 1]) {
  const int lane = threadIdx.x & 63, w = team_wave();
  const int m = lane & 15, q = lane >> 4;
  __syncthreads();
  if (lane < 16) {
    const int c = lane, o = 16 * w;
    double x[16];
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      double acc = 0.0;
#pragma unroll
      for (int k = 15; k > i; --k) acc = fma(sR[o + i][o + k], x[k], acc);     // x[k] = 0 for k > c
      x[i] = (i <= c) ? ((i == c) ? 1.0 : -acc) / sR[o + i][o + i] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) sV[o + i][o + c] = x[i];
  }
  for (int dist = 1; dist < NB / 16; ++dist) {
    __syncthreads();
    const int I = w, J = w + dist;
    if (J < NB / 16) {
      f64x4 t = (f64x4){0.0, 0.0, 0.0, 0.0}, v = t;
      for (int K = I + 1; K <= J; ++K)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          t = __builtin_amdgcn_mfma_f64_16x16x4f64(sR[16 * I + m][16 * K + 4 * ks + q], sV[16 * K + 4 * ks + q][16 * J + m],
                                                   t, 0, 0, 0);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        v = __builtin_amdgcn_mfma_f64_16x16x4f64(sV[16 * I + m][16 * I + 4 * ks + q], t[ks], v, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sV[16 * I + 4 * r + q][16 * J + m] = -v[r];
    }
  }
  __syncthreads();
}

// Inverses of all diagonal blocks of R at once, one work-group per block; the inverse replaces the
// diagonal block of A (upper part, zeros below), which until now still held the unfactored block.  A
// block that was the second of a panel pair also brings its R12 (rows of the block before it) from the
// side buffer into A.
__global__ __launch_bounds__(256) void diag_inverse_kernel(const double* __restrict__ Rdiag,
                                                           const double* __restrict__ R12buf,
                                                           const int* __restrict__ pair_flag,
                                                           double* __restrict__ A, int d) {
  __shared__ double s[NB][NB + 1];
  __shared__ double x[NB][NB + 1];
  const int p0 = blockIdx.x * NB;
  const int nb = (d - p0 < NB) ? d - p0 : NB;
  const int tid = threadIdx.x;
  const double* src = Rdiag + (long)blockIdx.x * NB * NB;
  const bool pair = pair_flag[blockIdx.x] != 0;
  {
    double v[16], r12[16];
    fetch_tile64(src, [](int, int) { return true; }, [](int i, int j) { return (long)i * NB + j; }, v);
    if (pair)
      fetch_tile64(R12buf + (long)blockIdx.x * NB * NB, [](int, int) { return true; },
                   [](int i, int j) { return (long)i * NB + j; }, r12);
    put_tile64(s, v);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int e = tid + 256 * t;
      const int i = e >> 6, j = e & 63;
      if (pair && j < nb) A[(long)(p0 - NB + i) * d + p0 + j] = r12[t];
    }
  }
  invert64(s, x);
  for (int e = tid; e < NB * NB; e += 256) {
    const int i = e / NB, j = e % NB;
    if (i < nb && j < nb) A[(long)(p0 + i) * d + p0 + j] = (j >= i) ? x[i][j] : 0.0;
    // the block to the left of the diagonal one: the 128-tile products of the inversion read it as
    // part of a triangular operand, where it stands for zeros
    if (p0 > 0 && i < nb) A[(long)(p0 + i) * d + p0 - NB + j] = 0.0;
  }
}

// 64 x 64 x 64 fp64 product on the matrix cores for a 256-thread work-group: wavefront w owns
// the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 tiles of v_mfma_f64_16x16x4_f64.
//   A operand: lane l holds A[m = l % 16][k = l / 16];  B operand: B[k = l / 16][n = l % 16];
//   D: register r of lane l is D[4 * r + l / 16][l % 16].
// sa is [m][k]; sb is [k][n], or [n][k] when B_T (second operand given by rows, as in a SYRK).
// With the 65-double row pitch every 16-lane group reads 16 distinct bank pairs.
struct Quad64 {
  f64x4 c[2][2];
};

__device__ __forceinline__ void quad_zero(Quad64& q) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) q.c[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
}

template <bool B_T, int K0 = 0, int K1 = NB>
__device__ __forceinline__ void quad_mfma_64(const double (*sa)[NB + 1], const double (*sb)[NB + 1],
                                             Quad64& q) {
  const int lane = threadIdx.x & 63, w = team_wave();
  const int m0 = (w >> 1) * 32 + (lane & 15), n0 = (w & 1) * 32 + (lane & 15);
  const int kq = lane >> 4;
#pragma unroll 4
  for (int k0 = K0; k0 < K1; k0 += 4) {
    const int k = k0 + kq;
    double a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = sa[m0 + 16 * i][k];
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = B_T ? sb[n0 + 16 * j][k] : sb[k][n0 + 16 * j];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        q.c[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], q.c[i][j], 0, 0, 0);
  }
}

// f(row, col, value) over this lane's 16 results, row / col inside the 64 x 64 tile
template <typename F>
__device__ __forceinline__ void quad_for_each(const Quad64& q, F f) {
  const int lane = threadIdx.x & 63, w = team_wave();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        f((w >> 1) * 32 + 16 * i + 4 * r + (lane >> 4), (w & 1) * 32 + 16 * j + (lane & 15),
          q.c[i][j][r]);
}

// Trailing update with the panel columns [k0, k0 + Kd):  A[i][j] -= sum_k A[i][k] A[j][k]  on the
// upper 64 x 64 tiles (bi <= bj) whose block column bj lies in [cb0, cb1).  Used twice:
//   inner: after each 64-column panel, only for the block columns of the same outer panel that
//          are still to be factored (Kd = 64);
//   outer: once per outer panel, for everything to its left (Kd = outer width, up to 512), so
//          the big trailing matrix is read and written 8 times less often.
__global__ __launch_bounds__(256) void syrk_trailing_kernel(double* __restrict__ A, int d, int k0,
                                                            int Kd, int cb0, int cb1) {
  __shared__ double si[NB][NB + 1];
  __shared__ double sj[NB][NB + 1];
  int tile = blockIdx.x, bj = cb0;
  while (tile >= bj + 1) {
    tile -= bj + 1;
    ++bj;
  }
  const int bi = tile;
  const int tid = threadIdx.x;
  const int k_end = (k0 + Kd < d) ? k0 + Kd : d;
  Quad64 q;
  quad_zero(q);
  double vi[16], vj[16];
  auto fetch = [&](int kc) {
    fetch_tile64(A, [&](int, int k) { return kc + k < k_end; },
                 [&](int i, int k) { return (long)(bi * NB + i) * d + kc + k; }, vi);
    fetch_tile64(A, [&](int, int k) { return kc + k < k_end; },
                 [&](int i, int k) { return (long)(bj * NB + i) * d + kc + k; }, vj);
  };
  fetch(k0);
  for (int kc = k0; kc < k_end; kc += NB) {
    put_tile64(si, vi);
    put_tile64(sj, vj);
    __syncthreads();
    if (kc + NB < k_end) fetch(kc + NB);          // in flight during the products below
    quad_mfma_64<true>(si, sj, q);
    __syncthreads();
  }
  // read-modify-write of the 16 results of this lane, all loads first
  double old[16];
  int n = 0;
  quad_for_each(q, [&](int r, int c, double) {
    const int i = bi * NB + r, j = bj * NB + c;
    old[n++] = A[(j >= i) ? (long)i * d + j : 0L];
  });
  n = 0;
  quad_for_each(q, [&](int r, int c, double v) {
    const int i = bi * NB + r, j = bj * NB + c;
    if (j >= i) A[(long)i * d + j] = old[n] - v;
    ++n;
  });
}

// ---- fp64 products on 128 x 128 tiles, operands streamed to LDS by the DMA path -------------
// For the wide layers.  A 64 x 64 tile moves 2 x 64 operand rows per 64 x 64 results, which at
// the fp64 matrix rate is more than the caches deliver, and its loads pass through registers,
// whose address arithmetic and LDS writes sit between the matrix instructions.  Here 256 threads
// own 128 x 128 results, wavefront w the 64 x 64 quadrant (w / 2, w % 2) as 4 x 4 tiles of
// v_mfma_f64_16x16x4_f64, and both operands reach LDS in slices of 16 along K through the LDS-DMA
// path (global_load_lds_dwordx4: 64 lanes x 16 bytes land in 1 KB of LDS, no registers involved),
// double-buffered: the requests for slice s + 1 go out right behind the first operand reads of
// slice s.  64 KB of LDS and fewer than 256 registers: two work-groups per compute unit.
//
// LDS image of a slice of an operand given by rows ([row][k], k contiguous in memory): row r
// (128 bytes = 8 pairs of doubles) keeps pair p at position p ^ ((r / 2) % 8).  The DMA writes
// lane-linear, so the lane that fills position q of row r fetches pair q ^ ((r / 2) % 8).  An
// operand read (16 rows x one column per quarter wave) then touches 16 distinct bank pairs;
// unswizzled, rows 128 bytes apart would share two.
// LDS image of a slice of an operand given as [k][n] (n contiguous): k-row k (1 KB = 64 pairs)
// keeps pair c at position c ^ (8 (k % 2)), so that the two k-rows a half wave reads lie in
// different halves of the banks.
//
// Requirements (the launchers fall back to the 64-tile kernels otherwise): even leading
// dimensions and 16-byte aligned slices; K ranges that are multiples of 32.  Rows (columns) past
// an operand's limit are clamped to a valid one: their products land in results never stored.
constexpr int kGemmTile = 128;
constexpr int kGemmK = 16;
constexpr unsigned kGemmOpBytes = kGemmTile * kGemmK * sizeof(double);       // one operand slice
constexpr unsigned kGemmStageBytes = 2 * kGemmOpBytes;
constexpr size_t kGemmLdsBytes = 2 * kGemmStageBytes;

struct Acc128 {
  f64x4 c[4][4];
};

// 64 lanes x 16 bytes from gptr (per lane) to the 1 KB of LDS at byte address lds_addr (uniform,
// passed in M0, which these kernels use for nothing else).  One outstanding vector-memory operation.  M0 has to be one
// wait state old when the load reads it, and the compiler does not look into assembly: the s_nop.
__device__ __forceinline__ void dma_1k_f64(const double* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(gptr) : "memory");
}
// ... from base (uniform) + off bytes (per lane)
__device__ __forceinline__ void dma_1k(const char* base, unsigned off, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(off), "s"(base) : "memory");
}
__device__ __forceinline__ void wait_all_vm() {
  __builtin_amdgcn_s_waitcnt(0x0070 | 0x0f00);      // vmcnt 0; expcnt / lgkmcnt at their maxima
}

// ... and this wavefront's LDS reads have returned: the slot they read is requested anew behind the barrier that
// follows.  (The compiler moves products over a barrier, and with them the wait for their operands.)
__device__ __forceinline__ void wait_vm_and_reads() {
  asm volatile("" ::: "memory");                    // the reads stay above
  __builtin_amdgcn_s_waitcnt(0x0070);               // vmcnt 0, lgkmcnt 0; expcnt at its maximum
}

// DMA sources of wavefront w for slice 0 of an operand given by rows: rows [32 w, 32 w + 32) of the
// tile that starts at row0, 8 rows per request.
__device__ __forceinline__ void gemm128_row_sources(const double* base, long ld, int row0, int row_limit,
                                                    int k_begin, int w, int lane, const double* (&src)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 32 * w + 8 * j + (lane >> 3);
    const int pair = (lane & 7) ^ ((r >> 1) & 7);
    const int g = (row0 + r < row_limit) ? row0 + r : row_limit - 1;
    src[j] = base + (long)g * ld + k_begin + 2 * pair;
  }
}
// ... of an operand given as [k][n]: k-rows [4 w, 4 w + 4) of the slice, columns [col0, col0 + 128)
__device__ __forceinline__ void gemm128_col_sources(const double* base, long ld, int k_begin, int col0,
                                                    int col_limit, int w, int lane, const double* (&src)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int pair = lane ^ ((j & 1) << 3);                    // (4 w + j) % 2 == j % 2
    const int col = (col0 + 2 * pair < col_limit) ? col0 + 2 * pair : col0;
    src[j] = base + (long)(k_begin + 4 * w + j) * ld + col;
  }
}

// q += A B over n_stage (even) slices.  B_ROWS: B is given by rows like A (C = A B^T, the SYRK
// form), else as [k][n].  step_a / step_b: elements between consecutive slices of a source.
template <bool B_ROWS>
__device__ __forceinline__ void gemm128_accumulate(const double* const (&src_a)[4], const double* const (&src_b)[4],
                                                   long step_a, long step_b, int n_stage, Acc128& q) {
  extern __shared__ __align__(16) double gemm128_lds[];
  typedef __attribute__((address_space(3))) double lds_f64;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned lds0 = (unsigned)(size_t)(lds_f64*)gemm128_lds;
  auto request = [&](int s) {
    const unsigned slot = lds0 + (unsigned)(s & 1) * kGemmStageBytes + (unsigned)w * 4096u;
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_1k_f64(src_a[j] + s * step_a, slot + j * 1024u);
#pragma unroll
    for (int j = 0; j < 4; ++j) dma_1k_f64(src_b[j] + s * step_b, slot + kGemmOpBytes + j * 1024u);
  };
  // operand reads: lane (m = lane % 16, kq = lane / 16) takes column 4 t + kq of rows m + 16 i
  const int l15 = lane & 15, kq = lane >> 4;
  const unsigned sw = (unsigned)((((kq >> 1) ^ (l15 >> 1)) << 4) | ((kq & 1) << 3));
  unsigned a_off[4], b_off[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a_off[t] = ((unsigned)(((w >> 1) * 64 + l15) * 128) + sw) ^ (unsigned)(32 * t);
    b_off[t] = kGemmOpBytes + (((unsigned)(((w & 1) * 64 + l15) * 128) + sw) ^ (unsigned)(32 * t));
  }
  // [k][n] form: byte = 1024 k + 16 (pair ^ 8 (k % 2)) + 8 (n % 2) with k = 4 t + kq, n = 64 (w % 2) + 16 j + m
  const unsigned b_base = kGemmOpBytes + (unsigned)(kq * 1024 + (w & 1) * 512 + l15 * 8);
  const unsigned b_even = b_base + (unsigned)((kq & 1) * 128), b_odd = b_base + (unsigned)(((kq & 1) ^ 1) * 128);
  const char* const lds_bytes = reinterpret_cast<const char*>(gemm128_lds);
  auto compute = [&](unsigned stage_off, int next) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = *reinterpret_cast<const double*>(lds_bytes + stage_off + a_off[t] + i * 2048);
        if constexpr (B_ROWS)
          b[i] = *reinterpret_cast<const double*>(lds_bytes + stage_off + b_off[t] + i * 2048);
        else
          b[i] = *reinterpret_cast<const double*>(lds_bytes + stage_off + ((i & 1) ? b_odd : b_even) + t * 4096 +
                                                  (i >> 1) * 256);
      }
      if (t == 0 && next >= 0) request(next);      // behind the first reads, ahead of the products
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          q.c[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], q.c[i][j], 0, 0, 0);
    }
  };
  if (n_stage <= 0) return;
  request(0);
  for (int s = 0; s < n_stage; s += 2) {
    wait_vm_and_reads();                           // this wavefront's part of slice s has landed, s - 1 is read out
    __builtin_amdgcn_s_barrier();                  // ... everyone's has, and is
    asm volatile("" ::: "memory");
    compute(0u, s + 1);
    wait_vm_and_reads();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    compute(kGemmStageBytes, (s + 2 < n_stage) ? s + 2 : -1);
  }
}

// f(i, j, r, row, col): result register r of tile (i, j) of this lane and where it sits in the 128 x 128 tile
template <typename F>
__device__ __forceinline__ void acc128_for_each_in_row(int i, F f) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      f(j, r, (w >> 1) * 64 + 16 * i + 4 * r + (lane >> 4), (w & 1) * 64 + 16 * j + (lane & 15));
}

// ---- the same on 64 x 64 tiles ---------------------------------------------------------------
// For launches with too few 128-tiles to fill the chip: the updates inside an outer block, the K = 512 updates of
// the last 4096 columns, the lower levels of the inversion tree.  256 threads own 64 x 64 results, wavefront w the
// 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 tiles.  Such launches are short and their work-groups few, so
// what bounds them is memory latency: a ring of four slices of 16 (64 KB of LDS, two work-groups per CU)
// keeps three in flight, against one 64-deep chunk staged through registers (by panels at d = 3584 the trailing
// updates took 550 us instead of 675 and the inversion products 430 instead of 670).
// Same images as above; a [k][n] slice has 512-byte rows, two per request.
constexpr int kRing64 = 4;
constexpr unsigned kOp64Bytes = NB * kGemmK * sizeof(double);
constexpr unsigned kStage64Bytes = 2 * kOp64Bytes;
constexpr size_t kGemm64LdsBytes = kRing64 * kStage64Bytes;

__device__ __forceinline__ void gemm64_row_sources(const double* base, long ld, int row0, int row_limit, int k_begin,
                                                   int w, int lane, const double* (&src)[2]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = 16 * w + 8 * j + (lane >> 3);
    const int pair = (lane & 7) ^ ((r >> 1) & 7);
    const int g = (row0 + r < row_limit) ? row0 + r : row_limit - 1;
    src[j] = base + (long)g * ld + k_begin + 2 * pair;
  }
}
// (the 64 columns from col0 on exist)
__device__ __forceinline__ void gemm64_col_sources(const double* base, long ld, int k_begin, int col0, int w, int lane,
                                                   const double* (&src)[2]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int k = 4 * w + 2 * j + (lane >> 5), pair = (lane & 31) ^ ((lane >> 5) << 3);
    src[j] = base + (long)(k_begin + k) * ld + col0 + 2 * pair;
  }
}

// q += A B over n_stage slices (all 256 threads, kGemm64LdsBytes of dynamic LDS)
template <bool B_ROWS>
__device__ __forceinline__ void gemm64_accumulate(const double* const (&src_a)[2], const double* const (&src_b)[2],
                                                  long step_a, long step_b, int n_stage, Quad64& q) {
  extern __shared__ __align__(16) double gemm128_lds[];
  typedef __attribute__((address_space(3))) double lds_f64;
  if (n_stage <= 0) return;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(team_wave());
  const unsigned lds0 = (unsigned)(size_t)(lds_f64*)gemm128_lds + (unsigned)w * 2048u;
  const int last = n_stage - 1;
  // slices past the last are requested as the last again, into slots nobody reads any more: the number of
  // outstanding requests, which the waits count, is the same in every iteration
  auto request = [&](int s) {
    const unsigned slot = lds0 + (unsigned)(s % kRing64) * kStage64Bytes;
    const int sc = s < last ? s : last;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma_1k_f64(src_a[j] + sc * step_a, slot + j * 1024u);
#pragma unroll
    for (int j = 0; j < 2; ++j) dma_1k_f64(src_b[j] + sc * step_b, slot + kOp64Bytes + j * 1024u);
  };
  const int l15 = lane & 15, kq = lane >> 4;
  const unsigned sw = (unsigned)((((kq >> 1) ^ (l15 >> 1)) << 4) | ((kq & 1) << 3));
  const unsigned a_row = (unsigned)(((w >> 1) * 32 + l15) * 128) + sw;
  const unsigned b_row = (unsigned)(((w & 1) * 32 + l15) * 128) + sw;
  const unsigned b_col = (unsigned)(kq * 512 + (w & 1) * 256 + l15 * 8);
  const unsigned b_sel[2] = {b_col + (unsigned)((kq & 1) * 128), b_col + (unsigned)(((kq & 1) ^ 1) * 128)};
  const char* const lds_bytes = reinterpret_cast<const char*>(gemm128_lds);
#pragma unroll
  for (int s = 0; s < kRing64 - 1; ++s) request(s);
  for (int s = 0; s < n_stage; ++s) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(8 | 0x0070);            // vmcnt 8: all but the two youngest slices of this wavefront;
                                                       // lgkmcnt 0: its reads of slice s - 1, whose slot is next
    __builtin_amdgcn_s_barrier();                      // ... of all, and slice s - 1 is read out
    asm volatile("" ::: "memory");
    const char* st = lds_bytes + (unsigned)(s % kRing64) * kStage64Bytes;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *reinterpret_cast<const double*>(st + (a_row ^ (unsigned)(32 * t)) + i * 2048);
        if constexpr (B_ROWS)
          b[i] = *reinterpret_cast<const double*>(st + kOp64Bytes + (b_row ^ (unsigned)(32 * t)) + i * 2048);
        else
          b[i] = *reinterpret_cast<const double*>(st + kOp64Bytes + b_sel[i] + t * 2048);
      }
      if (t == 0) request(s + kRing64 - 1);            // behind the first reads, ahead of the products
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          q.c[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], q.c[i][j], 0, 0, 0);
    }
  }
  wait_all_vm();                                       // nothing may still be writing LDS when the work-group ends
}

// ---- the factor and its inverse in one sweep over the panel pairs -----------------------------
// With pairs t = 0, 1, .. from the right (128 columns p_t .. each, L_t = R[0:p_t, p_t ..] above the diagonal block), the
// inverse grows from the bottom: with V[i, c] = sum_s R[i, s] X[s, c] over the pairs s that are done,
//     X[p_t, p_t] = R[p_t, p_t]^-1,     X[p_t, c] = -X[p_t, p_t] V[p_t, c],     V[0:p_t, c] += L_t X[p_t, c]   (c >= p_t).
// The factorisation waits only for its next 128 columns.  So the launch of pair t carries, beside the chain of the
// diagonal block, which occupies one compute unit per 64 rows above it,
//     the inverse of pair t - 1's diagonal block, updates of the columns left of pair t by the L up to L_{t-1}, and
//     updates of V by the L X up to L_{t-2} X[p_{t-2}, :],
// the short launch behind it, which updates the columns of pair t + 1 by L_t, carries X[p_{t-1}, c].  All of
// these are products of depth 128 on 64 x 64 tiles; a tile may wait for several pairs and take their products in one
// visit (Hosted::plan).  L_t and X[p_t, :] go to rings, X to U at once; V lives in A, in the places that the
// factorisation has left.
//
// A hosted work-group of 512 threads works on two tiles at a time, one per team, in step (rings of their own, barriers
// in common; images and slices of the 64-tile engine).  A launch with nothing else (8192 columns, half of the pairs done) runs at 44 TFLOP/s with one pair
// a visit, 46 with two, 55 with eight; without any loads or LDS reads it would reach 61.  It ran at 41, 41 and 50 before
// the operands were read ahead over the barriers, the requests went behind the products and the old values of a tile had
// their registers to themselves (a copy of them in the loop waits for memory); that all operands came from one place in
// L2 made no difference.
constexpr size_t kPairLdsBytes = (size_t)(4 * NB * (NB + 1) + 2 * NB * 16) * sizeof(double);
constexpr int kPairThreads = 512;
constexpr int kPairCols = 2 * NB;
static_assert(2 * kGemm64LdsBytes <= kPairLdsBytes, "two rings");

struct Hosted {
  int inv_p;                      // first column of the pair to invert, -1: none
  const double *inv_r1, *inv_r2, *inv_r12;
  double* inv_x;                  // X[inv_p, :], leading dimension ld
  float* U;                       // d x d
  int d;
  const double *L, *X;            // rings: pair s in slot s % (every + 2)
  int t, n, every;                // beside pair t of n
  // Update of A: tiles (i <= j) of the column pairs whose turn it is, u_far of them, from the left, every 2 `every`
  // blocks from u_b on, then of pair t + 1; n_u tiles, but for the first u_skip.  By the pairs [lo, t).
  int u_b, u_far, n_u_far, n_u, u_skip, u_lo, u_lo_next;
  // V: row pairs likewise, then pair t - 1; all columns of the pairs before t - 1.  By the pairs [lo, t - 1).
  int v_b, v_far, n_v, v_lo, v_lo_next;
  int n_early, head;              // work-groups that start with the panel's, and the rounds that are theirs alone

  __host__ __device__ int first_block(int s) const { return 2 * (n - 1 - s); }
  __host__ __device__ int far_tiles(int m) const { return m * (2 * u_b + 3) + 2 * every * m * (m - 1); }
  __host__ __device__ int n_tiles() const { return n_u - u_skip + n_v; }
  __host__ __device__ int pairs() const { return (n_tiles() + 1) / 2; }

  // Where the tiles of launch t come from: pair c of the columns is due at t = c - 1, its last time, and before that
  // whenever (t + c) is a multiple of `every`, and takes what has come since its last time; pair r of the rows of V
  // is due at t = r + 1 and whenever (t + r) is such a multiple.
  __host__ void plan() {
    const int far = n - 1 - (n - 1 + t) % every;                // the leftmost pair whose turn it is
    const int back_u = (2 * t + 1) % every, back_v = (2 * t - 1) % every;
    if (t >= 1 && t < n) {
      u_b = first_block(far);
      u_far = far >= t + 2 ? (far - (t + 2)) / every + 1 : 0;
      n_u_far = far_tiles(u_far);
      n_u = n_u_far + (t + 1 < n ? 2 * first_block(t + 1) + 3 : 0);
      u_lo = t > every ? t - every : 0;
      u_lo_next = back_u && t > back_u ? t - back_u : u_lo;
    }
    if (t >= 2) {
      v_b = first_block(far);
      v_far = far >= t ? (far - t) / every + 1 : 0;
      n_v = 2 * (2 * (t - 1)) * (v_far + 1);
      v_lo = t - 1 > every ? t - 1 - every : 0;
      v_lo_next = back_v && t - 1 > back_v ? t - 1 - back_v : v_lo;
    }
  }

  // Tile number x (of the update, then of V): its block and the pairs [lo, hi] whose contributions it takes.
  struct Place {
    int i, j, lo, hi;
    bool update, begun;
  };
  __device__ __forceinline__ Place place(int x) const {
    Place p;
    p.update = x < n_u - u_skip;                                // (uniform over a team)
    if (p.update) {
      x += u_skip;
      int b;
      if (x < n_u_far) {
        const float f = (float)(2 * u_b + 3 - 2 * every);
        int m = (int)((sqrtf(f * f + (float)(8 * every) * (float)x) - f) / (float)(4 * every));
        while (far_tiles(m) > x) --m;
        while (far_tiles(m + 1) <= x) ++m;
        x -= far_tiles(m);
        b = u_b + 2 * every * m;
        p.lo = u_lo;
      } else {
        x -= n_u_far;
        b = first_block(t + 1);
        p.lo = u_lo_next;
      }
      p.i = x <= b ? x : x - (b + 1);
      p.j = x <= b ? b : b + 1;
      p.hi = t - 1;
      p.begun = true;
    } else {
      x -= n_u - u_skip;
      const int cols = 2 * (t - 1), row = x / cols, m = row >> 1;
      p.i = (m < v_far ? v_b + 2 * every * m : first_block(t - 1)) + (row & 1);
      p.j = first_block(t - 2) + x % cols;
      p.lo = m < v_far ? v_lo : v_lo_next;
      const int from = n - 1 - (p.j >> 1);                      // V begins with the pair of these columns
      p.begun = from < p.lo;
      if (!p.begun) p.lo = from;
      p.hi = t - 2;
    }
    return p;
  }

  __device__ __forceinline__ void invert(int ld) const {
    extern __shared__ __align__(16) double gemm128_lds[];
    typedef double Row[NB + 1];
    const int team = team_id(), tid = team_tid();
    Row* sR = reinterpret_cast<Row*>(gemm128_lds) + team * NB;
    Row* sV = reinterpret_cast<Row*>(gemm128_lds) + (2 + team) * NB;
    double v[16];
    const double* src = team ? inv_r2 : inv_r1;
    fetch_tile64(src, [](int, int) { return true; }, [](int i, int j) { return (long)i * NB + j; }, v);
    put_tile64(sR, v);
    for (int e = tid; e < NB * NB; e += 256)                    // (the inversion leaves the blocks below the diagonal alone)
      if ((e >> 6) > (e & 63)) sV[e >> 6][e & 63] = 0.0;
    if (team == 0) fetch_tile64(inv_r12, [](int, int) { return true; }, [](int i, int j) { return (long)i * NB + j; }, v);
    invert64(sR, sV);
    Row* const s0 = reinterpret_cast<Row*>(gemm128_lds);        // R12; X11 in s0 + 2 NB, X22 in s0 + 3 NB
    if (team == 0) put_tile64(s0, v);
    __syncthreads();
    Quad64 q;
    if (team == 0) {                                            // R12 X22
      quad_zero(q);
      quad_mfma_64<false>(s0, s0 + 3 * NB, q);
      quad_for_each(q, [&](int r, int c, double x) { (s0 + NB)[r][c] = x; });
    }
    __syncthreads();
    auto put = [&](int i, int j, double x) {                    // row i, column j of the pair's block
      inv_x[(long)i * ld + inv_p + j] = x;
      if (inv_p + i < d && inv_p + j < d) U[(long)(inv_p + i) * d + inv_p + j] = (float)x;
    };
    if (team == 0) {                                            // -X11 (R12 X22)
      quad_zero(q);
      quad_mfma_64<false>(s0 + 2 * NB, s0 + NB, q);
      quad_for_each(q, [&](int r, int c, double x) { put(r, NB + c, -x); });
    }
    for (int e = tid; e < NB * NB; e += 256) {
      const int i = e / NB, j = e % NB;
      put(team * NB + i, team * NB + j, sV[i][j]);
      if (team) inv_x[(long)(NB + i) * ld + inv_p + j] = 0.0;   // left of X22: part of the operand X[p, p]
    }
  }

  // (Pointers are the same for all lanes, whose 32-bit offsets stay: a request takes no vector arithmetic.)
  struct Tile {
    char* C;                        // its place in A
    const char *a, *b;              // sources of slice 0, but for the slot of the rings
    long step_b;                    // bytes from slice to slice of b
    unsigned of_b[2];               // (the lane's)
    int from, lo, hi;               // pairs [lo, hi]; those before lo are multiplied to keep step, and dropped
    bool update, store, diag, begun;
  };
  __device__ __forceinline__ Tile tile(double* __restrict__ A, int ld, int number) const {
    Tile x;
    const int n_all = n_tiles();
    x.store = number < n_all;
    const Place p = place(x.store ? number : n_all - 1);
    const int other = number ^ 1;                               // of the other team
    int len = p.hi - p.lo + 1;
    if (other < n_all) {
      const Place o = place(other);
      if (o.hi - o.lo + 1 > len) len = o.hi - o.lo + 1;
    }
    x.from = __builtin_amdgcn_readfirstlane(p.hi - len + 1);
    x.lo = __builtin_amdgcn_readfirstlane(p.lo);
    x.hi = p.hi;
    x.update = p.update;
    x.begun = p.begun;
    const int row0 = __builtin_amdgcn_readfirstlane(p.i) * NB, col0 = __builtin_amdgcn_readfirstlane(p.j) * NB;
    x.C = reinterpret_cast<char*>(A + (long)row0 * ld + col0);
    x.diag = row0 == col0;
    x.a = reinterpret_cast<const char*>(L + (long)row0 * kPairCols);
    x.b = reinterpret_cast<const char*>(x.update ? L + (long)col0 * kPairCols : X + col0);
    x.step_b = (x.update ? 1 : ld) * (long)(kGemmK * sizeof(double));
    return x;
  }
  __device__ __forceinline__ long slot(int s, int ld) const { return (long)(s % (every + 2)) * ld * kPairCols; }

  // This team's tiles, the slices of all of them one stream through the ring: the first slices and the old values of
  // the next tile are on their way while the present one is multiplied.
  __device__ __forceinline__ void tiles(double* __restrict__ A, int ld, int wg, int n_wg) const {
    const int n = pairs(), alone = n_early * head, early = wg < n_early && wg < n ? min(head, (n - wg + n_early - 1) / n_early) : 0;
    const int count = early + (alone + wg < n ? (n - alone - wg + n_wg - 1) / n_wg : 0);
    auto number = [&](int k) {
      return 2 * (k < early ? wg + k * n_early : alone + wg + (k - early) * n_wg) + team_id();
    };
    extern __shared__ __align__(16) double gemm128_lds[];
    typedef __attribute__((address_space(3))) double lds_f64;
    if (count <= 0) return;
    constexpr int kSlices = kPairCols / kGemmK;                 // of a tile and a pair
    const int team = team_id(), lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(team_wave());
    const unsigned ring = team * (unsigned)kGemm64LdsBytes;
    const unsigned lds0 = (unsigned)(size_t)(lds_f64*)gemm128_lds + ring + (unsigned)w * 2048u;
    unsigned of_rows[2], of_cols[2];                            // this lane's bytes, as in gemm64_{row,col}_sources
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 16 * w + 8 * j + (lane >> 3), k = 4 * w + 2 * j + (lane >> 5);
      of_rows[j] = (unsigned)(r * kPairCols + 2 * ((lane & 7) ^ ((r >> 1) & 7))) * 8u;
      of_cols[j] = (unsigned)(k * ld + 2 * ((lane & 31) ^ ((lane >> 5) << 3))) * 8u;
    }
    auto request = [&](const Tile& x, long off, int s) {
      const unsigned at = lds0 + (unsigned)(s % kRing64) * kStage64Bytes;
      const char* const a = x.a + off + s * (long)(kGemmK * sizeof(double));
      const char* const b = x.b + off + s * x.step_b;
#pragma unroll
      for (int j = 0; j < 2; ++j) dma_1k(a, of_rows[j], at + j * 1024u);
#pragma unroll
      for (int j = 0; j < 2; ++j) dma_1k(b, x.of_b[j], at + kOp64Bytes + j * 1024u);
    };
    auto tile_at = [&](int k) {
      Tile x = tile(A, ld, number(k));
#pragma unroll
      for (int j = 0; j < 2; ++j) x.of_b[j] = x.update ? of_rows[j] : of_cols[j];
      return x;
    };
    const int l15 = lane & 15, kq = lane >> 4;
    const unsigned sw = (unsigned)((((kq >> 1) ^ (l15 >> 1)) << 4) | ((kq & 1) << 3));
    const unsigned a_row = (unsigned)(((w >> 1) * 32 + l15) * 128) + sw;
    const unsigned b_row = (unsigned)(((w & 1) * 32 + l15) * 128) + sw;
    const unsigned b_col = (unsigned)(kq * 512 + (w & 1) * 256 + l15 * 8);
    const unsigned b_sel[2] = {b_col + (unsigned)((kq & 1) * 128), b_col + (unsigned)(((kq & 1) ^ 1) * 128)};
    const char* const lds_bytes = reinterpret_cast<const char*>(gemm128_lds) + ring;
    const int r0 = (w >> 1) * 32 + kq, c0 = (w & 1) * 32 + l15; // this lane's results: rows r0 + 16 i + 4 r, columns c0 + 16 j
    double old[16];
    const unsigned of_result = (unsigned)(r0 * ld + c0) * 8u;
    const long row4 = 4l * ld * (long)sizeof(double);
    auto result = [&](const Tile& x, int i, int j, int r) {
      return reinterpret_cast<double*>(x.C + (4 * i + r) * row4 + of_result) + 16 * j;
    };
    auto load_old = [&](const Tile& x) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) old[8 * i + 4 * j + r] = *result(x, i, j, r);
    };
    auto slot_of = [&](const Tile& x, int pair) { return slot(pair > x.lo ? pair : x.lo, ld) * (long)sizeof(double); };
    Tile x = tile_at(0), y = x;
    int pair = x.from, left = count;                            // tiles left, this one included
    long off = slot_of(x, pair);
#pragma unroll
    for (int s = 0; s < kRing64 - 1; ++s) request(x, off, s);
    load_old(x);
    // The operands of the next four products are read while the present four are multiplied, so the barrier of slice
    // s + 1 lies in the middle of slice s, with products before and behind it that need nothing.
    // vmcnt there: slice s + 1 has landed.  Younger than its four requests are those of slice s + 2 (4) and, in the
    // first two slices of a tile, its 16 old values and the 16 stores of the tile before.  (The compiler, which does not
    // know of the requests, waits as well: for 20 down to 17 outstanding operations at the head of a tile, where it clears
    // the accumulators, so that by then most of the stores have drained, and for 15 in the stores of all but the plain
    // update.  The counts hold all the same; a wait too many only costs its time.)
    int begin = 20;
    Quad64 q;
    double a[2][2], b[2][2];
    auto slice = [&](int s) { return lds_bytes + (unsigned)(s % kRing64) * kStage64Bytes; };
    auto read = [&](const char* st, int t, bool update) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[t & 1][i] = *reinterpret_cast<const double*>(st + (a_row ^ (unsigned)(32 * t)) + i * 2048);
        const unsigned at = update ? (b_row ^ (unsigned)(32 * t)) + i * 2048u : b_sel[i] + t * 2048u;
        b[t & 1][i] = *reinterpret_cast<const double*>(st + kOp64Bytes + at);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int t) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          q.c[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t & 1][i], b[t & 1][j], q.c[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(8 | (1 << 14) | 0x0070);         // 24: slice 0 of the first tile
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read(slice(0), 0, x.update);
    for (;;) {                                                  // tiles
      quad_zero(q);
      for (;;) {                                                // pairs (a loop of its own: the old values stay in place)
        // what comes next: the tile's next pair, or the next tile.  The last is followed by itself: requests into slots
        // that nobody reads any more
        const bool ends = pair == x.hi;
        int next = pair + 1;
        if (ends) {
          if (left > 1) y = tile_at(count - left + 1);
          next = y.from;
        }
        const long next_off = slot_of(y, next);
#pragma unroll
        for (int s = 0; s < kSlices; ++s) {
          read(slice(s), 1, x.update);
          multiply(0);
          read(slice(s), 2, x.update);
          multiply(1);
          asm volatile("" ::: "memory");
          __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt 0: on every path
          if (s > 1 || begin == 4) __builtin_amdgcn_s_waitcnt(4 | 0x0070);
          else if (begin == 20) __builtin_amdgcn_s_waitcnt(4 | (1 << 14) | 0x0070);
          else __builtin_amdgcn_s_waitcnt(4 | (2 << 14) | 0x0070);                  // 36
          __builtin_amdgcn_s_barrier();                           // slice s - 1 is read out, by all
          asm volatile("" ::: "memory");
          read(slice(s), 3, x.update);
          multiply(2);
          if (s + kRing64 - 1 < kSlices) request(x, off, s + kRing64 - 1);
          else request(y, next_off, s + kRing64 - 1 - kSlices);
          read(slice(s + 1), 0, s + 1 < kSlices ? x.update : y.update);
          multiply(3);
        }
        off = next_off;
        const bool dropped = pair < x.lo;
        pair = next;
        if (ends) break;
        if (dropped) quad_zero(q);
        begin = 4;
      }
      if (!x.store) break;                                      // a team's last, when the tiles are odd in number
      // (every lane stores, below the diagonal what it read: the waits count on 16 stores)
      const double sign = x.update ? -1.0 : 1.0;
      auto store = [&](auto value) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) *result(x, i, j, r) = value(i, j, r, old[8 * i + 4 * j + r]);
      };
      if (x.diag)
        store([&](int i, int j, int r, double o) { return c0 + 16 * j < r0 + 16 * i + 4 * r ? o : o - q.c[i][j][r]; });
      else if (x.begun)
        store([&](int i, int j, int r, double o) { return fma(sign, q.c[i][j][r], o); });
      else
        store([&](int i, int j, int r, double) { return q.c[i][j][r]; });
      if (--left == 0) break;
      x = y;
      load_old(x);
      begin = 36;
    }
    wait_all_vm();                                              // nothing may still be writing LDS when the work-group ends
  }

  __device__ __forceinline__ void run(double* __restrict__ A, int ld, int wg, int n_wg) const {
    if (inv_p >= 0) {                                           // it counts as a work-group that starts late
      if (wg == 0) {
        invert(ld);
        __syncthreads();
        wg = n_wg;
      }
      --wg;
    }
    tiles(A, ld, wg, n_wg);
  }
};

__global__ __launch_bounds__(kPairThreads) void hosted_kernel(double* __restrict__ A, int ld, Hosted host) {
  host.run(A, ld, blockIdx.x, gridDim.x);
}

// q += A B like gemm64_accumulate for the upper or lower half of a tile: 32 rows of A (src_a: 8 rows a wavefront),
// wavefront w has the 16 columns from 16 w on, rows 16 i + 4 r + lane / 16 in q[i][r].
__device__ __forceinline__ const double* gemm32_row_source(const double* base, long ld, int row0, int k_begin, int w, int lane) {
  const int r = 8 * w + (lane >> 3);
  return base + (long)(row0 + r) * ld + k_begin + 2 * ((lane & 7) ^ ((r >> 1) & 7));
}
template <bool B_ROWS>
__device__ __forceinline__ void gemm32_accumulate(const double* src_a, const double* const (&src_b)[2], long step_a,
                                                  long step_b, int n_stage, f64x4 (&q)[2]) {
  extern __shared__ __align__(16) double gemm128_lds[];
  typedef __attribute__((address_space(3))) double lds_f64;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(team_wave());
  const unsigned lds0 = (unsigned)(size_t)(lds_f64*)gemm128_lds + (unsigned)w * 1024u;
  const int last = n_stage - 1;
  auto request = [&](int s) {                          // (slices past the last like there)
    const unsigned slot = lds0 + (unsigned)(s % kRing64) * kStage64Bytes;
    const int sc = s < last ? s : last;
    dma_1k_f64(src_a + sc * step_a, slot);
#pragma unroll
    for (int j = 0; j < 2; ++j) dma_1k_f64(src_b[j] + sc * step_b, slot + kOp64Bytes + (unsigned)w * 1024u + j * 1024u);
  };
  const int l15 = lane & 15, kq = lane >> 4;
  const unsigned sw = (unsigned)((((kq >> 1) ^ (l15 >> 1)) << 4) | ((kq & 1) << 3));
  const unsigned a_row = (unsigned)(l15 * 128) + sw, b_row = (unsigned)((16 * w + l15) * 128) + sw;
  const unsigned b_col = (unsigned)(kq * 512 + (w ^ (kq & 1)) * 128 + l15 * 8);
  const char* const lds_bytes = reinterpret_cast<const char*>(gemm128_lds);
#pragma unroll
  for (int s = 0; s < kRing64 - 1; ++s) request(s);
  for (int s = 0; s < n_stage; ++s) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(6 | 0x0070);            // vmcnt 6: all but the two youngest slices; lgkmcnt 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const char* st = lds_bytes + (unsigned)(s % kRing64) * kStage64Bytes;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const double b = *reinterpret_cast<const double*>(st + kOp64Bytes + (B_ROWS ? b_row ^ (unsigned)(32 * t) : b_col + t * 2048u));
      double a[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const double*>(st + (a_row ^ (unsigned)(32 * t)) + i * 2048);
      if (t == 0) request(s + kRing64 - 1);
#pragma unroll
      for (int i = 0; i < 2; ++i) q[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b, q[i], 0, 0, 0);
    }
  }
  wait_all_vm();                                       // nothing may still be writing LDS when the work-group ends
}

// The short launch between two pairs, half of a 64 x 64 tile per work-group of 256 threads: first the tiles (i <= j), j in
// blocks [u0, u0 + 2), of the update by Lu (n_u of them), then X[xp, c] = -X[xp, xp] V[xp, c] for the column blocks c from
// xc0 on (n_x tiles), then the first tiles of `left`, which the launch before left out.  Its length is that of a tile's
// products, 512 matrix instructions of 64 cycles on four matrix cores, and a round trip to memory: whole tiles, which
// leave half of the compute units idle at 3584 columns, took 8.3 us (1284 us for the whole of it, 1241 with halves).
__global__ __launch_bounds__(256, 2) void pair_link_kernel(double* __restrict__ A, int ld, const double* __restrict__ Lu,
                                                           int u0, int n_u, double* __restrict__ X, int xp, int xc0,
                                                           int n_x, Hosted left, float* __restrict__ U, int d) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(team_wave());
  const int number = blockIdx.x >> 1, half = (blockIdx.x & 1) * (NB / 2);
  f64x4 q[2] = {(f64x4){0.0, 0.0, 0.0, 0.0}, (f64x4){0.0, 0.0, 0.0, 0.0}};
  const int row_of = half + (lane >> 4), col_of = 16 * w + (lane & 15);     // results: rows row_of + 16 i + 4 r of the tile
  const double* src_b[2];
  const bool left_out = number >= n_u + n_x;
  if (number < n_u || left_out) {
    int j = number <= u0 ? u0 : u0 + 1, i = number <= u0 ? number : number - (u0 + 1);
    int lo = 0, hi = 0;
    if (left_out) {
      const Hosted::Place p = left.place(number - n_u - n_x);
      i = p.i;
      j = p.j;
      lo = p.lo;
      hi = p.hi;
    }
    double* const C = A + (long)i * NB * ld + j * NB;
    double old[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) old[e] = C[(long)(row_of + 4 * e) * ld + col_of];
    __builtin_amdgcn_sched_barrier(0);
    for (int s = lo; s <= hi; ++s) {
      if (left_out) Lu = left.L + left.slot(s, ld);
      if (s > lo) __syncthreads();
      gemm64_row_sources(Lu, kPairCols, j * NB, j * NB + NB, 0, w, lane, src_b);
      gemm32_accumulate<true>(gemm32_row_source(Lu, kPairCols, i * NB + half, 0, w, lane), src_b, kGemmK, kGemmK,
                              kPairCols / kGemmK, q);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int r = row_of + 4 * e;
      if (i < j || col_of >= r) C[(long)r * ld + col_of] = old[e] - q[e >> 2][e & 3];
    }
    return;
  }
  const int t = number - n_u, r0 = (t & 1) * NB, c0 = (xc0 + (t >> 1)) * NB;
  gemm64_col_sources(A, ld, xp + r0, c0, w, lane, src_b);                   // (left of X22 there are zeros)
  gemm32_accumulate<false>(gemm32_row_source(X, ld, r0 + half, xp + r0, w, lane), src_b, kGemmK, (long)kGemmK * ld,
                           (kPairCols - r0) / kGemmK, q);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int r = r0 + row_of + 4 * e, c = c0 + col_of;
    const double v = -q[e >> 2][e & 3];
    X[(long)r * ld + c] = v;
    if (xp + r < d && c < d) U[(long)(xp + r) * d + c] = (float)v;
  }
}

// Two adjacent 64-column panels -- block b1 (columns p1 ..) and block b2 = b1 + 1 -- in one
// launch, one work-group per 64 rows above them.  With the diagonal 128 x 128 block
// [D11 D12; D12^T D22] every work-group computes for itself
//     D22 = R22 R22^T,   R12 = D12 R22^-T,   D11 - R12 R12^T = R11 R11^T
// and for its own rows [A1 A2] of the two panels
//     X2 = A2 R22^-T,    X1 = (A1 - X2 R12^T) R11^-T.
// The solves and products run on the fp64 matrix cores.  This halves the number of dependent launches of
// the panel chain (each is short and latency-bound).  A work-group is two teams of four wavefronts.  The first
// walks the chain of the diagonal block; the second solves the work-group's rows beside it and updates them in the
// intervals between the barriers of the second factorisation, whose matrix cores are nearly idle, in pieces that end
// before the chain reaches the next barrier.  So R22 and its inverses stay where they are while R11 is factored in
// the place of A1, which waits in registers (56 rows of work-groups: 33 -> 24 us).  Work-group 0 writes R11, R22 to
// Rdiag and R12 to R12buf (never into A, whose blocks later-scheduled work-groups still read) and sets the
// pair flag of b2, so that the inverse step puts R12 in place.
// The rows' results go to L (leading dimension ldl; row r, column j of the pair at L[r ldl + j]), which may be their own
// place in A.  Work-groups from `panel_wgs` on carry other tiles of the update (Hosted).
__global__ __launch_bounds__(kPairThreads) void panel_pair_kernel(double* A, int d, int p1, int nb2, int n_above,
                                                                  double* L, int ldl,
                                                                  int panel_wgs, Hosted host,
                                                                  double* __restrict__ Rdiag1,
                                                                  double* __restrict__ Rdiag2,
                                                                  double* __restrict__ R12buf,
                                                                  int* __restrict__ pair_flag1,
                                                                  int* __restrict__ pair_flag2, int* info) {
  if ((int)blockIdx.x >= panel_wgs) {
    host.run(A, d, blockIdx.x - panel_wgs, gridDim.x - panel_wgs);
    return;
  }
  extern __shared__ __align__(16) double gemm128_lds[];
  double* const dyn = gemm128_lds;
  typedef double Row[NB + 1];
  Row* sR22 = reinterpret_cast<Row*>(dyn);          // R22, then A1 - X2 R12^T -> X1
  Row* sR12 = sR22 + NB;                            // D12 -> R12
  Row* sR11 = sR12 + NB;                            // D11 - R12 R12^T -> R11
  Row* sA2 = sR11 + NB;                             // own rows, columns of b2
  Inv16* sInv22 = reinterpret_cast<Inv16*>(dyn + 4 * NB * (NB + 1));
  Inv16* sInv11 = sInv22 + NB / 16;
  const int tid = team_tid();
  const bool chain = threadIdx.x < 256;             // team of the diagonal block; the other has the rows
  const int p2 = p1 + NB;
  const int r0 = blockIdx.x * NB;
  const bool first = blockIdx.x == 0, rows = n_above > 0;
  const bool vec = nb2 == NB && d % 2 == 0;

  // D11 (chain) or A1 (rows) in the product's layout, needed after the first factorisation
  Quad64 base;
  quad_zero(base);
  auto fetch_quad = [&](int row0) {
    const int lane = threadIdx.x & 63, w = team_wave();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          base.c[i][j][r] = A[(long)(row0 + (w >> 1) * 32 + 16 * i + 4 * r + (lane >> 4)) * d + p1 + (w & 1) * 32 + 16 * j +
                              (lane & 15)];
  };
  if (chain) {
    double v22[16], v12[16];
    fetch_tile(A, d, p2, p2, nb2, nb2, true, vec, v22);
    fetch_tile(A, d, p1, p2, NB, nb2, false, vec, v12);
    fetch_quad(p1);
    put_tile(sR22, vec, v22);
    put_tile(sR12, vec, v12);
  } else if (rows) {                                // (the rows above a full panel are all there)
    double v2[16];
    fetch_tile(A, d, r0, p2, NB, nb2, false, vec, v2);
    fetch_quad(r0);
    put_tile(sA2, vec, v2);
  }
  factor64_blocked(sR22, sInv22, info, p2, first, chain);
  f64x4 acc[4];
  Quad64 q;
  quad_zero(q);
  if (chain) {
    trsm64_blocked(sR12, sR22, sInv22);             // R12 = D12 R22^-T
  } else if (rows) {                                // X2 = A2 R22^-T
    trsm_load(acc, sA2);
    trsm_block_step<3>(acc, sA2, sR22, sInv22);
    trsm_block_step<2>(acc, sA2, sR22, sInv22);
  }
  __syncthreads();
  if (chain) {
    quad_mfma_64<true>(sR12, sR12, q);              // D11 - R12 R12^T
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) q.c[i][j] = base.c[i][j] - q.c[i][j];
    quad_for_each(q, [&](int r, int c, double v) { sR11[r][c] = v; });
  } else if (rows) {
    trsm_block_step<1>(acc, sA2, sR22, sInv22);
    trsm_block_step<0>(acc, sA2, sR22, sInv22);
  }
  factor64_blocked(sR11, sInv11, info, p1, first, chain, [&](auto step) {
    constexpr int S = decltype(step)::value;
    if constexpr (S == 1) {
      if (first)
        for (int e = tid; e < NB * NB; e += 256) {
          Rdiag2[e] = sR22[e / NB][e % NB];
          R12buf[e] = sR12[e / NB][e % NB];
        }
    }
    if (!rows) return;
    if constexpr (S == 0) {                         // X2 is finished
      for (int e = tid; e < NB * NB; e += 256) {
        const int i = e / NB, j = e % NB;
        if (j < nb2) L[(long)(r0 + i) * ldl + NB + j] = sA2[i][j];
      }
    }
    // A1 - X2 R12^T, in the place of R22
    if constexpr (S == 2) quad_mfma_64<true, 0, 20>(sA2, sR12, q);
    if constexpr (S == 4) quad_mfma_64<true, 20, 40>(sA2, sR12, q);
    if constexpr (S == 6) {
      quad_mfma_64<true, 40, NB>(sA2, sR12, q);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) q.c[i][j] = base.c[i][j] - q.c[i][j];
      quad_for_each(q, [&](int r, int c, double v) { sR22[r][c] = v; });
    }
  });
  if (first && !chain) {
    for (int e = tid; e < NB * NB; e += 256) Rdiag1[e] = sR11[e / NB][e % NB];
    if (tid == 0) {
      *pair_flag1 = 0;
      *pair_flag2 = 1;
    }
  }
  if (!rows) return;
  if (chain) trsm64_blocked(sR22, sR11, sInv11);
  __syncthreads();
  for (int e = threadIdx.x; e < NB * NB; e += kPairThreads) {
    const int i = e / NB, j = e % NB;
    L[(long)(r0 + i) * ldl + j] = sR22[i][j];
  }
}

// The trailing update on this engine.  Tile order: the hardware deals work-groups to the 8 dies in
// turn (work-group b runs on die b % 8, each die with an L2 of its own).  Die x takes the row tiles
// I = x, x + 8, ... of every band of 4 column tiles, four consecutive work-groups sharing one row
// strip; a band's four column strips (2 MB at depth 512) stay in that die's L2 while its row tiles
// stream past.  Needs d even, Kd a multiple of 32, k0 + Kd <= d.
constexpr int kTrailBand = 4;

// Row tiles of band `band` that die x works on: I = x + 8 n, n < the value returned.  The band's
// last column is min(cbeg + 128 (4 band + 4), cend) - 1; row tiles beyond it lie below the diagonal.
__host__ __device__ inline int trail_band_rows(int band, int x, int cbeg, int cend) {
  long last = (long)cbeg + (long)kGemmTile * kTrailBand * (band + 1);
  if (last > cend) last = cend;
  const int i_last = (int)((last - 1) / kGemmTile);
  return (i_last >= x) ? (i_last - x) / 8 + 1 : 0;
}

__global__ __launch_bounds__(256, 2) void syrk_trailing128_kernel(double* __restrict__ A, int d, int k0,
                                                                  int Kd, int cb0, int cb1) {
  const int cbeg = cb0 * NB, cend = cb1 * NB;
  const int n_col_tiles = (cend - cbeg + kGemmTile - 1) / kGemmTile;
  const int n_band = (n_col_tiles + kTrailBand - 1) / kTrailBand;
  const int x = blockIdx.x & 7;
  int rem = blockIdx.x >> 3, band = 0;
  for (; band < n_band; ++band) {
    const int cnt = trail_band_rows(band, x, cbeg, cend) * kTrailBand;
    if (rem < cnt) break;
    rem -= cnt;
  }
  if (band == n_band) return;
  const int tj = band * kTrailBand + (rem & (kTrailBand - 1));
  if (tj >= n_col_tiles) return;
  const int row0 = (x + 8 * (rem / kTrailBand)) * kGemmTile;
  const int col0 = cbeg + tj * kGemmTile;
  if (row0 > col0 + kGemmTile - 1) return;      // wholly below the diagonal

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Acc128 q;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) q.c[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
  const double* src_i[4];
  const double* src_j[4];
  gemm128_row_sources(A, d, row0, cend, k0, w, lane, src_i);
  gemm128_row_sources(A, d, col0, cend, k0, w, lane, src_j);
  gemm128_accumulate<true>(src_i, src_j, kGemmK, kGemmK, Kd / kGemmK, q);
  // read-modify-write, one row of tiles (16 values per lane) at a time, loads first
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double old[16];
    acc128_for_each_in_row(i, [&](int j, int r, int row, int col) {
      const int gi = row0 + row, gj = col0 + col;
      const bool in = gi < cend && gj < cend && gj >= gi;
      old[4 * j + r] = A[in ? (long)gi * d + gj : 0L];
    });
    acc128_for_each_in_row(i, [&](int j, int r, int row, int col) {
      const int gi = row0 + row, gj = col0 + col;
      if (gi < cend && gj < cend && gj >= gi) A[(long)gi * d + gj] = old[4 * j + r] - q.c[i][j][r];
    });
  }
}

// Work-groups of a launch of the 128-tile update over column blocks [cb0, cb1): 8 dies times the
// longest list, which is die 0's.
static int trail128_grid(int cb0, int cb1) {
  const int cbeg = cb0 * NB, cend = cb1 * NB;
  const int n_col_tiles = (cend - cbeg + kGemmTile - 1) / kGemmTile;
  const int n_band = (n_col_tiles + kTrailBand - 1) / kTrailBand;
  int slots = 0;
  for (int band = 0; band < n_band; ++band) slots += trail_band_rows(band, 0, cbeg, cend) * kTrailBand;
  return 8 * slots;
}
// The trailing update on 64 x 64 tiles of the DMA engine, upper tiles (bi <= bj), bj in [cb0, cb1).
// Needs d even, Kd a multiple of 16, k0 + Kd <= d.
__global__ __launch_bounds__(256, 2) void syrk_trailing64_kernel(double* __restrict__ A, int d, int k0, int Kd,
                                                                 int cb0, int cb1) {
  int tile = blockIdx.x, bj = cb0;
  while (tile >= bj + 1) {
    tile -= bj + 1;
    ++bj;
  }
  const int row0 = tile * NB, col0 = bj * NB;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Quad64 q;
  quad_zero(q);
  // this lane's 16 old values, requested first: they arrive under the products
  double old[16];
  int n = 0;
  quad_for_each(q, [&](int r, int c, double) {
    const int i = row0 + r, j = col0 + c;
    old[n++] = A[(j >= i) ? (long)i * d + j : 0L];
  });
  __builtin_amdgcn_sched_barrier(0);
  const double* src_i[2];
  const double* src_j[2];
  gemm64_row_sources(A, d, row0, row0 + NB, k0, w, lane, src_i);
  gemm64_row_sources(A, d, col0, col0 + NB, k0, w, lane, src_j);
  gemm64_accumulate<true>(src_i, src_j, kGemmK, kGemmK, Kd / kGemmK, q);
  n = 0;
  quad_for_each(q, [&](int r, int c, double v) {
    const int i = row0 + r, j = col0 + c;
    if (j >= i) A[(long)i * d + j] = old[n] - v;
    ++n;
  });
}

// Below this many column blocks left to update (the last 4096 columns) the 64-tile kernel has more work-groups to spread
// over the chip.
constexpr int kTrail128MinBlocks = 64;
// ... and a level of the inversion tree with fewer 128-tiles than this (two per compute unit)
constexpr long kInverse128MinTiles = 512;

// ---------------------------------------------------------------- invert -------------------
// Node `node` of tree depth `depth` over the block range [0, P): ranges are halved
// (left half gets the extra block).  Returns false if the path ends in a leaf earlier.
__device__ __forceinline__ bool tree_node(int P, int depth, int node, int& lo, int& mid, int& hi) {
  lo = 0;
  hi = P;
  for (int l = depth - 1; l >= 0; --l) {
    if (hi - lo < 2) return false;
    const int m = lo + (hi - lo + 1) / 2;
    if ((node >> l) & 1) lo = m; else hi = m;
  }
  if (hi - lo < 2) return false;
  mid = lo + (hi - lo + 1) / 2;
  return true;
}

// One 64 x 64 output tile of C = op(A) * op(B) in fp64, 256 threads, 4 x 4 per thread.
// MODE 1: tmp = R12 * U22      (B upper triangular: k-tiles 0..tj, diagonal tile masked)
// MODE 2: A12 = -U11 * tmp     (A upper triangular: k-tiles ti..M-1, diagonal tile masked)
template <int MODE>
__global__ __launch_bounds__(256) void tri_inverse_level_kernel(double* __restrict__ A, int d,
                                                                double* __restrict__ tmp, int ldt,
                                                                int P, int depth) {
  __shared__ double sa[NB][NB + 1];
  __shared__ double sb[NB][NB + 1];
  int lo, mid, hi;
  if (!tree_node(P, depth, blockIdx.z, lo, mid, hi)) return;
  const int Mb = mid - lo, Nb = hi - mid;        // in blocks
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (ti >= Mb || tj >= Nb) return;
  const int tid = threadIdx.x;
  const int row0 = (lo + ti) * NB;               // global rows of the output tile
  const int col0 = (mid + tj) * NB;              // global cols of the output tile (in A)
  Quad64 q;
  quad_zero(q);
  const int kb_begin = (MODE == 1) ? 0 : ti;
  const int kb_end = (MODE == 1) ? tj + 1 : Mb;
  double va[16], vb[16];
  auto fetch = [&](int kb) {
    if (MODE == 1) {
      // A operand: R12[row0+i][(mid+kb)*NB + j];  B operand: U22[(mid+kb)*NB+i][col0+j]
      fetch_tile64(A, [&](int i, int j) { return row0 + i < d && (mid + kb) * NB + j < d; },
                   [&](int i, int j) { return (long)(row0 + i) * d + (mid + kb) * NB + j; }, va);
      fetch_tile64(A,
                   [&](int i, int j) {
                     const int br = (mid + kb) * NB + i, bc = col0 + j;
                     return br < d && bc < d && br <= bc;
                   },
                   [&](int i, int j) { return (long)((mid + kb) * NB + i) * d + col0 + j; }, vb);
    } else {
      // A operand: U11[row0+i][(lo+kb)*NB + j];  B operand: tmp[(lo+kb)*NB+i][tj*NB+j]
      fetch_tile64(A,
                   [&](int i, int j) {
                     const int gr = row0 + i, gc = (lo + kb) * NB + j;
                     return gr < d && gc < d && gr <= gc;
                   },
                   [&](int i, int j) { return (long)(row0 + i) * d + (lo + kb) * NB + j; }, va);
      fetch_tile64(tmp, [&](int i, int) { return (lo + kb) * NB + i < d; },
                   [&](int i, int j) { return (long)((lo + kb) * NB + i) * ldt + tj * NB + j; }, vb);
    }
  };
  if (kb_begin < kb_end) fetch(kb_begin);
  for (int kb = kb_begin; kb < kb_end; ++kb) {
    put_tile64(sa, va);
    put_tile64(sb, vb);
    __syncthreads();
    if (kb + 1 < kb_end) fetch(kb + 1);             // in flight during the products below
    quad_mfma_64<false>(sa, sb, q);
    __syncthreads();
  }
  quad_for_each(q, [&](int r, int c, double v) {
    const int i = row0 + r;
    if (i >= d) return;
    if (MODE == 1) {
      tmp[(long)i * ldt + tj * NB + c] = v;
    } else if (col0 + c < d) {
      A[(long)i * d + col0 + c] = -v;
    }
  });
}

// The same two products on the 128-tile engine (d a multiple of 64).  Tile (ti, tj) of 128 x 128:
//   MODE 1: tmp[rows][tj] = R12[rows][k] U22[k][tj], k over the columns of U22 up to the tile's last
//           (U22 is upper triangular; the block left of a diagonal block holds zeros);
//   MODE 2: U12[rows][tj] = -U11[rows][k] tmp[k][tj], k from the tile's first row on.
// A node with an odd number of blocks leaves half a tile hanging over: its rows / columns are
// clamped on the way in and skipped on the way out.
template <int MODE>
__global__ __launch_bounds__(256, 2) void tri_inverse_level128_kernel(double* __restrict__ A, int d,
                                                                      double* __restrict__ tmp, int ldt,
                                                                      int P, int depth) {
  int lo, mid, hi;
  if (!tree_node(P, depth, blockIdx.z, lo, mid, hi)) return;
  const int n_rows = (mid - lo) * NB, n_cols = (hi - mid) * NB;
  // K ranges grow with the tile column (MODE 1) or shrink with the tile row (MODE 2).  The slow grid axis
  // walks them from the longest down, the fast axis the tiles of equal length, which go to the 8 XCDs in
  // turn: every XCD gets the same mix, and the last tiles to start are the shortest.  (Columns on the fast
  // axis, rotated by the row: MODE 1 954 us a launch at d = 8192 against 795.  Super-blocks of
  // 4 x 4 tiles per XCD, for L2 reuse, were slower too.)
  const int r_loc = (int)(MODE == 1 ? blockIdx.x : blockIdx.y) * kGemmTile;                           // inside the node
  const int c_loc = (int)(MODE == 1 ? gridDim.y - 1 - blockIdx.y : blockIdx.x) * kGemmTile;
  if (r_loc >= n_rows || c_loc >= n_cols) return;
  const int row0 = lo * NB + r_loc, row_limit = mid * NB;     // global rows of the tile
  const int col0 = mid * NB + c_loc, col_limit = hi * NB;     // global columns of the tile (in A)
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Acc128 q;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) q.c[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
  const double* src_a[4];
  const double* src_b[4];
  if (MODE == 1) {
    const int k_begin = mid * NB;
    const int k_end = (col0 + kGemmTile < col_limit) ? col0 + kGemmTile : col_limit;
    gemm128_row_sources(A, d, row0, row_limit, k_begin, w, lane, src_a);
    gemm128_col_sources(A, d, k_begin, col0, col_limit, w, lane, src_b);
    gemm128_accumulate<false>(src_a, src_b, kGemmK, (long)kGemmK * d, (k_end - k_begin) / kGemmK, q);
  } else {
    const int k_begin = row0, k_end = row_limit;
    gemm128_row_sources(A, d, row0, row_limit, k_begin, w, lane, src_a);
    gemm128_col_sources(tmp, ldt, k_begin, c_loc, n_cols, w, lane, src_b);
    gemm128_accumulate<false>(src_a, src_b, kGemmK, (long)kGemmK * ldt, (k_end - k_begin) / kGemmK, q);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    acc128_for_each_in_row(i, [&](int j, int r, int row, int col) {
      const int gi = row0 + row;
      if (gi >= row_limit || c_loc + col >= n_cols) return;
      if (MODE == 1) tmp[(long)gi * ldt + c_loc + col] = q.c[i][j][r];
      else A[(long)gi * d + col0 + col] = -q.c[i][j][r];
    });
}

// The same two products on 64 x 64 tiles of the DMA engine (d a multiple of 64).
template <int MODE>
__global__ __launch_bounds__(256, 2) void tri_inverse_level64_kernel(double* __restrict__ A, int d,
                                                                     double* __restrict__ tmp, int ldt, int P,
                                                                     int depth) {
  int lo, mid, hi;
  if (!tree_node(P, depth, blockIdx.z, lo, mid, hi)) return;
  // longest K range first: the last tile column (MODE 1) / the first tile row (MODE 2)
  const int ti = (MODE == 1) ? blockIdx.x : blockIdx.y;
  const int tj = (MODE == 1) ? (hi - mid) - 1 - (int)blockIdx.y : (int)blockIdx.x;
  if (ti >= mid - lo || tj < 0 || tj >= hi - mid) return;
  const int row0 = (lo + ti) * NB, col0 = (mid + tj) * NB;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Quad64 q;
  quad_zero(q);
  const double* src_a[2];
  const double* src_b[2];
  if (MODE == 1) {
    const int k_begin = mid * NB, k_end = col0 + NB;
    gemm64_row_sources(A, d, row0, row0 + NB, k_begin, w, lane, src_a);
    gemm64_col_sources(A, d, k_begin, col0, w, lane, src_b);
    gemm64_accumulate<false>(src_a, src_b, kGemmK, (long)kGemmK * d, (k_end - k_begin) / kGemmK, q);
  } else {
    const int k_begin = row0, k_end = mid * NB;
    gemm64_row_sources(A, d, row0, row0 + NB, k_begin, w, lane, src_a);
    gemm64_col_sources(tmp, ldt, k_begin, tj * NB, w, lane, src_b);
    gemm64_accumulate<false>(src_a, src_b, kGemmK, (long)kGemmK * ldt, (k_end - k_begin) / kGemmK, q);
  }
  quad_for_each(q, [&](int r, int c, double v) {
    if (MODE == 1) tmp[(long)(row0 + r) * ldt + tj * NB + c] = v;
    else A[(long)(row0 + r) * d + col0 + c] = -v;
  });
}

// U (fp32) <- upper triangle of A, zeros below; one 64 x 64 block per work-group.
__global__ __launch_bounds__(256) void prep_store_kernel(const double* __restrict__ A, int d,
                                                         float* __restrict__ U) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  const int j = bj * NB + (threadIdx.x & 63), i0 = bi * NB + (threadIdx.x >> 6);
  double a[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = i0 + 4 * t;
    a[t] = 0.0;
    if (bj >= bi) a[t] = A[(j >= i && i < d && j < d) ? (long)i * d + j : 0L];
  }
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    const int i = i0 + 4 * t;
    if (i < d && j < d) U[(long)i * d + j] = (j >= i) ? (float)a[t] : 0.f;
  }
}

static int tree_depth(int P) {   // number of levels that contain at least one internal node
  int depth = 0, width = P;
  while (width >= 2) {
    width = (width + 1) / 2;
    ++depth;
  }
  return depth;
}

struct PrepLayout {
  size_t a_off, tmp_off, rdiag_off, r12_off, flag_off, scal_off, total;
  int P, ldt;
};

// How many pairs a tile of the update or of V waits for: its old values are read and written once for all of them, but
// the rounds of tiles are coarser.  By the padded width: up to 4608 columns the chain has to be filled evenly (4608: 2106 us with one pair, 2113
// with two, 2138 with three; 5120: 2672, 2641, 2645), beyond the products take the time (6016: 3888, 3766, 3787; 6272:
// 4168 with two, 4166 with three; 6400: 4393, 4383; 6656: 5022 with one, 4832, 4802; 8192: 8905, 8208, 8077, 8362 with
// four; 12288: 28.7 ms, 25.2, 24.1, 24.3).
constexpr int kOnePairMax = 4608, kThreePairsMin = 6400;
// The sweep over panel pairs: A padded to whole pairs, rings of L_t and of X[p_t, :].
struct SweepLayout {
  size_t a_off, l_off, x_off, rdiag_off, r12_off, flag_off, scal_off, total;
  int n_pair, ld, every, slots;
};
static SweepLayout sweep_layout(int d) {
  SweepLayout L;
  L.n_pair = bpdq_ceil_div(d, kPairCols);
  L.ld = L.n_pair * kPairCols;
  L.every = L.ld <= kOnePairMax ? 1 : L.ld < kThreePairsMin ? 2 : 3;
  L.slots = L.every + 2;
  size_t off = 0;
  L.a_off = off;     off += (size_t)L.ld * L.ld * sizeof(double);
  L.l_off = off;     off += (size_t)L.slots * L.ld * kPairCols * sizeof(double);
  L.x_off = off;     off += (size_t)L.slots * L.ld * kPairCols * sizeof(double);
  L.rdiag_off = off; off += (size_t)2 * L.n_pair * NB * NB * sizeof(double);
  L.r12_off = off;   off += (size_t)2 * L.n_pair * NB * NB * sizeof(double);
  L.flag_off = off;  off += bpdq_align_up((size_t)2 * L.n_pair * sizeof(int), 256);
  L.scal_off = off;  off += 256;
  L.total = off;
  return L;
}
// One panel has nothing to pair or to hide (d <= 64: 46 us by pairs, 23 to 27 by panels).  From there on the pairs are
// quicker (65: 45 us against 55, 192: 88.6 against 89.7, 384: 132 against 165, 1600: 530 against 755, 3584: 1245 against
// 1939, 6016: 3781 against 5079, 8192: 8095 against 9760, 11008: 17.9 ms against 19.7, 12288: 24.0 against 25.2) until a
// tile's traffic costs more than the chain that it hides (14336: 37.7 ms against 37.8, 16384: 54.8 against 53.4).  Widths
// off 64 gain more (4097: 1735 us against 3084, 8191: 8143 against 12848).
constexpr int kSweepMin = NB + 1, kSweepMax = 12288;
static bool sweep_pays(int d) { return d >= kSweepMin && d <= kSweepMax; }

static PrepLayout prep_layout(int d) {
  PrepLayout L;
  L.P = bpdq_ceil_div(d, NB);
  L.ldt = ((L.P + 1) / 2) * NB;
  size_t off = 0;
  L.a_off = off;    off += bpdq_align_up((size_t)d * d * sizeof(double), 256);
  L.tmp_off = off;  off += bpdq_align_up((size_t)d * L.ldt * sizeof(double), 256);
  L.rdiag_off = off; off += bpdq_align_up((size_t)L.P * NB * NB * sizeof(double), 256);
  L.r12_off = off;  off += bpdq_align_up((size_t)L.P * NB * NB * sizeof(double), 256);
  L.flag_off = off; off += bpdq_align_up((size_t)L.P * sizeof(int), 256);
  L.scal_off = off; off += 256;
  L.total = off;
  return L;
}

#define BPDQ_TRY(expr)              \
  do {                              \
    const int rc_ = (expr);         \
    if (rc_ != 0) return rc_;       \
  } while (0)

// The trailing update of column blocks [cb0, cb1) by the factored columns [k0, k0 + depth).
static int launch_trailing(hipStream_t st, double* A, int d, int k0, int depth, int cb0, int cb1) {
  if (cb1 <= cb0) return 0;
  const bool dma = d % 2 == 0 && depth % 32 == 0 && k0 + depth <= d;
  const int tiles = (cb1 * (cb1 + 1) - cb0 * (cb0 + 1)) / 2;
  if (dma && cb0 == 0 && cb1 >= kTrail128MinBlocks) {
    hipLaunchKernelGGL(syrk_trailing128_kernel, dim3(trail128_grid(cb0, cb1)), dim3(256), kGemmLdsBytes, st,
                       A, d, k0, depth, cb0, cb1);
  } else if (dma) {
    hipLaunchKernelGGL(syrk_trailing64_kernel, dim3(tiles), dim3(256), kGemm64LdsBytes, st, A, d, k0, depth, cb0, cb1);
  } else {
    // the ragged right edge: a panel of fewer than 64 columns, or rows that are not 16-byte aligned
    hipLaunchKernelGGL(syrk_trailing_kernel, dim3(tiles), dim3(256), 0, st, A, d, k0, depth, cb0, cb1);
  }
  BPDQ_LAUNCH_CHECK();
  return 0;
}

}  // namespace bpdq

using namespace bpdq;

static int prepare_by_pairs(const float* H, int d, float damp, float* U, unsigned char* dead, int* info, char* base,
                            hipStream_t stream) {
  const SweepLayout L = sweep_layout(d);
  const int ld = L.ld, P = 2 * L.n_pair, n = L.n_pair;
  double* A = reinterpret_cast<double*>(base + L.a_off);
  double* ring = reinterpret_cast<double*>(base + L.l_off);
  double* X = reinterpret_cast<double*>(base + L.x_off);
  double* Rdiag = reinterpret_cast<double*>(base + L.rdiag_off);
  double* R12 = reinterpret_cast<double*>(base + L.r12_off);
  double* scal = reinterpret_cast<double*>(base + L.scal_off);
  int* flag = reinterpret_cast<int*>(base + L.flag_off);
  BPDQ_HIP_TRY(bpdq_lds_limit<&panel_pair_kernel>(kPairLdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&hosted_kernel>(kPairLdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&pair_link_kernel>(kGemm64LdsBytes));
  hipLaunchKernelGGL(prep_diag_kernel, dim3(1), dim3(1024), 0, stream, H, d, damp, dead, scal, info);
  BPDQ_LAUNCH_CHECK();
  hipLaunchKernelGGL(prep_load_kernel, dim3(P, P), dim3(256), 0, stream, H, d, scal, A, ld, U);
  BPDQ_LAUNCH_CHECK();
  auto first_block = [&](int t) { return 2 * (n - 1 - t); };
  auto l_slot = [&](int t) { return ring + (size_t)(t % L.slots) * ld * kPairCols; };
  auto x_slot = [&](int t) { return X + (size_t)(t % L.slots) * ld * kPairCols; };
  auto beside = [&](int t) {
    Hosted h{};
    h.inv_p = -1;
    h.U = U;
    h.d = d;
    h.L = ring;
    h.X = X;
    h.t = t;
    h.n = n;
    h.every = L.every;
    if (t >= 1) {
      const int b = first_block(t - 1);
      h.inv_p = b * NB;
      h.inv_r1 = Rdiag + (size_t)b * NB * NB;
      h.inv_r2 = Rdiag + (size_t)(b + 1) * NB * NB;
      h.inv_r12 = R12 + (size_t)(b + 1) * NB * NB;
      h.inv_x = x_slot(t - 1);
    }
    h.plan();
    return h;
  };
  // One work-group to a compute unit.  Those on the compute units that the panel's work-groups leave have `head` rounds
  // of tiles to themselves, the time of the chain; what is left then is for all.  (3584 columns: 1357 us with one such
  // round, 1272 with two, 1242 with three, 1239 with four.  Where a tile takes two or three pairs a round is that much
  // longer: 6016 3772 with one, 3779, 3905 with three; 8192 8095, 8370, 8698.)
  constexpr int kCus = 256;
  const int kHead = L.every == 1 ? 3 : 1;
  // Tiles of the update to leave to the link launch: it has one tile on most compute units and takes a second at 3 us,
  // a round of tiles beside the pair, once there are more than two, takes 10.  (3584 columns: 1286 us if none is left,
  // 1247, 1242 and 1268 if up to 128, 256 and 512 are; 8192: 8148, 8140, 8095, 8170.  From how many rounds on makes no
  // difference: 1239, 1242 and 1238 us from two, three and four.)
  auto spread = [&](Hosted& h, int taken) -> int {              // returns the work-groups
    h.head = kHead;
    h.n_early = (kCus - taken > 64 ? kCus - taken : 64) - (h.inv_p >= 0 ? 1 : 0);
    const int alone = h.n_early * h.head, n_pairs = h.pairs();
    const bool late = n_pairs > alone;
    const int rounds = bpdq_ceil_div(late ? n_pairs - alone : n_pairs, late ? kCus : h.n_early);
    const int over = 2 * ((late ? n_pairs - alone : n_pairs) - (rounds - 1) * (late ? kCus : h.n_early));
    if (rounds + (late ? h.head : 0) > 2 && over <= 256 && over <= h.n_u_far) h.u_skip = over;   // (not the link's columns)
    if (h.pairs() > alone) return kCus;
    return (h.inv_p >= 0 ? 1 : 0) + (h.pairs() < h.n_early ? h.pairs() : h.n_early);
  };
  // behind the pair t: the columns of pair t + 1 by L_t, X[p_{t-1}, :] right of its own columns, what was left over
  auto link = [&](int t, Hosted h) -> int {
    const int n_left = h.u_skip;
    h.u_skip = 0;
    const int u0 = t + 1 < n ? first_block(t + 1) : 0, n_u = t + 1 < n ? 2 * u0 + 3 : 0;
    const int xb = t >= 1 ? first_block(t - 1) : P, n_x = t >= 1 ? 2 * (P - xb - 2) : 0;
    if (n_u + n_x + n_left == 0) return 0;
    hipLaunchKernelGGL(pair_link_kernel, dim3(2 * (n_u + n_x + n_left)), dim3(256), kGemm64LdsBytes, stream, A, ld, l_slot(t), u0,
                       n_u, t >= 1 ? x_slot(t - 1) : X, xb * NB, xb + 2, n_x, h, U, d);
    BPDQ_LAUNCH_CHECK();
    return 0;
  };
  for (int t = 0; t < n; ++t) {
    const int b = first_block(t), panel = b > 0 ? b : 1;
    Hosted h = beside(t);
    const int hosted = spread(h, panel);
    hipLaunchKernelGGL(panel_pair_kernel, dim3(panel + hosted), dim3(kPairThreads), kPairLdsBytes, stream, A, ld,
                       b * NB, NB, b, l_slot(t), kPairCols, panel, h, Rdiag + (size_t)b * NB * NB,
                       Rdiag + (size_t)(b + 1) * NB * NB, R12 + (size_t)(b + 1) * NB * NB, flag + b, flag + b + 1, info);
    BPDQ_LAUNCH_CHECK();
    BPDQ_TRY(link(t, h));
  }
  Hosted h = beside(n);
  const int hosted = spread(h, 0);
  hipLaunchKernelGGL(hosted_kernel, dim3(hosted), dim3(kPairThreads), kPairLdsBytes, stream, A, ld, h);
  BPDQ_LAUNCH_CHECK();
  return link(n, h);
}

extern "C" size_t bpdq_prepare_workspace_bytes(int d_in) {
  if (d_in <= 0) return 0;
  const size_t a = prep_layout(d_in).total, b = sweep_pays(d_in) ? sweep_layout(d_in).total : 0;
  return a > b ? a : b;
}

extern "C" int bpdq_prepare(const float* H, int d_in, float damp, float* U, unsigned char* dead,
                            int* info, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!H) return -1;
  if (d_in <= 0) return -2;
  if (!(damp >= 0.f)) return -3;
  if (!U) return -4;
  if (!info) return -6;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) return -7;
  const PrepLayout L = prep_layout(d_in);
  if (ws_bytes < L.total) return -8;
  char* base = static_cast<char*>(ws);
  if (sweep_pays(d_in) && ws_bytes >= sweep_layout(d_in).total)
    return prepare_by_pairs(H, d_in, damp, U, dead, info, base, stream);
  double* A = reinterpret_cast<double*>(base + L.a_off);
  double* tmp = reinterpret_cast<double*>(base + L.tmp_off);
  double* Rdiag = reinterpret_cast<double*>(base + L.rdiag_off);
  double* scal = reinterpret_cast<double*>(base + L.scal_off);
  double* R12buf = reinterpret_cast<double*>(base + L.r12_off);
  int* pair_flag = reinterpret_cast<int*>(base + L.flag_off);
  const int d = d_in, P = L.P;
  BPDQ_HIP_TRY(bpdq_lds_limit<&panel_pair_kernel>(kPairLdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&syrk_trailing128_kernel>(kGemmLdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&syrk_trailing64_kernel>(kGemm64LdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&tri_inverse_level64_kernel<1>>(kGemm64LdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&tri_inverse_level64_kernel<2>>(kGemm64LdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&tri_inverse_level128_kernel<1>>(kGemmLdsBytes));
  BPDQ_HIP_TRY(bpdq_lds_limit<&tri_inverse_level128_kernel<2>>(kGemmLdsBytes));

  hipLaunchKernelGGL(prep_diag_kernel, dim3(1), dim3(1024), 0, stream, H, d, damp, dead, scal, info);
  BPDQ_LAUNCH_CHECK();
  hipLaunchKernelGGL(prep_load_kernel, dim3(P, P), dim3(256), 0, stream, H, d, scal, A, d, static_cast<float*>(nullptr));
  BPDQ_LAUNCH_CHECK();

  // outer panels of kOuter blocks, from the right; inside one, 64-column panels from the right
  constexpr int kOuter = 8;
  for (int ob1 = P; ob1 > 0; ob1 -= kOuter) {
    const int ob0 = ob1 > kOuter ? ob1 - kOuter : 0;
    int p = ob1 - 1;
    while (p >= ob0) {
      int first_blk, width;                  // blocks [first_blk, p] factored by this launch
      if (p - 1 >= ob0) {                    // a pair of panels
        const int b1 = p - 1, p1 = b1 * NB;
        const int nb2 = (d - p * NB < NB) ? d - p * NB : NB;
        hipLaunchKernelGGL(panel_pair_kernel, dim3(b1 > 0 ? b1 : 1), dim3(kPairThreads), kPairLdsBytes, stream,
                           A, d, p1, nb2, b1, A + p1, d, b1 > 0 ? b1 : 1, Hosted{}, Rdiag + (size_t)b1 * NB * NB,
                           Rdiag + (size_t)p * NB * NB, R12buf + (size_t)p * NB * NB,
                           pair_flag + b1, pair_flag + p, info);
        first_blk = b1;
        width = NB + nb2;
      } else {                               // a single panel (odd count at the left edge)
        const int p0 = p * NB;
        const int nb = (d - p0 < NB) ? d - p0 : NB;
        hipLaunchKernelGGL(panel_factor_kernel, dim3(p > 0 ? p : 1), dim3(256), 0, stream, A, d, p0,
                           nb, p, Rdiag + (size_t)p * NB * NB, pair_flag + p, info);
        first_blk = p;
        width = nb;
      }
      BPDQ_LAUNCH_CHECK();
      if (first_blk > ob0) {
        BPDQ_TRY(launch_trailing(stream, A, d, first_blk * NB, width, ob0, first_blk));
      }
      p = first_blk - 1;
    }
    if (ob0 > 0) {
      const int depth = (ob1 - ob0) * NB;
      BPDQ_TRY(launch_trailing(stream, A, d, ob0 * NB, depth, 0, ob0));
    }
  }

  hipLaunchKernelGGL(diag_inverse_kernel, dim3(P), dim3(256), 0, stream, Rdiag, R12buf, pair_flag, A, d);
  BPDQ_LAUNCH_CHECK();
  const int depth = tree_depth(P);
  for (int dd = depth - 1; dd >= 0; --dd) {
    // at depth dd a node spans at most ceil(P / 2^dd) blocks
    int span = P;
    for (int l = 0; l < dd; ++l) span = (span + 1) / 2;
    const int half = (span + 1) / 2;
    const long tiles128 = ((long)((half + 1) / 2) * ((half + 1) / 2)) << dd;
    if (d % NB == 0 && tiles128 >= kInverse128MinTiles) {
      dim3 grid((half + 1) / 2, (half + 1) / 2, 1 << dd);
      hipLaunchKernelGGL(tri_inverse_level128_kernel<1>, grid, dim3(256), kGemmLdsBytes, stream, A, d, tmp,
                         L.ldt, P, dd);
      BPDQ_LAUNCH_CHECK();
      hipLaunchKernelGGL(tri_inverse_level128_kernel<2>, grid, dim3(256), kGemmLdsBytes, stream, A, d, tmp,
                         L.ldt, P, dd);
      BPDQ_LAUNCH_CHECK();
      continue;
    }
    dim3 grid(half, half, 1 << dd);
    if (d % NB == 0) {
      hipLaunchKernelGGL(tri_inverse_level64_kernel<1>, grid, dim3(256), kGemm64LdsBytes, stream, A, d, tmp, L.ldt, P, dd);
      BPDQ_LAUNCH_CHECK();
      hipLaunchKernelGGL(tri_inverse_level64_kernel<2>, grid, dim3(256), kGemm64LdsBytes, stream, A, d, tmp, L.ldt, P, dd);
      BPDQ_LAUNCH_CHECK();
      continue;
    }
    hipLaunchKernelGGL(tri_inverse_level_kernel<1>, grid, dim3(256), 0, stream, A, d, tmp, L.ldt, P, dd);
    BPDQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(tri_inverse_level_kernel<2>, grid, dim3(256), 0, stream, A, d, tmp, L.ldt, P, dd);
    BPDQ_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(prep_store_kernel, dim3(P, P), dim3(256), 0, stream, A, d, U);
  BPDQ_LAUNCH_CHECK();
  return 0;
}
