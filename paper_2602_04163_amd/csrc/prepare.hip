// Step 2 of the pass: damping and U = chol(H^-1), H^-1 = U^T U with U upper triangular
// (paper Sec. 3.1, "Quantization Error Compensation").
//
// Route: with Ht = H + lambda I, factor Ht = R R^T with R UPPER triangular (a Cholesky
// factorisation that runs from the last column to the first).  Then
// Ht^-1 = R^-T R^-1 = (R^-1)^T (R^-1), so U = R^-1: one factorisation plus one triangular
// inverse (2/3 d^3 flops) and Ht^-1 is never formed.  Everything runs in fp64 inside the
// workspace; the result is rounded to fp32 once, on output.
//
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
__global__ __launch_bounds__(256) void prep_load_kernel(const float* __restrict__ H, int d,
                                                        const double* __restrict__ scal,
                                                        double* __restrict__ A) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj < bi) return;
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
    if (i >= d || j >= d) continue;
    double v = (j >= i) ? (double)h[t] : 0.0;
    if (i == j) v = (h[t] == 0.f ? 1.0 : v) + lam;
    A[(long)i * d + j] = v;
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
template <int J>
__device__ __forceinline__ void eliminate16(double (&a)[16], double (&w)[4], double& raw_own, int i) {
  double row[J > 0 ? J : 1], wr[4];
  const double piv_raw = row_bcast<J>(a[J]);
#pragma unroll
  for (int e = J - 1; e >= 0; --e) row[e] = row_bcast<J>(a[e]);
#pragma unroll
  for (int ks = J / 4; ks < 4; ++ks) wr[ks] = row_bcast<J>(w[ks]);      // columns left of J are still zero in row J
  const double piv = piv_raw > 0.0 ? piv_raw : 1.0;
  if (i == J) raw_own = piv_raw;
  const double t = a[J] * fast_rcp(piv);
#pragma unroll
  for (int e = J - 1; e >= 0; --e) a[e] = fma(-t, row[e], a[e]);
  const double tm = (i < J) ? t : 0.0;
#pragma unroll
  for (int ks = J / 4; ks < 4; ++ks) w[ks] = fma(-tm, wr[ks], w[ks]);
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
__device__ __forceinline__ void factor64_blocked(double (*sD)[NB + 1], Inv16* sRinv, int* info, int p0, bool report,
                                                 bool active = true) {
  if (!active) {                            // the other team of a 512-thread work-group keeps the barriers company
#pragma unroll 1
    for (int n = 0; n < 2 * (NB / 16) + 1; ++n) __syncthreads();
    return;
  }
  const int lane = threadIdx.x & 63, w = team_wave();
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
      f64x4 x = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) x = __builtin_amdgcn_mfma_f64_16x16x4f64(at[ks], wi[ks], x, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) sD[16 * w + 4 * r + q][c0 + m] = x[r];
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
    int t = 0;
    for (int tk = J - 1; tk >= 0; --tk)     // the next panel's tiles first
      for (int ti = tk; ti >= 0; --ti, ++t) {
        if ((t & 3) != w) continue;
        f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sD[16 * ti + m][c0 + 4 * ks + q], sD[16 * tk + m][c0 + 4 * ks + q],
                                                     acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) sD[16 * ti + 4 * r + q][16 * tk + m] -= acc[r];
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
template <int J>
__device__ __forceinline__ void trsm_block_step(double (*sX)[NB + 1], const double (*sR)[NB + 1], const Inv16* sRinv) {
  const int lane = threadIdx.x & 63, i0 = 16 * team_wave();
  const int lm = lane & 15, lq = lane >> 4;
  double a[4];
  f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)                                                    // A[m][k] = A_J, B[k][n] = Rinv[n][k]
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[i0 + lm][16 * J + 4 * ks + lq], sRinv[J][lm][4 * ks + lq], acc, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) sX[i0 + 4 * r + lq][16 * J + lm] = acc[r];            // D[4r + l/16][l%16]
  if constexpr (J > 0) {
    // X_J back in operand layout (this wavefront's own rows: LDS serves a wavefront in order)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[ks] = sX[i0 + lm][16 * J + 4 * ks + lq];
    f64x4 upd[J];
#pragma unroll
    for (int Jp = 0; Jp < J; ++Jp) {
      upd[Jp] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)                                                // B[k][n] = R[J'n][Jk]
        upd[Jp] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], sR[16 * Jp + lm][16 * J + 4 * ks + lq], upd[Jp], 0, 0, 0);
    }
#pragma unroll
    for (int Jp = 0; Jp < J; ++Jp)
#pragma unroll
      for (int r = 0; r < 4; ++r) sX[i0 + 4 * r + lq][16 * Jp + lm] -= upd[Jp][r];
    trsm_block_step<J - 1>(sX, sR, sRinv);
  }
}

__device__ __forceinline__ void trsm64_blocked(double (*sX)[NB + 1], const double (*sR)[NB + 1], const Inv16* sRinv) {
  trsm_block_step<NB / 16 - 1>(sX, sR, sRinv);
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
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
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

template <bool B_T>
__device__ __forceinline__ void quad_mfma_64(const double (*sa)[NB + 1], const double (*sb)[NB + 1],
                                             Quad64& q) {
  const int lane = threadIdx.x & 63, w = team_wave();
  const int m0 = (w >> 1) * 32 + (lane & 15), n0 = (w & 1) * 32 + (lane & 15);
  const int kq = lane >> 4;
#pragma unroll 4
  for (int k0 = 0; k0 < NB; k0 += 4) {
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

// Two adjacent 64-column panels -- block b1 (columns p1 ..) and block b2 = b1 + 1 -- in one
// launch, one work-group per 64 rows above them.  With the diagonal 128 x 128 block
// [D11 D12; D12^T D22] every work-group computes for itself
//     D22 = R22 R22^T,   R12 = D12 R22^-T,   D11 - R12 R12^T = R11 R11^T
// and for its own rows [A1 A2] of the two panels
//     X2 = A2 R22^-T,    X1 = (A1 - X2 R12^T) R11^-T.
// The solves and products run on the fp64 matrix cores.  This halves the number of dependent launches of
// the panel chain (each is short and latency-bound).  A work-group is two teams of four wavefronts: the
// first walks the chain of the diagonal block, the second solves and updates the work-group's rows beside it
// and stores what is finished, so that of the rows only the last solve comes after the chain (one team that
// did both in turn took 40.5 us a launch at d = 3584, two take 34.4).  Work-group 0 writes R11, R22 to
// Rdiag and R12 to R12buf (never into A, whose blocks later-scheduled work-groups still read) and sets the
// pair flag of b2, so that the inverse step puts R12 in place.
constexpr size_t kPairLdsBytes = (size_t)(4 * NB * (NB + 1) + NB * 16) * sizeof(double);
constexpr int kPairThreads = 512;

__global__ __launch_bounds__(kPairThreads) void panel_pair_kernel(double* __restrict__ A, int d, int p1,
                                                                  int nb2, int n_above,
                                                                  double* __restrict__ Rdiag1,
                                                                  double* __restrict__ Rdiag2,
                                                                  double* __restrict__ R12buf,
                                                                  int* __restrict__ pair_flag1,
                                                                  int* __restrict__ pair_flag2, int* info) {
  extern __shared__ double dyn[];
  typedef double Row[NB + 1];
  Row* sR = reinterpret_cast<Row*>(dyn);            // R22, then R11
  Row* sR12 = sR + NB;                              // D12 -> R12
  Row* sA1 = sR12 + NB;                             // own rows, columns of b1
  Row* sA2 = sA1 + NB;                              // own rows, columns of b2
  Inv16* sRinv = reinterpret_cast<Inv16*>(dyn + 4 * NB * (NB + 1));
  const int tid = team_tid();
  const bool chain = threadIdx.x < 256;             // team of the diagonal block; the other has the rows
  const int p2 = p1 + NB;
  const int r0 = blockIdx.x * NB;
  const bool first = blockIdx.x == 0, rows = n_above > 0;
  const bool vec = nb2 == NB && d % 2 == 0;

  Quad64 d11;                                       // D11 in the product's layout, needed after the first factorisation
  quad_zero(d11);
  if (chain) {
    double v22[16], v12[16];
    fetch_tile(A, d, p2, p2, nb2, nb2, true, vec, v22);
    fetch_tile(A, d, p1, p2, NB, nb2, false, vec, v12);
    const int lane = threadIdx.x & 63, w = team_wave();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          d11.c[i][j][r] = A[(long)(p1 + (w >> 1) * 32 + 16 * i + 4 * r + (lane >> 4)) * d + p1 + (w & 1) * 32 + 16 * j +
                             (lane & 15)];
    put_tile(sR, vec, v22);
    put_tile(sR12, vec, v12);
  } else if (rows) {                                // (the rows above a full panel are all there)
    double v1[16], v2[16];
    fetch_tile(A, d, r0, p2, NB, nb2, false, vec, v2);
    fetch_tile(A, d, r0, p1, NB, NB, false, vec, v1);
    put_tile(sA2, vec, v2);
    put_tile(sA1, vec, v1);
  }
  factor64_blocked(sR, sRinv, info, p2, first, chain);
  // R12 = D12 R22^-T and X2 = A2 R22^-T
  if (chain) {
    trsm64_blocked(sR12, sR, sRinv);
  } else {
    if (first)
      for (int e = tid; e < NB * NB; e += 256) Rdiag2[e] = sR[e / NB][e % NB];
    if (rows) trsm64_blocked(sA2, sR, sRinv);
  }
  __syncthreads();
  if (chain) {
    Quad64 q;
    quad_zero(q);
    quad_mfma_64<true>(sR12, sR12, q);              // D11 - R12 R12^T  (R22 is no longer needed)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) q.c[i][j] = d11.c[i][j] - q.c[i][j];
    quad_for_each(q, [&](int r, int c, double v) { sR[r][c] = v; });
  } else {
    if (rows) {
      Quad64 q;
      quad_zero(q);
      quad_mfma_64<true>(sA2, sR12, q);             // A1 - X2 R12^T
      quad_for_each(q, [&](int r, int c, double v) { sA1[r][c] -= v; });
      for (int e = tid; e < NB * NB; e += 256) {    // X2 is finished
        const int i = e / NB, j = e % NB;
        if (j < nb2) A[(long)(r0 + i) * d + p2 + j] = sA2[i][j];
      }
    }
    if (first)
      for (int e = tid; e < NB * NB; e += 256) R12buf[e] = sR12[e / NB][e % NB];
  }
  factor64_blocked(sR, sRinv, info, p1, first, chain);
  if (first && !chain) {
    for (int e = tid; e < NB * NB; e += 256) Rdiag1[e] = sR[e / NB][e % NB];
    if (tid == 0) {
      *pair_flag1 = 0;
      *pair_flag2 = 1;
    }
  }
  if (!rows) return;
  if (chain) trsm64_blocked(sA1, sR, sRinv);
  __syncthreads();
  for (int e = threadIdx.x; e < NB * NB; e += kPairThreads) {
    const int i = e / NB, j = e % NB;
    A[(long)(r0 + i) * d + p1 + j] = sA1[i][j];
  }
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
// passed in M0, which these kernels use for nothing else).  One outstanding vector-memory operation.
__device__ __forceinline__ void dma_1k_f64(const double* gptr, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(gptr) : "memory");
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
// For launches with too few 128-tiles to fill the chip: the layers up to 4096 columns, the updates inside
// an outer block, the lower levels of the inversion tree.  256 threads own 64 x 64 results, wavefront w the
// 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 tiles.  Such launches are short and their work-groups few, so
// what bounds them is memory latency: a ring of four slices of 16 (64 KB of LDS, two work-groups per CU)
// keeps three in flight, against one 64-deep chunk staged through registers.  At d = 3584
// the trailing updates take 550 us instead of 675 and the inversion products 430 instead of 670.
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
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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

// Below this many column blocks the 64-tile kernel has more work-groups to spread over the chip.
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

extern "C" size_t bpdq_prepare_workspace_bytes(int d_in) {
  if (d_in <= 0) return 0;
  return prep_layout(d_in).total;
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
  hipLaunchKernelGGL(prep_load_kernel, dim3(P, P), dim3(256), 0, stream, H, d, scal, A);
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
                           A, d, p1, nb2, b1, Rdiag + (size_t)b1 * NB * NB,
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
