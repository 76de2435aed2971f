// Step 1 of the pass: calibration Hessian H += scale * Xc^T Xc (paper Sec. 3.1, H = X X^T).
//
// A symmetric rank-k update on the matrix cores, in three kernels that share everything but the
// tile product: fp32 MFMAs (bpdq_hessian_accumulate_f32), bf16 MFMAs on three exact bf16 pieces
// of every value (bpdq_hessian_accumulate_bf16x3; mfma_split_bf16.h), or fp16 MFMAs on two fp16
// halves of every value, split and laid out in operand order by a streaming pre-pass
// (bpdq_hessian_accumulate; mfma_split_f16.h; its small calls are one launch of their own,
// hess_small_kernel, which has none of what follows).  Only the upper triangle
// of 256 x 256 tiles is computed, and of a diagonal tile only the 32 x 32 blocks on or above the diagonal.
// The token axis is cut into deterministic slices so that the work-groups fill the 256 compute
// units in whole rounds: off-diagonal tiles into S_off slices, diagonal tiles (5/8 of the work
// per token) into fewer, longer slices S_diag, so that every work-group costs about the same.
// Slice partials go to the workspace and are summed in a fixed order (no float atomics, so H is
// bit-reproducible).
#include <type_traits>

#include "mfma_kmajor.h"
#include "mfma_split_bf16.h"
#include "mfma_split_f16.h"

namespace bpdq {

constexpr int kNumCU = 256;   // MI355X: 8 XCDs x 32 compute units
constexpr int kNumXCD = 8;
constexpr int kTileFloats = HessGemm::kTileM * HessGemm::kTileN;

struct HessPlan {
  int nb;               // tile rows / cols
  int n_off, n_diag;    // off-diagonal and diagonal tiles of the upper triangle
  int S_off, S_diag;    // token slices per off-diagonal / diagonal tile
  int k_off, k_diag;    // tokens per slice (multiples of the stage depth)
  bool direct;          // one slice each: accumulate into H without partials
  int items() const { return n_off * S_off + n_diag * S_diag; }
  size_t ws_bytes() const { return direct ? 0 : (size_t)items() * kTileFloats * sizeof(float); }
};

// Makespan (us) of the busiest XCD: work-groups go round-robin to the XCDs and, inside one, to
// the first free of its 32 compute units; all off-diagonal slices are dispatched first.
static double hess_makespan(int n_full, double c_full, int n_short, double c_short) {
  const int per = kNumCU / kNumXCD;
  const int nf = bpdq_ceil_div(n_full, kNumXCD), ns = bpdq_ceil_div(n_short, kNumXCD);
  double free_at[kNumCU / kNumXCD];
  const int q = nf / per, r = nf % per;
  for (int i = 0; i < per; ++i) free_at[i] = (q + (i < r ? 1 : 0)) * c_full;
  for (int j = 0; j < ns; ++j) {
    int m = 0;
    for (int i = 1; i < per; ++i)
      if (free_at[i] < free_at[m]) m = i;
    free_at[m] += c_short;
  }
  double t = 0.0;
  for (int i = 0; i < per; ++i) t = free_at[i] > t ? free_at[i] : t;
  return t;
}

// Measured: a sum of squares (the diagonal of H) accumulated by chained MFMAs comes out low, the
// more so the longer the chain: about -9e-7 relative after 16 k tokens on the fp32 path, -4.5e-6 after
// 52 k tokens and -2.5e-6 after 8 k tokens on the bf16 path, -2.8e-7 after 8 k tokens on the fp16 path.  On the fp32 path
// that is what fp32 sums do: the instruction is an ascending chain of fused multiply-adds rounded to nearest, bit
// for bit (256 x 256 entries after 511, 4096 and 16384 tokens of widely spread sizes).  How the 16-bit instructions round
// inside was not established.  All paths end every
// chain after kChainTokens[kind] tokens; the partial sums are added by ordinary fp32 additions, few enough not to drift.
constexpr int kChainTokens[3] = {16384, 8192, 8192};
constexpr int kMaxSlices = 64;

// kind 0: fp32 MFMA kernel; kind 1: split-bf16 kernel (about 1.8 times the rate per token);
// kind 2: pre-split fp16 kernel (about twice the rate of kind 1)
enum : int { kKindF32 = 0, kKindBf16x3 = 1, kKindF16x2 = 2, kNumKinds = 3 };

// fine: slices down to 64 tokens (fp16 path), which takes more partial tiles than the 256-token slices that a
// workspace may have been sized for; see hessian_accumulate.
static HessPlan plan_hessian(int n_tok, int d_in, int kind, bool fine) {
  // the last plan of each kind, per host thread: a stream of equal calls plans once
  constexpr int kSlots = 2 * kNumKinds;
  thread_local HessPlan cache[kSlots];
  thread_local int cache_n[kSlots] = {-1, -1, -1, -1, -1, -1}, cache_d[kSlots] = {-1, -1, -1, -1, -1, -1};
  const int slot = kind + (fine ? kNumKinds : 0);
  if (n_tok == cache_n[slot] && d_in == cache_d[slot]) return cache[slot];
  HessPlan p;
  p.nb = bpdq_ceil_div(d_in, HessGemm::kTileM);
  p.n_diag = p.nb;
  p.n_off = p.nb * (p.nb - 1) / 2;
  p.S_off = p.S_diag = 1;
  p.k_off = p.k_diag = (int)bpdq_align_up((size_t)(n_tok > 0 ? n_tok : 1), HessGemm::kStageK);
  p.direct = true;
  if (n_tok > 0 && p.n_off + p.n_diag < 4 * kNumCU) {
    // per-token MFMA time of one 256 x 256 tile, fixed cost per work-group, cost per partial tile
    constexpr double kUsPerTok[kNumKinds] = {0.26, 0.14, 0.055};
    constexpr double kDiagFrac[kNumKinds] = {0.64, 0.64, 0.60};
    const double us_per_tok = kUsPerTok[kind], us_fixed = 8.0, us_per_partial = 0.131;
    const double diag_frac = kDiagFrac[kind];
    // shortest slice: 64 tokens where the pre-pass has made a stage cheap (a call of 512 tokens on 256
    // channels is one tile: 2 slices took 13 us, 6 take 10), 256 otherwise
    const int min_slice = fine && kind == kKindF16x2 ? 64 : 256;
    const int s_max = n_tok / min_slice < kMaxSlices ? (n_tok / min_slice < 1 ? 1 : n_tok / min_slice) : kMaxSlices;
    // every accumulation chain stays short (see kChainTokens)
    int s_min = bpdq_ceil_div(n_tok, kChainTokens[kind]);
    if (s_min > s_max) s_min = s_max;
    double best = 1e300;
    for (int So = s_min; So <= s_max; ++So) {
      // More slices only add to the fixed and the partial-tile cost.  Once these and an even spread of the
      // products over the chip (no makespan is below that; 1e-9 for the rounding of the sums) exceed the best,
      // no later So can win: the plan of a search to s_max at a fraction of its host time (4096 x 3584, fp16 path:
      // 309 us -> 1.5; all three kinds through the size query: 430 -> 20).  A program whose calls differ in shape pays
      // this each time.
      const int Sd_least = (int)(So * 0.625 + 0.5) - 1 > s_min ? (int)(So * 0.625 + 0.5) - 1 : s_min;
      const double products = (double)n_tok * us_per_tok * (p.n_off + p.n_diag * diag_frac);
      const double least = (products + (double)(p.n_off * So + p.n_diag * Sd_least) * us_fixed) / kNumCU +
                           (So > 1 ? (double)(p.n_off * So + p.n_diag * Sd_least) * us_per_partial : 0.0);
      if (least * (1.0 - 1e-9) >= best * 0.998) break;
      for (int dd = -1; dd <= 1; ++dd) {
        int Sd = (int)(So * 0.625 + 0.5) + dd;
        if (Sd < s_min) Sd = s_min;
        if (Sd > s_max) Sd = s_max;
        const int ko = (int)bpdq_align_up((size_t)bpdq_ceil_div(n_tok, So), HessGemm::kStageK);
        const int kd = (int)bpdq_align_up((size_t)bpdq_ceil_div(n_tok, Sd), HessGemm::kStageK);
        double t = hess_makespan(p.n_off * So, ko * us_per_tok + us_fixed, p.n_diag * Sd,
                                 kd * us_per_tok * diag_frac + us_fixed);
        if (So > 1 || Sd > 1) t += (double)(p.n_off * So + p.n_diag * Sd) * us_per_partial;
        if (t < best * 0.998) {
          best = t;
          p.S_off = So; p.S_diag = Sd; p.k_off = ko; p.k_diag = kd;
        }
      }
    }
    p.direct = (p.S_off == 1 && p.S_diag == 1);
  }
  cache[slot] = p; cache_n[slot] = n_tok; cache_d[slot] = d_in;
  return p;
}

// Tile orders.  The 32 tiles an XCD has in flight stream their 256-channel panels through its L2,
// so an order is as good as the number of different panels a run of 32 consecutive tiles meets.
// The triangle is cut into blocks of kTileBlock panels: the blocks on the diagonal are cliques
// (every pair of kTileBlock panels: 28 tiles on 8 panels), the others kTileBlock x kTileBlock
// squares (64 tiles on 16 panels); blocks are taken column by column, tiles row-major inside.
// On 74 x 74 tiles a run of 32 meets 13 panels on average, in plain row-major order 32.  Measured
// against row-major in one process: 6.5 % less time at 116 x 116 tiles, 2-3 % at 74 and 32, none at 14.
constexpr int kTileBlock = 8;

// seq-th tile of that order -> (bi, bj).  DIAG: the diagonal tiles are part of the sequence
// (bi <= bj), else only bi < bj.  seq must be below the number of such tiles.
template <bool DIAG>
__device__ __forceinline__ void block_order_tile(int seq, int nb, int& bi, int& bj) {
  const int n_blk = bpdq_ceil_div(nb, kTileBlock);
  bi = bj = 0;
  for (int bc = 0; bc < n_blk; ++bc) {
    const int c0 = bc * kTileBlock, mc = (c0 + kTileBlock < nb ? kTileBlock : nb - c0);
    // the column of blocks above the diagonal one: bc full squares of kTileBlock x mc tiles
    const int above = bc * kTileBlock * mc;
    if (seq < above) {
      const int br = seq / (kTileBlock * mc), t = seq % (kTileBlock * mc);
      bi = br * kTileBlock + t / mc;
      bj = c0 + t % mc;
      return;
    }
    seq -= above;
    const int clique = DIAG ? mc * (mc + 1) / 2 : mc * (mc - 1) / 2;
    if (seq < clique) {
      for (int r = 0; r < mc; ++r) {
        const int cnt = DIAG ? mc - r : mc - 1 - r;
        if (seq < cnt) {
          bi = c0 + r;
          bj = c0 + r + (DIAG ? 0 : 1) + seq;
          return;
        }
        seq -= cnt;
      }
    }
    seq -= clique;
  }
}

// off-diagonal tile index -> (bi, bj), bi < bj
__device__ __forceinline__ void decode_off_tile(int tile, int nb, int& bi, int& bj) {
  block_order_tile<false>(tile, nb, bi, bj);
}

// Work-group -> work item.  Work-groups are handed to the 8 XCDs round-robin (work-group w runs
// on XCD w % 8), each XCD has its own L2, and items are numbered slice-major (item = slice *
// tiles + tile).  Taken in that order every XCD would work on all token slices at once and each
// L2 would stream the whole of X: 8 x the traffic.  Instead XCD x takes the slices congruent to
// x modulo 8, tile after tile: the work-groups running on an XCD at one time walk the same
// tokens in step, its L2 serves every 256-channel block of a stage to all of them from one
// fetch, and each token is fetched by one XCD only.  Slices beyond the last multiple of 8 keep
// the plain order.  The map is a bijection on the items, so partials and reduction are unchanged.
__device__ __forceinline__ int xcd_item(int w, int n_off_items, const HessPlan& p) {
  int base = 0, tiles = p.n_off, slices = p.S_off;
  if (w >= n_off_items) {
    base = n_off_items;
    tiles = p.n_diag;
    slices = p.S_diag;
  }
  const int j = w - base;
  const int grouped = tiles * (slices / kNumXCD) * kNumXCD;   // items of the slices that are remapped
  if (j >= grouped) return w;
  // j % 8 names the XCD up to a fixed rotation (base need not be a multiple of 8)
  const int y = j % kNumXCD, q = j / kNumXCD;
  return base + ((q / tiles) * kNumXCD + y) * tiles + q % tiles;
}

// Tile order of a launch without token slices (wide layers: more tiles than the chip runs at
// once): the block order above over the whole upper triangle, diagonal tiles included, and XCD x
// takes the runs of 32 numbered x, x + 8, ... of that sequence (work-group w runs on XCD w % 8).
// Work-group w -> tile; false beyond the last tile.
__host__ __device__ inline int direct_grid(int nb) {
  const int tiles = nb * (nb + 1) / 2;
  return bpdq_ceil_div(tiles, kNumCU) * kNumCU;
}
__device__ __forceinline__ bool direct_tile(int w, int nb, int& bi, int& bj) {
  const int per = kNumCU / kNumXCD;                       // 32
  const int x = w % kNumXCD, n = w / kNumXCD;
  const int seq = ((n / per) * kNumXCD + x) * per + n % per;
  if (seq >= nb * (nb + 1) / 2) return false;
  block_order_tile<true>(seq, nb, bi, bj);
  return true;
}

// SPLIT false: fp32 matrix cores (v_mfma_f32_32x32x2_f32); true: three bf16 pieces per value and
// six bf16 products per fp32 product (v_mfma_f32_32x32x16_bf16), same accumulator layout.
template <bool SPLIT>
__device__ __forceinline__ void hess_syrk_body(const float* __restrict__ X, int n_tok, int d,
                                               long ldx, float scale, float* __restrict__ H,
                                               float* __restrict__ partial, const HessPlan& p) {
  const int n_off_items = p.n_off * p.S_off;
  const int item = xcd_item(blockIdx.x, n_off_items, p);
  int bi, bj, k_begin, k_end;
  if (item < n_off_items) {
    decode_off_tile(item % p.n_off, p.nb, bi, bj);
    k_begin = (item / p.n_off) * p.k_off;
    k_end = min(n_tok, k_begin + p.k_off);
  } else {
    const int j = item - n_off_items;
    bi = bj = j % p.n_diag;
    k_begin = (j / p.n_diag) * p.k_diag;
    k_end = min(n_tok, k_begin + p.k_diag);
  }
  HessGemm::Acc acc;
  HessGemm::zero(acc);
  const int r0 = bi * HessGemm::kTileM, c0 = bj * HessGemm::kTileN;
  // diagonal tile: only the 32 x 32 blocks on or above the diagonal are computed
  if (bi == bj) {
    if constexpr (SPLIT) SplitSyrk::run<true>(X, ldx, r0, c0, d, k_begin, k_end, acc);
    else HessGemm::run<2>(X, ldx, r0, d, X, ldx, c0, d, k_begin, k_end, acc);
  } else {
    if constexpr (SPLIT) SplitSyrk::run<false>(X, ldx, r0, c0, d, k_begin, k_end, acc);
    else HessGemm::run<0>(X, ldx, r0, d, X, ldx, c0, d, k_begin, k_end, acc);
  }
  if (p.direct) {
    auto emit = [&](int row, int col, float v) {
      const int r = r0 + row, c = c0 + col;
      if (r < d && c < d) H[(long)r * d + c] += scale * v;
    };
    if (bi == bj) HessGemm::for_each_diag(acc, emit);
    else HessGemm::for_each(acc, emit);
  } else {
    float* out = partial + (long)item * kTileFloats;
    auto emit = [&](int row, int col, float v) { out[row * HessGemm::kTileN + col] = v; };
    if (bi == bj) HessGemm::for_each_diag(acc, emit);
    else HessGemm::for_each(acc, emit);
  }
}

__global__ __launch_bounds__(HessGemm::kThreads) void hess_syrk_f32_kernel(
    const float* __restrict__ X, int n_tok, int d, long ldx, float scale, float* __restrict__ H,
    float* __restrict__ partial, HessPlan p) {
  hess_syrk_body<false>(X, n_tok, d, ldx, scale, H, partial, p);
}

__global__ __launch_bounds__(SplitSyrk::kThreads) void hess_syrk_bf16x3_kernel(
    const float* __restrict__ X, int n_tok, int d, long ldx, float scale, float* __restrict__ H,
    float* __restrict__ partial, HessPlan p) {
  hess_syrk_body<true>(X, n_tok, d, ldx, scale, H, partial, p);
}

// ---- pre-pass of the fp16 path ---------------------------------------------------------------
// (1) per-channel largest magnitude, as partial maxima over token ranges; of a large call, of every kSampleStep-th token;
// (2) per channel the power of two that brings that maximum into [2^13, 2^14) (so every half is
//     far from the ends of the fp16 range whatever the activations' units), and its inverse;
// (3) the split itself: X -> planes[piece][token / 8][channel] (see mfma_split_f16.h), zeros for
//     the tokens up to the next multiple of 32 and the channels up to the next multiple of 256.
// Bound by HBM: with a sample X is read 17/16 times and the planes are written, 262144 x 3584 in 1.5 ms against 2.07 with a
// pass for the maxima of all tokens in front.
// A sample's largest is at most the channel's, so its factor is at least that of all tokens: no half is coarser for it.
// What it may miss is values of more than 4 to 8 times its largest, which leave the half range.  The split looks for them and
// takes the maximum of a channel that has one; a second split then does the runs of 16 channels that hold such a
// channel again, with the factor of all tokens for that channel, and ends at once for the others.  Where a run is known
// to hold one, the first split reads on for the maxima and no longer writes: the two together are then the pass over all
// tokens and the split behind it.  They write planes twice where the values come late.
// Runs of 16 channels are whole lines of the planes and half lines of X.  262144 x 3584, Student-t(4) tokens / one late value
// in every 64 channels, us: runs of 64 channels 9763 / 10473, 32 9558 / 9638, 16 9485 / 9493, single channels 9791 / 9461; the pass
// over all tokens 9488.  Every 8th, 16th, 32nd token: 9246, 9485, 9628 on Student-t(4) tokens; the sample itself takes 113 us with
// every 8th, 64 with every 16th.
constexpr int kSampleStep = 16;
// Values (tokens times channels) from which on the scales come from a sample.  us on activations not read before, scales of all
// tokens / of a sample on normal tokens / on Student-t(4) tokens / one late value in every 64 channels / in every channel:
//   262144 x 3584 9544 / 9007 / 9540 / 9503 / 10451;  65536 x 3584 2410 / 2263 / 2405 / 2432 / 2612;
//   131072 x 1024 618 / 548 / 647 / 642 / 748;  16384 x 8192 2762 / 2655 / 2802 / 2750 / 2848;  8192 x 18944 6635 / 6508 / 6670 / 6630 / 6691;
// and below the line
//   32768 x 3584 1216 / 1139 / 1227 / 1228 / 1320;  65536 x 1024 332 / 299 / 333 / 340 / 388;  8192 x 8192 1597 / 1552 / 1607 / 1603 / 1652;
//   16384 x 3584 639 / 606 / 639 / 636 / 684;  65536 x 256 106 / 88 / 101 / 104 / 109.
// So the gain on tokens without outliers does not end at the line; below it a call's time follows from its size alone.
constexpr long kSampleValues = 1L << 27;
constexpr int kColmaxRows = 1024;      // tokens per partial maximum
constexpr int kSplitKgPerWG = 16;      // k-groups (8 tokens each) per work-group of the split
constexpr float kHalfMax = 65504.0f;
constexpr int kBeyondWGs = 8192;       // work-groups of the second split
enum : int { kAllTokens = 0, kSampled = 1, kBeyond = 2 };       // maxima of all tokens; of a sample; the second split

template <bool SAMPLED>
__global__ __launch_bounds__(256) void hess_colmax_kernel(const float* __restrict__ X, int n_tok, int d,
                                                          long ldx, float* __restrict__ pmax, int d_pad) {
  constexpr int kStep = SAMPLED ? kSampleStep : 1, kFlight = SAMPLED ? 16 : 8;
  __shared__ float4 red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = blockIdx.x * 256 + lane * 4;
  const int t0 = blockIdx.y * kColmaxRows;
  const int t1 = min(n_tok, t0 + kColmaxRows);
  float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c < d) {                                    // d % 4 == 0: the float4 is inside the row
    const float* p = X + c;
    for (int t = t0 + wave * kStep; t < t1; t += 4 * kFlight * kStep) {    // kFlight rows of this wavefront in flight
      float4 v[kFlight];
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int tt = min(t + 4 * u * kStep, t1 - 1);    // past the end: the last row again
        v[u] = *reinterpret_cast<const float4*>(p + (long)tt * ldx);
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        m.x = fmaxf(m.x, fabsf(v[u].x)); m.y = fmaxf(m.y, fabsf(v[u].y));
        m.z = fmaxf(m.z, fabsf(v[u].z)); m.w = fmaxf(m.w, fabsf(v[u].w));
      }
    }
  }
  red[wave][lane] = m;
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 o = red[w][lane];
      m.x = fmaxf(m.x, o.x); m.y = fmaxf(m.y, o.y); m.z = fmaxf(m.z, o.z); m.w = fmaxf(m.w, o.w);
    }
    *reinterpret_cast<float4*>(pmax + (long)blockIdx.y * d_pad + c) = m;     // c < d_pad always
  }
}

// exponent of the power of two that brings a channel's largest magnitude into [2^13, 2^14)
__device__ __forceinline__ int channel_exponent(float m) {
  int e = 0;
  if (m > 0.f && m < 3.0e38f) {
    int ex;
    (void)frexpf(m, &ex);           // m = f * 2^ex, f in [0.5, 1)
    e = 14 - ex;                    // m * 2^e in [2^13, 2^14)
    e = e > 100 ? 100 : (e < -100 ? -100 : e);
  }
  return e;
}

// A sample also clears row 0 of the partial maxima, which then takes the maxima of channels with values beyond the range.
template <bool SAMPLED>
__global__ __launch_bounds__(256) void hess_scale_kernel(float* pmax, int n_split,
                                                         int d_pad, float* __restrict__ mul,
                                                         float* __restrict__ inv) {
  // 16 channels per work-group, the partial maxima of a channel dealt to 16 threads
  __shared__ float red[16][16];
  const int c = blockIdx.x * 16 + (threadIdx.x & 15), q = threadIdx.x >> 4;
  float m = 0.f;
  for (int s = q; s < n_split; s += 16) m = fmaxf(m, pmax[(long)s * d_pad + c]);
  red[q][threadIdx.x & 15] = m;
  __syncthreads();
  if (q) return;
#pragma unroll
  for (int w = 1; w < 16; ++w) m = fmaxf(m, red[w][threadIdx.x]);
  // a sample of zeros says nothing: the largest factor, under which anything that counts is out of range
  const int e = SAMPLED && m == 0.f ? 100 : channel_exponent(m);
  mul[c] = ldexpf(1.0f, e);
  inv[c] = ldexpf(1.0f, -e);
  if (SAMPLED) pmax[c] = 0.f;
}

__device__ __forceinline__ unsigned pack_halves(_Float16 a, _Float16 b) {
  return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}

// operand vectors of eight values scaled by s: the high and the low halves, zeros from `count` values on
__device__ __forceinline__ void split_halves(const float (&x)[8], float s, int count, uint4& hv, uint4& lv) {
  unsigned hw[4], lw[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    _Float16 h[2], l[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float xs = (2 * q + e < count) ? x[2 * q + e] * s : 0.f;
      h[e] = (_Float16)xs;                       // round to nearest even
      l[e] = (_Float16)(xs - (float)h[e]);       // exact difference, then rounded
    }
    hw[q] = pack_halves(h[0], h[1]);
    lw[q] = pack_halves(l[0], l[1]);
  }
  hv = make_uint4(hw[0], hw[1], hw[2], hw[3]);
  lv = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

// any of the run of 16 lanes
__device__ __forceinline__ bool any_of_run(bool b) { return ((__ballot(b) >> (threadIdx.x & 48)) & 0xffffu) != 0; }

// top (kSampled: written, kBeyond: read): per channel 0, or the largest magnitude of all tokens where that, scaled, is beyond the
// half range.  (Non-negative floats order like their bits; a NaN, which the maximum passes over, needs no other factor.)
template <int TURN>
__global__ __launch_bounds__(256) void hess_split_f16_kernel(const float* __restrict__ X, int n_tok, int d,
                                                             long ldx, const float* __restrict__ mul, float* __restrict__ inv,
                                                             unsigned* top, uint4* __restrict__ planes, long n_kg,
                                                             int d_pad) {
  const int ch = blockIdx.x * 256 + threadIdx.x;
  const bool live = ch < d;
  const int chc = live ? ch : d - 1;
  float s = mul[chc];
  bool write = true;
  if constexpr (TURN == kSampled)                 // known already: the second split writes the channel
    write = !any_of_run(__hip_atomic_load(top + ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u);
  if constexpr (TURN == kBeyond) {
    const float m = __builtin_bit_cast(float, top[ch]);
    if (!any_of_run(m != 0.f)) return;
    if (m != 0.f) {
      const int e = channel_exponent(m);
      s = ldexpf(1.0f, e);
      if (blockIdx.y == 0) inv[ch] = ldexpf(1.0f, -e);
    }
  }
  const float* p = X + chc;
  const int t_last = n_tok - 1;
  float m = 0.f;
  for (long kg0 = (long)blockIdx.y * kSplitKgPerWG; kg0 < n_kg; kg0 += (long)gridDim.y * kSplitKgPerWG) {
    for (int g = 0; g < kSplitKgPerWG; g += 2) {
      const long kg = kg0 + g;
      if (kg >= n_kg) break;
      float x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const long t = 8 * kg + i;
        x[i] = p[(t < t_last ? t : (long)t_last) * ldx];
      }
      if constexpr (TURN == kSampled) {
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(x[i]));      // (tokens past the end repeat the last)
        if (!write) continue;
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (kg + half >= n_kg) break;
        uint4 hv, lv;
        split_halves(reinterpret_cast<const float(&)[8]>(x[8 * half]), s, live ? n_tok - 8 * (int)(kg + half) : 0, hv, lv);
        planes[(kg + half) * d_pad + ch] = hv;
        planes[(n_kg + kg + half) * d_pad + ch] = lv;
      }
    }
  }
  if constexpr (TURN == kSampled)
    if (live && m * s > kHalfMax) atomicMax(top + ch, __builtin_bit_cast(unsigned, m));
}

// The whole pre-pass in one launch for calls of at most 4096 tokens: a work-group holds all tokens of 16
// channels in registers (NI times 8 floats per thread), so X is read once and the maximum, the scale and the
// split need no second pass and no launches of their own.  Bound by HBM: X read once, the planes written
// once.  Thread (lane % 16) = channel, the 64 others = k-groups of 8 consecutive tokens, so a thread's
// eight values are one operand vector.  A row segment is 64 bytes, half a cache line: neighbouring
// channel blocks run on the same XCD (work-group w runs on XCD w % 8), whose L2 then serves both halves
// from one fetch.  4096 x 3584: 42 -> 21 us, the call 201 -> 178 us;
// 512 x 256, when it took this way: 21 -> 4 us, the call 35 -> 15 us with shorter slices and the reduction's mirror image.
constexpr int kFusedChannels = 16;
constexpr int kFusedThreads = 1024;
constexpr int kFusedTokens = 4096;

template <int NI>
__global__ __launch_bounds__(kFusedThreads) void hess_prepass_f16_kernel(const float* __restrict__ X, int n_tok, int d,
                                                                         long ldx, uint4* __restrict__ planes,
                                                                         long n_kg, int d_pad,
                                                                         float* __restrict__ inv) {
  __shared__ float red[kFusedThreads / 64][kFusedChannels];
  const int n_blk = d_pad / kFusedChannels;               // a multiple of 16
  const int blk = (blockIdx.x % kNumXCD) * (n_blk / kNumXCD) + blockIdx.x / kNumXCD;
  const int c = threadIdx.x & 15, tg = threadIdx.x >> 4;  // 64 token groups
  const int ch = blk * kFusedChannels + c;
  const bool live = ch < d;
  const float* p = X + (live ? ch : d - 1);
  float x[NI][8];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = 8 * (tg + 64 * i) + e;
      x[i][e] = p[(long)(t < n_tok ? t : n_tok - 1) * ldx];
    }
  __builtin_amdgcn_sched_barrier(0);                      // all loads before the first use
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(x[i][e]));      // (tokens past the end repeat the last one)
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  if ((threadIdx.x & 63) < 16) red[threadIdx.x >> 6][c] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kFusedThreads / 64; ++w) m = fmaxf(m, red[w][c]);
  const int e2 = live ? channel_exponent(m) : 0;
  const float s = ldexpf(1.0f, e2);
  if (threadIdx.x < 16) inv[ch] = ldexpf(1.0f, -e2);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const long kg = tg + 64 * i;
    if (kg >= n_kg) break;
    uint4 hv, lv;
    split_halves(x[i], s, live ? n_tok - 8 * (int)kg : 0, hv, lv);
    planes[kg * d_pad + ch] = hv;
    planes[(n_kg + kg) * d_pad + ch] = lv;
  }
}

// A whole small call in one launch: one TILE x TILE tile of H (16 or 32) to a work-group, WAVES wavefronts that share
// the tokens.  A lane holds its tokens of both operands in registers (NI of each), so X is read once per tile; every
// channel is brought to [2^13, 2^14) like above (the range of the two-halves path; a channel with an infinity gets the
// factor NaN, one with a NaN, which the maximum passes over, becomes NaN by its products), and the products go through the fp32 matrix cores in chains of at most kSmallChain tokens, whose
// sums are added in order, the wavefronts' in 64 bits.  The 32 x 32 blocks on the diagonal come whole, as from the tile kernels; `sym` writes
// the mirror image instead.  Bound by its latency, one round trip to memory and a reduction, while the tiles fit the
// chip once; beyond that by reading a tile's channels again for every tile, which the 256 x 256 tiles do not.
// Three launches (pre-pass, tile product, reduction) -> one, on activations not read before, and on the same ones again:
// 512 x 256 14.8 -> 6.8 us, 13.8 -> 5.4; 256 x 1024 19.9 -> 13.2, 19.5 -> 10.9; 2048 x 256 20.7 -> 17.0, 19.0 -> 11.4.
// Error of H against 64 bits (relative Frobenius, loud channels) 2e-8 .. 7e-8, 5e-8 .. 1.2e-7 before.
constexpr int kSmallChain = 32;

template <int TILE, int WAVES, int NI>
__global__ __launch_bounds__(64 * WAVES) void hess_small_kernel(const float* __restrict__ X, int n_tok, int d, long ldx,
                                                                float scale, float* __restrict__ H, int sym) {
  constexpr int kPer = 64 / TILE;                          // tokens an instruction takes
  constexpr int kAcc = TILE * TILE / 64;                   // results of a lane
  constexpr int kOut = TILE * TILE / (64 * WAVES) > 0 ? TILE * TILE / (64 * WAVES) : 1;      // ... of a thread at the end
  typedef float acc_t __attribute__((ext_vector_type(kAcc)));
  __shared__ float red[WAVES][TILE * TILE];
  __shared__ float top[WAVES][2][TILE];
  // 32 x 32 block (bi, bj) of the upper triangle, its tile (ti, tj)
  constexpr int kSub = 32 / TILE;
  const int blk = blockIdx.x / (kSub * kSub), sub = blockIdx.x % (kSub * kSub);
  int bj = (int)((sqrtf(8.0f * (float)blk + 1.0f) - 1.0f) * 0.5f);
  while (bj * (bj + 1) / 2 > blk) --bj;
  while ((bj + 1) * (bj + 2) / 2 <= blk) ++bj;
  const int bi = blk - bj * (bj + 1) / 2;
  const int ti = kSub * bi + sub / kSub, tj = kSub * bj + sub % kSub;
  const int r0 = TILE * ti, c0 = TILE * tj;
  if (r0 >= d || c0 >= d || (sym && ti > tj)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane % TILE, kq = lane / TILE;
  const bool diag = ti == tj;                              // both operands are the same channels
  const float* pa = X + (r0 + m < d ? r0 + m : d - 1);
  const float* pb = X + (c0 + m < d ? c0 + m : d - 1);
  const int t0 = wave * kPer * NI + kq;
  float a[NI], b[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int t = t0 + kPer * i;
    const long off = (long)(t < n_tok ? t : n_tok - 1) * ldx;
    a[i] = pa[off];
    b[i] = diag ? a[i] : pb[off];
  }
  float old[kOut];
  bool mine[kOut];
#pragma unroll
  for (int q = 0; q < kOut; ++q) {
    const int e = tid + 64 * WAVES * q, row = r0 + e / TILE, col = c0 + e % TILE;
    mine[q] = e < TILE * TILE && row < d && col < d && !(sym && row > col);
    old[q] = H[mine[q] ? (long)row * d + col : 0L];
  }
  __builtin_amdgcn_sched_barrier(0);                       // all loads before the first use
  // largest magnitude of a channel (tokens past the end repeat the last one)
  float ma = 0.f, mb = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) { ma = fmaxf(ma, fabsf(a[i])); mb = fmaxf(mb, fabsf(b[i])); }
#pragma unroll
  for (int x = TILE; x < 64; x *= 2) { ma = fmaxf(ma, __shfl_xor(ma, x, 64)); mb = fmaxf(mb, __shfl_xor(mb, x, 64)); }
  if (kq == 0) { top[wave][0][m] = ma; top[wave][1][m] = mb; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) { ma = fmaxf(ma, top[w][0][m]); mb = fmaxf(mb, top[w][1][m]); }
  const int ea = channel_exponent(ma), eb = channel_exponent(mb);
  const float sa = (ma < INFINITY) ? ldexpf(1.0f, ea) : NAN, sb = (mb < INFINITY) ? ldexpf(1.0f, eb) : NAN;
  constexpr int kLen = kSmallChain / kPer, kChains = NI > kLen ? NI / kLen : 1;
  acc_t part[kChains] = {};
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const bool in = t0 + kPer * i < n_tok;
    const float x = in ? a[i] * sa : 0.f, y = in ? b[i] * sb : 0.f;
    acc_t& acc = part[i % kChains];
    if constexpr (TILE == 16) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
    else acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
  }
  acc_t acc = part[0];
#pragma unroll
  for (int c = 1; c < kChains; ++c) acc += part[c];
  // D register i of lane l: row 4 (l / TILE) + i % 4 (+ 8 (i / 4) in the 32 x 32 form), column l % TILE
#pragma unroll
  for (int i = 0; i < kAcc; ++i) red[wave][(8 * (i / 4) + 4 * kq + i % 4) * TILE + m] = acc[i];
  __syncthreads();                                         // (the maxima are read out too)
  if (wave == 0 && kq == 0) { top[0][0][m] = ldexpf(1.0f, -ea); top[0][1][m] = ldexpf(1.0f, -eb); }
  double v[kOut];
#pragma unroll
  for (int q = 0; q < kOut; ++q) {
    const int e = tid + 64 * WAVES * q;
    v[q] = 0.0;
    if (e < TILE * TILE) {
#pragma unroll
      for (int w = 0; w < WAVES; ++w) v[q] += (double)red[w][e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kOut; ++q) {
    if (!mine[q]) continue;
    const int e = tid + 64 * WAVES * q, row = r0 + e / TILE, col = c0 + e % TILE;
    // in the activations' units again (powers of two), rounded once
    const float h = (float)((double)old[q] + (double)scale * (v[q] * (double)top[0][0][e / TILE] * (double)top[0][1][e % TILE]));
    H[(long)row * d + col] = h;
    if (sym && row < col) H[(long)col * d + row] = h;
  }
}

// The tile product of the fp16 path and its epilogue: every result is brought back to the
// activations' own units by the two channel factors (powers of two: exact).  DIRECT (p.direct): one slice
// per tile, added into H; else partial tiles.  (Kernels of their own, so that neither carries the other's code.)
template <bool DIRECT>
__global__ __launch_bounds__(SplitF16::kThreads, 1) void hess_syrk_f16x2_kernel(
    const uint4* __restrict__ planes, long n_kg, int d_pad, const float* __restrict__ inv, int n_tok,
    int d, float scale, float* __restrict__ H, float* __restrict__ partial, HessPlan p) {
  const int n_off_items = p.n_off * p.S_off;
  int item = 0, bi, bj, k_begin, k_end;
  if constexpr (DIRECT) {
    if (!direct_tile(blockIdx.x, p.nb, bi, bj)) return;
    k_begin = 0;
    k_end = n_tok;
  } else {
    item = xcd_item(blockIdx.x, n_off_items, p);
    if (item < n_off_items) {
      decode_off_tile(item % p.n_off, p.nb, bi, bj);
      k_begin = (item / p.n_off) * p.k_off;
      k_end = min(n_tok, k_begin + p.k_off);
    } else {
      const int j = item - n_off_items;
      bi = bj = j % p.n_diag;
      k_begin = (j / p.n_diag) * p.k_diag;
      k_end = min(n_tok, k_begin + p.k_diag);
    }
  }
  // two stages of 16 tokens per loop iteration; the planes are zero beyond n_tok
  const int n_stage = k_end > k_begin ? 2 * ((k_end - k_begin + 2 * SplitF16::kStageK - 1) / (2 * SplitF16::kStageK)) : 0;
  SplitF16::Acc acc;
  SplitF16::zero(acc);
  const int r0 = bi * SplitF16::kTile, c0 = bj * SplitF16::kTile;
  if (bi == bj) SplitF16::run<true>(planes, n_kg, d_pad, r0, c0, k_begin / 8, n_stage, acc);
  else SplitF16::run<false>(planes, n_kg, d_pad, r0, c0, k_begin / 8, n_stage, acc);
  // the LDS ring is free now: the channel factors of this tile's rows and columns
  extern __shared__ uint4 smem_f16[];
  float* sInv = reinterpret_cast<float*>(smem_f16);
  sInv[threadIdx.x] = inv[r0 + threadIdx.x];
  sInv[256 + threadIdx.x] = inv[c0 + threadIdx.x];
  __syncthreads();
  if constexpr (DIRECT) {
    // H += tile, in batches of 64 results per lane: all loads of a batch first, then its stores.  One load,
    // one wait, one store at a time -- what the compiler must make of a plain `+=`, since it cannot tell
    // the addresses apart -- left the matrix pipe idle for a quarter of a launch (4096 x 18944: 4.45 -> 3.54 ms).
    // A tile over the edge: blocks of 32 x 32 outside the matrix are passed over, entries outside it read
    // H[0] and are not stored.  (Without the former a call of one token on four channels took 20 us, 15.6
    // with a plain `+=`, and takes 8.5 now.)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto add = [&](auto in) {
      auto batch = [&](auto visit) {
        float old[64];
        visit([&](int row, int col, float, int n) { old[n] = H[in(row, col) ? (long)(r0 + row) * d + c0 + col : 0L]; });
        visit([&](int row, int col, float v, int n) {
          if (in(row, col)) H[(long)(r0 + row) * d + c0 + col] = old[n] + scale * (v * sInv[row] * sInv[256 + col]);
        });
      };
      if (bi == bj) {
        batch([&](auto f) { SplitF16::for_each_diag_in<0, 4>(acc, wave, in, f); });
        batch([&](auto f) { SplitF16::for_each_diag_in<4, 8>(acc, wave, in, f); });
        batch([&](auto f) { SplitF16::for_each_diag_in<8, 9>(acc, wave, in, f); });
      } else {
        batch([&](auto f) { SplitF16::for_each_in<0, 1>(acc, wave, in, f); });
        batch([&](auto f) { SplitF16::for_each_in<1, 2>(acc, wave, in, f); });
        batch([&](auto f) { SplitF16::for_each_in<2, 3>(acc, wave, in, f); });
        batch([&](auto f) { SplitF16::for_each_in<3, 4>(acc, wave, in, f); });
      }
    };
    if (r0 + SplitF16::kTile <= d && c0 + SplitF16::kTile <= d) add([](int, int) { return true; });
    else add([&](int row, int col) { return r0 + row < d && c0 + col < d; });
  } else {
    float* out = partial + (long)item * kTileFloats;
    auto emit = [&](int row, int col, float v) {
      out[row * SplitF16::kTile + col] = v * sInv[row] * sInv[256 + col];
    };
    if (bi == bj) SplitF16::for_each_diag(acc, emit);
    else SplitF16::for_each(acc, emit);
  }
}

// H[tile] += scale * sum_s partial[s][tile], slices added in index order.  64 work-groups per tile;
// tiles 0 .. n_off-1 are off-diagonal, the rest diagonal.  SYM (the last launch of a
// call that symmetrizes): the block's transpose goes to the lower triangle from the same registers, which
// spares small layers a launch (4 of 22 us at 512 x 256, when it took this way) and large ones a pass over the upper triangle.
// FLIGHT: slices in flight per wavefront.  A layer of few tiles has many slices and too few wavefronts to cover
// a load and a wait per slice (8192 tokens, 1 tile of 57 slices: the call 53.2 -> 47.4 us with eight in flight; 3 tiles
// 64.3 -> 58.2, 11 slices 23.5 -> 22.8); from 10 tiles on the wavefronts cover for one another (21 tiles of 10
// slices: 57.4 us, with eight 58.7).
constexpr int kReduceFewTiles = 6;
template <bool SYM, int FLIGHT>
__global__ __launch_bounds__(256) void hess_reduce_kernel(const float* __restrict__ partial,
                                                          HessPlan p, int d, float scale,
                                                          float* __restrict__ H) {
  __shared__ float sT[SYM ? 32 : 1][33];
  const int tile = blockIdx.x >> 6;
  // SYM: one 32 x 32 block; otherwise four whole rows of the tile (1 KB runs: 172 us against 198 for 3584 channels)
  const int e = ((blockIdx.x & 63) * 256 + threadIdx.x) * 4;
  const int row = SYM ? 32 * ((blockIdx.x & 63) >> 3) + (threadIdx.x >> 3) : e / HessGemm::kTileN;
  const int col = SYM ? 32 * (blockIdx.x & 7) + (threadIdx.x & 7) * 4 : e % HessGemm::kTileN;
  const int rb = row / 32, cb = col / 32;
  int bi, bj, S;
  long first, stride;
  if (tile < p.n_off) {
    decode_off_tile(tile, p.nb, bi, bj);
    S = p.S_off;
    first = tile;
    stride = p.n_off;
  } else {
    bi = bj = tile - p.n_off;
    S = p.S_diag;
    first = (long)p.n_off * p.S_off + bi;
    stride = p.n_diag;
    // blocks of 32 x 32 below the diagonal of a diagonal tile are never computed
    if (cb < rb) return;
  }
  const int r = bi * HessGemm::kTileM + row, c = bj * HessGemm::kTileN + col;
  const bool in = r < d && c < d;                     // d % 4 == 0: the four columns are in or out together
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  if (in) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* src = partial + first * kTileFloats + row * HessGemm::kTileN + col;
    // slices in index order, FLIGHT of them on their way at a time
    int sp = 0;
    if constexpr (FLIGHT > 1) {
      auto add = [&](auto count) {
        constexpr int kN = decltype(count)::value;
        float4 v[kN];
#pragma unroll
        for (int u = 0; u < kN; ++u) v[u] = *reinterpret_cast<const float4*>(src + (sp + u) * stride * kTileFloats);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kN; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
        sp += kN;
      };
      while (sp + FLIGHT <= S) add(std::integral_constant<int, FLIGHT>{});
      while (sp + 2 <= S) add(std::integral_constant<int, 2>{});
    }
    for (; sp < S; ++sp) {
      const float4 v = *reinterpret_cast<const float4*>(src + sp * stride * kTileFloats);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    float4* h = reinterpret_cast<float4*>(H + (long)r * d + c);
    o = *h;
    o.x += scale * s.x; o.y += scale * s.y; o.z += scale * s.z; o.w += scale * s.w;
    // a block on the diagonal: below it the mirror image is what counts
    const bool mirror_here = SYM && bi == bj && rb == cb;
    if (!mirror_here) {
      *h = o;
    } else {
      const float e[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (c + q >= r) H[(long)r * d + c + q] = e[q];
    }
  }
  if constexpr (SYM) {
    const int y = threadIdx.x >> 3, x = (threadIdx.x & 7) * 4;
    sT[y][x] = o.x; sT[y][x + 1] = o.y; sT[y][x + 2] = o.z; sT[y][x + 3] = o.w;
    __syncthreads();
    const int tr = bj * HessGemm::kTileN + 32 * cb + y, tc = bi * HessGemm::kTileM + 32 * rb + x;   // row, columns of H
    if (tr < d) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (tc + q < tr) H[(long)tr * d + tc + q] = sT[x + q][y];
    }
  }
}

// lower triangle <- transpose of the upper triangle, 32 x 32 tiles through LDS
__global__ __launch_bounds__(256) void symmetrize_kernel(float* __restrict__ H, int d) {
  __shared__ float t[32][33];
  const int bi = blockIdx.y, bj = blockIdx.x;      // tile (bi, bj) with bj >= bi is the source
  if (bj < bi) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int y = ty; y < 32; y += 8) {
    const int r = bi * 32 + y, c = bj * 32 + tx;
    t[y][tx] = (r < d && c < d) ? H[(long)r * d + c] : 0.f;
  }
  __syncthreads();
  for (int y = ty; y < 32; y += 8) {
    const int r = bj * 32 + y, c = bi * 32 + tx;     // destination (r, c) = source (c, r)
    if (r < d && c < d && r > c) H[(long)r * d + c] = t[tx][y];
  }
}

}  // namespace bpdq

using namespace bpdq;

// Tokens of the next launch: the chain length is bounded (kChainTokens).  A launch that adds
// straight into H (no slices) takes one chain's worth of tokens, a sliced one as many as its
// slices can cover; successive launches on one stream accumulate in order.
static int hessian_launch_tokens(int kind, bool fine, int n_left, int d_in) {
  const int chain = kChainTokens[kind];
  const long cover = (long)chain * kMaxSlices;
  int n = n_left > cover ? (int)cover : n_left;
  if (n > chain && plan_hessian(n, d_in, kind, fine).direct) n = chain;
  return n;
}

// Workspace of one launch of n_part tokens: split-K partial tiles, then (fp16 path) the split
// planes, the partial channel maxima and the two channel factors.
struct HessWs {
  size_t partial_off, planes_off, pmax_off, mul_off, inv_off, total;
  long n_kg;
  int d_pad, n_split;
};

static HessWs hessian_ws_layout(int kind, bool fine, int n_part, int d_in) {
  HessWs L{};
  size_t off = 0;
  L.partial_off = off;
  off += bpdq_align_up(plan_hessian(n_part, d_in, kind, fine).ws_bytes(), 256);
  if (kind == kKindF16x2) {
    L.d_pad = (int)bpdq_align_up((size_t)d_in, SplitF16::kTile);
    L.n_kg = (long)bpdq_align_up((size_t)n_part, 2 * SplitF16::kStageK) / 8;
    L.n_split = bpdq_ceil_div(n_part, kColmaxRows);
    L.planes_off = off; off += bpdq_align_up((size_t)2 * L.n_kg * L.d_pad * sizeof(uint4), 256);
    L.pmax_off = off;   off += bpdq_align_up((size_t)L.n_split * L.d_pad * sizeof(float), 256);
    L.mul_off = off;    off += bpdq_align_up((size_t)L.d_pad * sizeof(float), 256);
    L.inv_off = off;    off += bpdq_align_up((size_t)L.d_pad * sizeof(float), 256);
  }
  L.total = off;
  return L;
}

// the first launch of a call is its largest
static size_t hessian_ws_bytes(int kind, bool fine, int n_tok, int d_in) {
  return hessian_ws_layout(kind, fine, hessian_launch_tokens(kind, fine, n_tok, d_in), d_in).total;
}

// Calls that one launch serves best (hess_small_kernel), and its form.  Measured on activations that no call has read
// before (us, three launches / one; on the same ones again the one launch gains up to a third):
//   64 tokens: 512 channels 18.6 / 4.3, 1024 20.2 / 7.1, 2048 28.7 / 13.3, 3072 26.6 / 23.3.
//   65 tokens: 384 channels 41.7 / 6.4, 1024 21.7 / 13.0, 1536 23.8 / 21.7, 1728 47.4 / 24.4, beyond which the
//     256 x 256 tiles are quicker if the channels fill them or barely start another (1792 25.2 / 29.1, 1820 27.7 / 30.6,
//     2048 30.3 / 34.2; at 160 tokens 33.8 / 34.5, at 192 35.7 / 34.7) and slower if not (1856 31.3 / 29.7, 2044 48.9 / 36.2).
//   257 tokens: 512 channels 16.4 / 11.1, 704 17.9 / 15.4, 768 18.1 / 27.6: up to 704 every 32 x 32 tile has a compute
//     unit to itself (253 tiles).  512 tokens: 704 19.7 / 16.0, 768 20.3 / 28.6, 1024 24.2 / 36.0.
//   513 tokens: 512 channels 18.7 / 18.3 (1024 tokens: 21.1 / 18.6).
//   1025 tokens: 320 channels 21.1 / 16.9 (220 tiles), 352 21.1 / 26.0, 384 21.3 / 31.1; 2048: 320 25.3 / 17.4, 384 26.0 / 32.1.
// Small layers take 16 x 16 tiles, which occupy more compute units (256 tokens, 256 channels: 4.5 us, 6.4 with 32 x 32),
// and more wavefronts the more tokens there are.
enum SmallForm { kNotSmall, k16x4, k16x8, k16x16, k32x4, k32x8 };
static SmallForm hessian_small_form(int n_tok, int d_in) {
  if (n_tok <= 64) return d_in <= 512 ? k16x4 : d_in <= 3072 ? k32x4 : kNotSmall;
  if (n_tok <= 256) {
    if (d_in <= 384) return k16x8;
    return d_in <= 1728 || (d_in <= 2048 && (n_tok >= 192 || d_in % 256 >= 64)) ? k32x8 : kNotSmall;
  }
  if (n_tok <= 512) return d_in <= 256 ? k16x16 : d_in <= 512 ? k16x8 : d_in <= 704 ? k32x8 : kNotSmall;
  if (n_tok <= 1024) return d_in <= 512 ? k16x16 : kNotSmall;
  if (n_tok <= 2048) return d_in <= 320 ? k16x16 : kNotSmall;
  return kNotSmall;
}

static void launch_hessian_small(SmallForm form, const float* X, int n_tok, int d_in, int ldx, float scale, float* H,
                                 int symmetrize, hipStream_t stream) {
  const int nb = bpdq_ceil_div(d_in, 32), blocks = nb * (nb + 1) / 2;
  auto go = [&](auto kern, int tiles, int waves) {
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * waves), 0, stream, X, n_tok, d_in, (long)ldx, scale, H, symmetrize);
  };
  // NI: the tokens (64, 256, 512, 1024, 2048) over the lanes that share them
  switch (form) {
    case k16x4: return go(hess_small_kernel<16, 4, 4>, 4 * blocks, 4);
    case k16x8: return n_tok <= 256 ? go(hess_small_kernel<16, 8, 8>, 4 * blocks, 8) : go(hess_small_kernel<16, 8, 16>, 4 * blocks, 8);
    case k16x16:
      if (n_tok <= 512) return go(hess_small_kernel<16, 16, 8>, 4 * blocks, 16);
      return n_tok <= 1024 ? go(hess_small_kernel<16, 16, 16>, 4 * blocks, 16) : go(hess_small_kernel<16, 16, 32>, 4 * blocks, 16);
    case k32x4: return go(hess_small_kernel<32, 4, 8>, blocks, 4);
    default: return n_tok <= 256 ? go(hess_small_kernel<32, 8, 16>, blocks, 8) : go(hess_small_kernel<32, 8, 32>, blocks, 8);
  }
}

static int hessian_accumulate(int kind, const float* Xc, int n_tok, int d_in, int ldx, float scale,
                              float* H, int symmetrize, void* ws, size_t ws_bytes, void* stream_,
                              void* ev_begin = nullptr, void* ev_end = nullptr) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (kind < 0 || kind >= kNumKinds) return -11;
  if (n_tok < 0) return -2;
  if (d_in <= 0 || d_in % 4) return -3;
  if (ldx < d_in || ldx % 4) return -4;
  if (n_tok > 0 && (!Xc || (reinterpret_cast<uintptr_t>(Xc) & 15))) return -1;
  if (!H || (reinterpret_cast<uintptr_t>(H) & 15)) return -6;
  // A workspace that holds the coarse plan but not the fine one (sized for another call, say the larger
  // chunks before a short last one) gets the coarse plan.
  bool fine = kind == kKindF16x2;
  size_t need = n_tok > 0 ? hessian_ws_bytes(kind, fine, n_tok, d_in) : 0;
  if (fine && ws_bytes < need) {
    fine = false;
    need = hessian_ws_bytes(kind, fine, n_tok, d_in);
  }
  if (need > 0 && (!ws || (reinterpret_cast<uintptr_t>(ws) & 255))) return -8;
  if (ws_bytes < need) return -9;
  const SmallForm small = kind == kKindF16x2 && n_tok > 0 ? hessian_small_form(n_tok, d_in) : kNotSmall;
  if (small != kNotSmall) {
    if (ev_begin) BPDQ_HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(ev_begin), stream));
    launch_hessian_small(small, Xc, n_tok, d_in, ldx, scale, H, symmetrize, stream);
    BPDQ_LAUNCH_CHECK();
    if (ev_end) BPDQ_HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(ev_end), stream));
    return 0;
  }
  char* base = static_cast<char*>(ws);
  for (int done = 0; done < n_tok;) {
    const int n_part = hessian_launch_tokens(kind, fine, n_tok - done, d_in);
    const HessPlan p = plan_hessian(n_part, d_in, kind, fine);
    const HessWs L = hessian_ws_layout(kind, fine, n_part, d_in);
    float* partial = reinterpret_cast<float*>(base + L.partial_off);
    const float* Xpart = Xc + (long)done * ldx;
    const bool first = (done == 0);
    done += n_part;
    // (the pre-pass of the fp16 path precedes the first event; later launches' pre-passes fall
    // between the two events)
    auto mark_begin = [&]() -> int {
      if (first && ev_begin) BPDQ_HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(ev_begin), stream));
      return 0;
    };
    if (kind == kKindF32) {
      if (mark_begin()) return BPDQ_ERR_LAUNCH;
      BPDQ_HIP_TRY(bpdq_lds_limit<&hess_syrk_f32_kernel>(HessGemm::kLdsBytes));
      hipLaunchKernelGGL(hess_syrk_f32_kernel, dim3(p.items()), dim3(HessGemm::kThreads),
                         HessGemm::kLdsBytes, stream, Xpart, n_part, d_in, (long)ldx, scale, H,
                         partial, p);
    } else if (kind == kKindBf16x3) {
      if (mark_begin()) return BPDQ_ERR_LAUNCH;
      BPDQ_HIP_TRY(bpdq_lds_limit<&hess_syrk_bf16x3_kernel>(SplitSyrk::kLdsBytes));
      hipLaunchKernelGGL(hess_syrk_bf16x3_kernel, dim3(p.items()), dim3(SplitSyrk::kThreads),
                         SplitSyrk::kLdsBytes, stream, Xpart, n_part, d_in, (long)ldx, scale, H,
                         partial, p);
    } else {
      BPDQ_HIP_TRY(bpdq_lds_limit<&hess_syrk_f16x2_kernel<true>>(SplitF16::kLdsBytes));
      BPDQ_HIP_TRY(bpdq_lds_limit<&hess_syrk_f16x2_kernel<false>>(SplitF16::kLdsBytes));
      uint4* planes = reinterpret_cast<uint4*>(base + L.planes_off);
      float* pmax = reinterpret_cast<float*>(base + L.pmax_off);
      float* mul = reinterpret_cast<float*>(base + L.mul_off);
      float* inv = reinterpret_cast<float*>(base + L.inv_off);
      if (n_part <= kFusedTokens) {
        auto prepass = [&](auto kern) {
          hipLaunchKernelGGL(kern, dim3(L.d_pad / kFusedChannels), dim3(kFusedThreads), 0, stream, Xpart, n_part, d_in,
                             (long)ldx, planes, L.n_kg, L.d_pad, inv);
        };
        if (L.n_kg <= 64) prepass(hess_prepass_f16_kernel<1>);
        else if (L.n_kg <= 128) prepass(hess_prepass_f16_kernel<2>);
        else if (L.n_kg <= 256) prepass(hess_prepass_f16_kernel<4>);
        else prepass(hess_prepass_f16_kernel<8>);
        BPDQ_LAUNCH_CHECK();
      } else {
        const int cb = L.d_pad / SplitF16::kTile;
        const int kgs = bpdq_ceil_div((int)L.n_kg, kSplitKgPerWG);
        auto scales = [&](auto colmax, auto scale_of) -> int {
          hipLaunchKernelGGL(colmax, dim3(cb, L.n_split), dim3(256), 0, stream, Xpart, n_part, d_in, (long)ldx, pmax, L.d_pad);
          BPDQ_LAUNCH_CHECK();
          hipLaunchKernelGGL(scale_of, dim3(L.d_pad / 16), dim3(256), 0, stream, pmax, L.n_split, L.d_pad, mul, inv);
          BPDQ_LAUNCH_CHECK();
          return 0;
        };
        auto split = [&](auto kern, int grid_y) -> int {
          hipLaunchKernelGGL(kern, dim3(cb, grid_y), dim3(256), 0, stream, Xpart, n_part, d_in, (long)ldx, mul, inv,
                             reinterpret_cast<unsigned*>(pmax), planes, L.n_kg, L.d_pad);
          BPDQ_LAUNCH_CHECK();
          return 0;
        };
        if ((long)n_part * d_in < kSampleValues) {
          if (scales(hess_colmax_kernel<false>, hess_scale_kernel<false>)) return BPDQ_ERR_LAUNCH;
          if (split(hess_split_f16_kernel<kAllTokens>, kgs)) return BPDQ_ERR_LAUNCH;
        } else {
          if (scales(hess_colmax_kernel<true>, hess_scale_kernel<true>)) return BPDQ_ERR_LAUNCH;
          if (split(hess_split_f16_kernel<kSampled>, kgs)) return BPDQ_ERR_LAUNCH;
          const int rounds = cb < 2048 ? kBeyondWGs / cb + 1 : 4;          // a small grid where it ends at once
          if (split(hess_split_f16_kernel<kBeyond>, kgs < rounds ? kgs : rounds)) return BPDQ_ERR_LAUNCH;
        }
      }
      if (mark_begin()) return BPDQ_ERR_LAUNCH;
      auto tiles = [&](auto kern, int grid) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(SplitF16::kThreads), SplitF16::kLdsBytes, stream, planes, L.n_kg,
                           L.d_pad, inv, n_part, d_in, scale, H, partial, p);
      };
      if (p.direct) tiles(hess_syrk_f16x2_kernel<true>, direct_grid(p.nb));
      else tiles(hess_syrk_f16x2_kernel<false>, p.items());
    }
    BPDQ_LAUNCH_CHECK();
    if (done >= n_tok && ev_end) BPDQ_HIP_TRY(hipEventRecord(static_cast<hipEvent_t>(ev_end), stream));
    if (!p.direct) {
      const bool sym = symmetrize && done >= n_tok;
      auto reduce = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((p.n_off + p.n_diag) * 64), dim3(256), 0, stream, partial, p, d_in, scale, H);
      };
      if (p.n_off + p.n_diag <= kReduceFewTiles) sym ? reduce(hess_reduce_kernel<true, 8>) : reduce(hess_reduce_kernel<false, 8>);
      else sym ? reduce(hess_reduce_kernel<true, 1>) : reduce(hess_reduce_kernel<false, 1>);
      BPDQ_LAUNCH_CHECK();
      if (sym) return 0;
    }
  }
  if (symmetrize) {      // nothing accumulated, or the last launch added its tiles straight into H
    const int nt = bpdq_ceil_div(d_in, 32);
    hipLaunchKernelGGL(symmetrize_kernel, dim3(nt, nt), dim3(256), 0, stream, H, d_in);
    BPDQ_LAUNCH_CHECK();
  }
  return 0;
}

extern "C" size_t bpdq_hessian_workspace_bytes(int n_tok, int d_in) {
  if (n_tok <= 0 || d_in <= 0) return 0;
  // one workspace serves any of the kernels
  size_t need = 0;
  for (int kind = 0; kind < kNumKinds; ++kind) {
    const size_t b = hessian_ws_bytes(kind, true, n_tok, d_in);
    need = b > need ? b : need;
  }
  return need;
}

extern "C" int bpdq_hessian_accumulate_f32(const float* Xc, int n_tok, int d_in, int ldx, float scale,
                                           float* H, int symmetrize, void* ws, size_t ws_bytes,
                                           void* stream) {
  return hessian_accumulate(kKindF32, Xc, n_tok, d_in, ldx, scale, H, symmetrize, ws, ws_bytes, stream);
}

extern "C" int bpdq_hessian_accumulate_bf16x3(const float* Xc, int n_tok, int d_in, int ldx, float scale,
                                              float* H, int symmetrize, void* ws, size_t ws_bytes,
                                              void* stream) {
  return hessian_accumulate(kKindBf16x3, Xc, n_tok, d_in, ldx, scale, H, symmetrize, ws, ws_bytes, stream);
}

extern "C" int bpdq_hessian_accumulate_timed(int kernel, const float* Xc, int n_tok, int d_in, int ldx,
                                             float scale, float* H, int symmetrize, void* ws,
                                             size_t ws_bytes, void* stream, void* ev_begin, void* ev_end) {
  const int kind = kernel == BPDQ_HESSIAN_F16X2 ? kKindF16x2
                   : kernel == BPDQ_HESSIAN_BF16X3 ? kKindBf16x3
                   : kernel == BPDQ_HESSIAN_F32 ? kKindF32 : -1;
  if (kind < 0) return -1;
  const int rc = hessian_accumulate(kind, Xc, n_tok, d_in, ldx, scale, H, symmetrize, ws, ws_bytes, stream,
                                    ev_begin, ev_end);
  return rc < 0 && rc > -11 ? rc - 1 : rc;      // the arguments are shifted by one
}

// the default entry: two fp16 halves per scaled value
extern "C" int bpdq_hessian_accumulate(const float* Xc, int n_tok, int d_in, int ldx, float scale,
                                       float* H, int symmetrize, void* ws, size_t ws_bytes,
                                       void* stream) {
  return hessian_accumulate(kKindF16x2, Xc, n_tok, d_in, ldx, scale, H, symmetrize, ws, ws_bytes, stream);
}
