// Serving side: y = What x for one token from the stored bit-plane format (paper Eq. 1; Sec. 5
// discusses the inference kernel).  Regrouped per (row, group G):
//   y_r = sum_G ( C_0[r,G] S(G) + sum_i C_i[r,G] sum_{c in G} B_i[r,c] x_c ),   S(G) = sum_{c in G} x_c.
// A weight costs one masked add per plane and no multiply; a row reads bits/8 bytes per weight.
//
// A look-up table replaces the per-bit work: for every segment of 4 columns the 16 partial sums
// of its x values; a plane word then costs 8 look-ups instead of 32 masked adds.  The table of a
// chunk of up to 8192 columns (128 KB of LDS) is built once per work-group and chunk -- 15 adds per
// segment -- and used by all its rows: one wavefront owns ROWS rows at a time, 16 wavefronts per
// work-group, one work-group per CU.  fp32 accumulation in a fixed order.
//
// Layout.  A lane of a wavefront holds W words of a chunk of 64 W: consecutive ones, W l ... (one 16-byte load per
// plane and row at W = 4, and words that share a group's coefficients, or find theirs side by side), or, where
// that leaves lanes idle or does not fit the row, words l, l + 64 ... (pick_gemv).  The table is
// T[q][j][nibble][lane] (q = nibble position in a word, j = word of the lane): whatever the nibbles are, the lanes of
// a wavefront fall into consecutive banks -- the minimum of two cycles.  The nibble is a whole byte of the LDS
// address, so after splitting a word into the bytes of its even and odd nibbles (3 instructions) one v_perm_b32
// per look-up forms the address from the nibble and the lane's base; with the add that is 2.4 vector instructions
// per look-up.
//
// What bounds it: these instructions and the LDS reads (12 and 8 us on the 8192 x 29568 layer, by their counts,
// whose 83 MB of planes and half-precision coefficients need 16.3 us at 5.1 TB/s).  The plane words and coefficients of the next
// chunk or row pass, and the x values of the next chunk, are requested before the current one is worked on;
// without that every chunk waited for memory twice.
// Measured, back to back in a graph (one word per lane and load, no prefetch -> this): 8192 x 29568 k = 2
// g = 64 48.6 -> 27.1 us (3.1 TB/s of stored bytes), 8192 x 8192 k = 2 11.3 -> 7.7, 3584 x 18944 k = 3 40.6 -> 15.2,
// 3584 x 3584 k = 2 7.0 -> 4.2, 5000 x 8224 k = 4 g = 32 17.7 -> 16.5, 152064 x 1024 k = 1 24.9 -> 24.4.
#include "common.h"

namespace bpdq {

constexpr int kGemvThreads = 1024;
constexpr int kGemvWaves = kGemvThreads / 64;
constexpr int kGemvRowsSplit = 2 * 8 * 32 * kGemvWaves / 2;   // 4096: up to here one row per wavefront fills the CUs

template <int WPL>
constexpr size_t gemv_lds_bytes() { return (size_t)(8 * WPL * 16 * 64 + WPL * 64) * sizeof(float); }

// Plane words and coefficients of one (chunk, row pass) for this lane, as they come from memory: nothing is
// computed from them before their turn, or the request of the next item would wait for its data.
// W words per lane, NG groups among them.  PACKED: a row's NG halves come as one load.
template <int K, int W, int NG, int ROWS, bool PACKED>
struct GemvItem {
  uint32_t w[ROWS][K][W];
  uint32_t cp[ROWS][K + 1][PACKED ? NG / 2 : 1];
  _Float16 c[ROWS][K + 1][PACKED ? 1 : NG];
  __device__ __forceinline__ float coef(int q, int i, int g) const {
    if constexpr (PACKED) {
      const uint32_t h = cp[q][i][g >> 1];
      return (float)__builtin_bit_cast(_Float16, (unsigned short)((g & 1) ? h >> 16 : h));
    } else {
      return (float)c[q][i][g];
    }
  }
};

// Where a lane's words and their coefficients lie in a row, as byte offsets: one pair per word if STRIDED (word j of
// the lane is word 64 j + lane of the chunk), else one (its words are W lane ...).  The row is the wavefront's, so an
// item's addresses are a scalar and these.  Found once per chunk, but anew for every item if STRIDED: the pairs of four
// words would not fit the registers beside two items.
template <int W, bool STRIDED>
struct GemvPlace {
  static constexpr int kN = STRIDED ? W : 1;
  unsigned word[kN], coef[kN];
  __device__ __forceinline__ GemvPlace(int w0, int n_word, int wpg, int lane) {
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const int wl = STRIDED ? 64 * j + lane : W * lane;
      // past the end: the chunk's first words (the table is zero there, or the lane's sum is dropped)
      const unsigned wf = w0 + (wl < n_word ? wl : 0);
      word[j] = 4u * wf;
      coef[j] = 2u * (wf / (unsigned)wpg);
    }
  }
};

template <typename T>
__device__ __forceinline__ T gemv_load(const void* base, unsigned byte) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + byte);
}

template <int K, int W, int NG, int ROWS, bool STRIDED>
__device__ __forceinline__ void gemv_fetch(const uint32_t* __restrict__ planes, const _Float16* __restrict__ coefs,
                                           int d_out, int nw, int n_grp, int wpg, int r0, int w0, int n_word, int lane,
                                           const GemvPlace<W, STRIDED>& found,
                                           GemvItem<K, W, NG, ROWS, !STRIDED && (NG > 1)>& it) {
  typedef uint32_t words __attribute__((ext_vector_type(W == 1 ? 2 : W)));
  typedef uint32_t halves __attribute__((ext_vector_type(2)));
  const GemvPlace<W, STRIDED> at = STRIDED ? GemvPlace<W, STRIDED>(w0, n_word, wpg, lane) : found;
#pragma unroll
  for (int j = 0; j < GemvPlace<W, STRIDED>::kN; ++j) {
    if (j > 0 && 64 * j >= n_word) break;          // uniform
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
      const long r = r0 + q < d_out ? r0 + q : d_out - 1;
      const uint32_t* p = planes + r * nw;
      const _Float16* c = coefs + r * n_grp;
#pragma unroll
      for (int i = 0; i < K; ++i, p += (long)d_out * nw) {
        if constexpr (STRIDED || W == 1) {
          it.w[q][i][j] = gemv_load<uint32_t>(p, at.word[j]);
        } else {
          const words v = gemv_load<words>(p, at.word[0]);
#pragma unroll
          for (int e = 0; e < W; ++e) it.w[q][i][e] = v[e];
        }
      }
#pragma unroll
      for (int i = 0; i <= K; ++i, c += (long)d_out * n_grp) {
        if constexpr (STRIDED || NG == 1) {
          it.c[q][i][j] = gemv_load<_Float16>(c, at.coef[j]);
        } else if constexpr (NG == 2) {
          it.cp[q][i][0] = gemv_load<uint32_t>(c, at.coef[0]);
        } else {
          const halves v = gemv_load<halves>(c, at.coef[0]);
          it.cp[q][i][0] = v[0];
          it.cp[q][i][1] = v[1];
        }
      }
    }
  }
}

// K planes; W words per lane; NG groups among a lane's words (W / NG consecutive words share one);
// ROWS rows per wavefront and pass; STRIDED: see GemvPlace (then NG = W).
template <int K, int W, int NG, int ROWS, bool STRIDED>
__global__ __launch_bounds__(kGemvThreads) void gemv_planes_kernel(const uint32_t* __restrict__ planes,
                                                                   const _Float16* __restrict__ coefs,
                                                                   int d_out, int d_in, int group, int chunk_words,
                                                                   int passes,
                                                                   const float* __restrict__ x,
                                                                   float* __restrict__ y) {
  extern __shared__ float lds[];
  float* T = lds;                                        // [8][W][16][64]
  float* Sw = lds + 8 * W * 16 * 64;                     // [W][64]: sum of x over each word
  constexpr int kSegs = 8 * W;                           // table segments of a lane
  constexpr int kSegPerThread = (kSegs + kGemvWaves - 1) / kGemvWaves;
  const int nw = d_in / 32, n_grp = d_in / group, wpg = group / 32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row_step = gridDim.x * kGemvWaves * ROWS;
  const int row_first = (blockIdx.x * kGemvWaves + wave) * ROWS;

  auto fetch_x = [&](int w0, int n_word, float4 (&xv)[kSegPerThread]) {
#pragma unroll
    for (int s = 0; s < kSegPerThread; ++s) {
      const int id = wave + kGemvWaves * s;              // segment (q, j) = (id / W, id % W)
      const int wl = STRIDED ? 64 * (id % W) + lane : W * lane + id % W;
      const bool in = id < kSegs && wl < n_word;
      const float4 v = *reinterpret_cast<const float4*>(x + (in ? 32L * (w0 + wl) + 4 * (id / W) : 0L));
      xv[s] = in ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  typedef GemvItem<K, W, NG, ROWS, !STRIDED && (NG > 1)> Item;
  Item cur, nxt;
  float4 xv[kSegPerThread];
  const int n0 = nw < chunk_words ? nw : chunk_words;
  fetch_x(0, n0, xv);
  GemvPlace<W, STRIDED> at(0, n0, wpg, lane);
  gemv_fetch<K, W, NG, ROWS, STRIDED>(planes, coefs, d_out, nw, n_grp, wpg, row_first, 0, n0, lane, at, cur);
  float acc[ROWS];
#pragma unroll
  for (int q = 0; q < ROWS; ++q) acc[q] = 0.f;
  for (int w0 = 0; w0 < nw; w0 += chunk_words) {
    const int n_word = nw - w0 < chunk_words ? nw - w0 : chunk_words;
    const bool last_chunk = w0 + chunk_words >= nw;
    if (w0 > 0) __syncthreads();                         // the previous chunk's table is no longer read
#pragma unroll
    for (int s = 0; s < kSegPerThread; ++s) {
      const int id = wave + kGemvWaves * s;
      if (id < kSegs) {
        const float4 v = xv[s];
        float* t = T + (id * 16) * 64 + lane;
        const float s01 = v.x + v.y, s23 = v.z + v.w;
        const float e[16] = {0.f,  v.x,       v.y,       s01,       v.z, v.x + v.z, v.y + v.z, s01 + v.z,
                             v.w,  v.x + v.w, v.y + v.w, s01 + v.w, s23, v.x + s23, v.y + s23, s01 + s23};
#pragma unroll
        for (int n = 0; n < 16; ++n) t[n * 64] = e[n];
      }
    }
    __syncthreads();
    if (tid < 64 * W) {
      const int j = tid >> 6;
      float sw = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) sw += T[((q * W + j) * 16 + 15) * 64 + lane];
      Sw[tid] = sw;
    }
    __syncthreads();
    // the first item is here: or the look-ups below, reached with and without a request ahead of them, would wait for
    // everything in flight (vmcnt 0; the other counters at their maxima)
    __builtin_amdgcn_s_waitcnt(0x0f70);
    if (!last_chunk) {
      const int w1 = w0 + chunk_words;
      fetch_x(w1, nw - w1 < chunk_words ? nw - w1 : chunk_words, xv);
    }
    for (int p = 0; p < passes; ++p) {
      const int r0 = row_first + p * row_step;
      if (r0 >= d_out) break;                            // uniform over the wavefront
      // the next item: the next pass of this chunk, else the first pass of the next chunk
      const bool same = p + 1 < passes && r0 + row_step < d_out;
      int w_next = w0, n_next = n_word;
      if (!same && !last_chunk) {
        w_next = w0 + chunk_words;
        n_next = nw - w_next < chunk_words ? nw - w_next : chunk_words;
        at = GemvPlace<W, STRIDED>(w_next, n_next, wpg, lane);
      }
      if (same || !last_chunk)
        gemv_fetch<K, W, NG, ROWS, STRIDED>(planes, coefs, d_out, nw, n_grp, wpg, same ? r0 + row_step : row_first,
                                            w_next, n_next, lane, at, nxt);
      float sum[ROWS];
#pragma unroll
      for (int q = 0; q < ROWS; ++q) sum[q] = 0.f;
      // LDS byte addresses (the table starts at LDS address 0: the kernel has no other LDS)
      const unsigned base0 = 4u * lane, base1 = 4u * lane + 65536u;
      typedef const __attribute__((address_space(3))) float lds_float;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (STRIDED && g > 0 && 64 * g >= n_word) break; // uniform
        float s = 0.f;
#pragma unroll
        for (int j = g * (W / NG); j < (g + 1) * (W / NG); ++j) s += Sw[j * 64 + lane];
        const bool on = !STRIDED || 64 * g + lane < n_word;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          float t = fmaf(cur.coef(q, 0, g), s, sum[q]);
#pragma unroll
          for (int i = 0; i < K; ++i) {
            float m = 0.f;                               // one chain of eight adds per word
#pragma unroll
            for (int j = g * (W / NG); j < (g + 1) * (W / NG); ++j) {
              float mj = 0.f;
              const uint32_t w = cur.w[q][i][j];
              const uint32_t ev = w & 0x0f0f0f0fu, od = (w >> 4) & 0x0f0f0f0fu;
#pragma unroll
              for (int n = 0; n < 8; ++n) {
                // address bytes: 0 = lane, 1 = the nibble, 2 and 3 = upper half of the table or not
                const unsigned off = (unsigned)(n * W + j) * 4096u;
                const unsigned a = __builtin_amdgcn_perm((n & 1) ? od : ev, off >= 65536u ? base1 : base0,
                                                         0x03020000u | (unsigned)((4 + (n >> 1)) << 8));
                mj += *reinterpret_cast<lds_float*>(a + (off & 65535u));
              }
              m += mj;
            }
            t = fmaf(cur.coef(q, i + 1, g), m, t);
          }
          // a word past the end adds nothing, whatever its coefficient (zero times an infinite one is not zero)
          sum[q] = on ? t : sum[q];
        }
      }
      if (!STRIDED && W * lane >= n_word) {
#pragma unroll
        for (int q = 0; q < ROWS; ++q) sum[q] = 0.f;
      }
      if (passes == 1) {
#pragma unroll
        for (int q = 0; q < ROWS; ++q) acc[q] += sum[q];
      }
      if (passes > 1 || last_chunk) {
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          float v = passes == 1 ? acc[q] : sum[q];
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
          // this wavefront owns its rows: no race
          if (lane == 0 && r0 + q < d_out) {
            if (passes > 1 && w0 > 0) y[r0 + q] = y[r0 + q] + v;
            else y[r0 + q] = v;
          }
        }
      }
      cur = nxt;
    }
  }
}

// Launch of one instance: row groups of kGemvWaves * ROWS rows over at most 256 work-groups.  Two items of
// two rows fit the 128 registers of a 1024-thread work-group where a row's words and coefficients take at most
// kGemvItemRegs of them; otherwise rows are taken one at a time.
constexpr int kGemvItemRegs = 21;
template <int K, int W, int NG, int ROWS_, bool STRIDED>
static int launch_gemv(hipStream_t stream, const uint32_t* planes, const _Float16* coefs, int d_out, int d_in,
                       int group, const float* x, float* y) {
  constexpr int kRegs = K * W + (K + 1) * (!STRIDED && NG > 1 ? NG / 2 : NG);
  constexpr int ROWS = kRegs <= kGemvItemRegs ? ROWS_ : 1;
  BPDQ_HIP_TRY((bpdq_lds_limit<&gemv_planes_kernel<K, W, NG, ROWS, STRIDED>>(gemv_lds_bytes<W>())));
  const int nw = d_in / 32;
  // equal chunks, in whole lanes or (STRIDED) whole wavefronts
  const int n_chunk = bpdq_ceil_div(nw, 64 * W), unit = STRIDED ? 64 : W;
  const int chunk_words = bpdq_ceil_div(bpdq_ceil_div(nw, n_chunk), unit) * unit;
  const int units = bpdq_ceil_div(d_out, kGemvWaves * ROWS);
  const int passes = bpdq_ceil_div(units, 256);
  hipLaunchKernelGGL((gemv_planes_kernel<K, W, NG, ROWS, STRIDED>), dim3(bpdq_ceil_div(units, passes)), dim3(kGemvThreads),
                     gemv_lds_bytes<W>(), stream, planes, coefs, d_out, d_in, group, chunk_words, passes, x, y);
  BPDQ_LAUNCH_CHECK();
  return 0;
}

// Words per lane: the fewest that hold a row in one chunk, else four.  Consecutive ones, so that they are one
// load and share coefficients or find them side by side, where rows are whole lanes and a group is whole lanes or a
// lane whole groups -- unless they leave too many lanes idle: a row takes ceil(nw / 64) rounds of words
// strided over the lanes, and W n_chunk consecutive ones.  260 words (5 rounds to 8), 18944 rows, k = 2 g = 128:
// 27.6 us consecutive, 24.9 strided; 344 words (6 to 8), k = 4 47.5 and 40.8, but k = 2 8.6 and 8.6 at 4096 rows;
// 592 words (10 to 12) k = 2 12.4 and 13.3.
template <int K, int ROWS>
static int pick_gemv(hipStream_t stream, const uint32_t* planes, const _Float16* coefs, int d_out, int d_in, int group,
                     const float* x, float* y) {
  const int nw = d_in / 32, wpg = group / 32;
  if (nw <= 64) return launch_gemv<K, 1, 1, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y);
  const int W = nw <= 128 ? 2 : 4, strided = bpdq_ceil_div(nw, 64), consecutive = W * bpdq_ceil_div(nw, 64 * W);
  const bool idle = 8 * strided <= ((K >= 3 || wpg == 1) ? 6 : 5) * consecutive;
  const int per = wpg < W ? W / wpg : 1;               // groups to a lane
  const bool whole = nw % W == 0 && (wpg % W == 0 || W % wpg == 0) &&
                     reinterpret_cast<uintptr_t>(planes) % (4 * W) == 0 && reinterpret_cast<uintptr_t>(coefs) % (2 * per) == 0;
  if (W == 2) {
    if (!whole || idle) return launch_gemv<K, 2, 2, ROWS, true>(stream, planes, coefs, d_out, d_in, group, x, y);
    return per == 1 ? launch_gemv<K, 2, 1, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y)
                    : launch_gemv<K, 2, 2, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y);
  }
  if (!whole || idle) return launch_gemv<K, 4, 4, ROWS, true>(stream, planes, coefs, d_out, d_in, group, x, y);
  return per == 1   ? launch_gemv<K, 4, 1, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y)
         : per == 2 ? launch_gemv<K, 4, 2, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y)
                    : launch_gemv<K, 4, 4, ROWS, false>(stream, planes, coefs, d_out, d_in, group, x, y);
}

}  // namespace bpdq

using namespace bpdq;

extern "C" int bpdq_gemv(const uint32_t* planes, const uint16_t* coefs_h, int d_out, int d_in,
                         int bits, int group, const float* x, float* y, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!planes) return -1;
  if (!coefs_h || (reinterpret_cast<uintptr_t>(coefs_h) & 1)) return -2;
  if (d_out <= 0) return -3;
  if (d_in <= 0 || d_in % 32) return -4;
  if (bits < 1 || bits > 4) return -5;
  if (group < 32 || group % 32 || d_in % group) return -6;
  if (!x || (reinterpret_cast<uintptr_t>(x) & 15)) return -7;
  if (!y) return -8;
  const _Float16* ch = reinterpret_cast<const _Float16*>(coefs_h);
  const bool one = d_out <= kGemvRowsSplit;
  switch (bits) {
    case 1: return one ? pick_gemv<1, 1>(stream, planes, ch, d_out, d_in, group, x, y)
                       : pick_gemv<1, 2>(stream, planes, ch, d_out, d_in, group, x, y);
    case 2: return one ? pick_gemv<2, 1>(stream, planes, ch, d_out, d_in, group, x, y)
                       : pick_gemv<2, 2>(stream, planes, ch, d_out, d_in, group, x, y);
    case 3: return one ? pick_gemv<3, 1>(stream, planes, ch, d_out, d_in, group, x, y)
                       : pick_gemv<3, 2>(stream, planes, ch, d_out, d_in, group, x, y);
    default: return one ? pick_gemv<4, 1>(stream, planes, ch, d_out, d_in, group, x, y)
                        : pick_gemv<4, 2>(stream, planes, ch, d_out, d_in, group, x, y);
  }
}
