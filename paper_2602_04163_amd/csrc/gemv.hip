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
// Layout.  Lane l of a wavefront holds the WPL consecutive words WPL l ... of a chunk of 64 WPL words
// (one 16-byte load per plane and row at WPL = 4, and its words share a group's coefficients), and the
// table is T[q][j][nibble][lane] (q = nibble position in a word, j = word of the lane): whatever the
// nibbles are, the lanes of a wavefront fall into consecutive banks -- the minimum of two cycles.  The
// nibble is a whole byte of the LDS address, so after splitting a word into the bytes of its even and
// odd nibbles (3 instructions) one v_perm_b32 per look-up forms the address from the nibble and the
// lane's base; with the add that is 2.4 vector instructions per look-up.
//
// What bounds it: these instructions and the LDS reads (7 and 6 us on the 8192 x 29568 layer, whose
// 67 MB of planes and coefficients need 13 us at 5 TB/s).  The plane words and coefficients of the next
// chunk or row pass, and the x values of the next chunk, are requested before the current one is
// worked on; without that every chunk waited for memory twice.
// Measured, back to back in a graph (one word per lane and load, no prefetch -> this): 8192 x 29568 k = 2
// g = 64 50.5 -> 30.5 us (2.7 TB/s of stored bytes), 8192 x 8192 k = 2 13.6 -> 9.8, 3584 x 18944 k = 3
// 39.1 -> 16.9, 3584 x 3584 k = 2 7.1 -> 4.3 us.
#include "common.h"

namespace bpdq {

constexpr int kGemvThreads = 1024;
constexpr int kGemvWaves = kGemvThreads / 64;
constexpr int kGemvRowsSplit = 2 * 8 * 32 * kGemvWaves / 2;   // 4096: up to here one row per wavefront fills the CUs

template <int WPL>
constexpr size_t gemv_lds_bytes() { return (size_t)(8 * WPL * 16 * 64 + WPL * 64) * sizeof(float); }

// Plane words and coefficients of one (chunk, row pass) for this lane.
template <int K, int WPL, int NG, int ROWS>
struct GemvItem {
  uint32_t w[ROWS][K][WPL];
  _Float16 c[ROWS][K + 1][NG];
};

template <int K, int WPL, int NG, int ROWS>
__device__ __forceinline__ void gemv_fetch(const uint32_t* __restrict__ planes, const _Float16* __restrict__ coefs,
                                           int d_out, int nw, int n_grp, int wpg, bool vec, int r0, int w0,
                                           int n_word, int lane, GemvItem<K, WPL, NG, ROWS>& it) {
  typedef uint32_t words __attribute__((ext_vector_type(WPL == 1 ? 2 : WPL)));
  const int wl = WPL * lane;                     // first word of this lane inside the chunk
  const bool on = wl < n_word;
  const int wf = w0 + (on ? wl : 0);             // (idle lanes read the chunk's first words; their sums are dropped)
#pragma unroll
  for (int q = 0; q < ROWS; ++q) {
    const long r = r0 + q < d_out ? r0 + q : d_out - 1;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const uint32_t* p = planes + ((long)i * d_out + r) * nw + wf;
      if (WPL > 1 && vec) {
        const words v = *reinterpret_cast<const words*>(p);
#pragma unroll
        for (int j = 0; j < WPL; ++j) it.w[q][i][j] = v[j];
      } else {
#pragma unroll
        for (int j = 0; j < WPL; ++j) {
          const bool in = wl + j < n_word;
          const uint32_t v = p[in ? j : 0];
          it.w[q][i][j] = in ? v : 0u;
        }
      }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      int wg = wf + g * (WPL / NG);
      wg = wg < nw ? wg : nw - 1;
      const long G = wg / wpg;
#pragma unroll
      for (int i = 0; i <= K; ++i) {
        const _Float16 v = coefs[((long)i * d_out + r) * n_grp + G];
        // words past the end add nothing, whatever the coefficient: zero times an infinite one is not zero
        it.c[q][i][g] = (vec || wl + g * (WPL / NG) < n_word) ? v : (_Float16)0.f;
      }
    }
  }
}

// K planes; WPL words per lane; NG groups among a lane's words (WPL / NG consecutive words share one);
// ROWS rows per wavefront and pass.
template <int K, int WPL, int NG, int ROWS>
__global__ __launch_bounds__(kGemvThreads) void gemv_planes_kernel(const uint32_t* __restrict__ planes,
                                                                   const _Float16* __restrict__ coefs,
                                                                   int d_out, int d_in, int group, int chunk_words,
                                                                   int passes, int vec,
                                                                   const float* __restrict__ x,
                                                                   float* __restrict__ y) {
  extern __shared__ float lds[];
  float* T = lds;                                        // [8][WPL][16][64]
  float* Sw = lds + 8 * WPL * 16 * 64;                   // [WPL][64]: sum of x over each word
  constexpr int kSegs = 8 * WPL;                         // table segments of a lane
  constexpr int kSegPerThread = (kSegs + kGemvWaves - 1) / kGemvWaves;
  const int nw = d_in / 32, n_grp = d_in / group, wpg = group / 32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row_step = gridDim.x * kGemvWaves * ROWS;
  const int row_first = (blockIdx.x * kGemvWaves + wave) * ROWS;

  auto fetch_x = [&](int w0, int n_word, float4 (&xv)[kSegPerThread]) {
#pragma unroll
    for (int s = 0; s < kSegPerThread; ++s) {
      const int id = wave + kGemvWaves * s;              // segment (q, j) = (id / WPL, id % WPL)
      const int wl = WPL * lane + id % WPL;
      const bool in = id < kSegs && wl < n_word;
      const float4 v = *reinterpret_cast<const float4*>(x + (in ? 32L * (w0 + wl) + 4 * (id / WPL) : 0L));
      xv[s] = in ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  GemvItem<K, WPL, NG, ROWS> cur, nxt;
  float4 xv[kSegPerThread];
  const int n0 = nw < chunk_words ? nw : chunk_words;
  fetch_x(0, n0, xv);
  gemv_fetch<K, WPL, NG, ROWS>(planes, coefs, d_out, nw, n_grp, wpg, vec, row_first, 0, n0, lane, cur);
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
    if (tid < 64 * WPL) {
      const int j = tid >> 6;
      float sw = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) sw += T[((q * WPL + j) * 16 + 15) * 64 + lane];
      Sw[tid] = sw;
    }
    __syncthreads();
    if (!last_chunk) {
      const int w1 = w0 + chunk_words;
      fetch_x(w1, nw - w1 < chunk_words ? nw - w1 : chunk_words, xv);
    }
    for (int p = 0; p < passes; ++p) {
      const int r0 = row_first + p * row_step;
      if (r0 >= d_out) break;                            // uniform over the wavefront
      // the next item: the next pass of this chunk, else the first pass of the next chunk
      {
        const bool same = p + 1 < passes && r0 + row_step < d_out;
        const int rn = same ? r0 + row_step : row_first, wn = same ? w0 : w0 + chunk_words;
        if (wn < nw)
          gemv_fetch<K, WPL, NG, ROWS>(planes, coefs, d_out, nw, n_grp, wpg, vec, rn, wn,
                                       nw - wn < chunk_words ? nw - wn : chunk_words, lane, nxt);
      }
      float sum[ROWS];
#pragma unroll
      for (int q = 0; q < ROWS; ++q) sum[q] = 0.f;
      // LDS byte addresses (the table starts at LDS address 0: the kernel has no other LDS)
      const unsigned base0 = 4u * lane, base1 = 4u * lane + 65536u;
      typedef const __attribute__((address_space(3))) float lds_float;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float s = 0.f;
#pragma unroll
        for (int j = g * (WPL / NG); j < (g + 1) * (WPL / NG); ++j) s += Sw[j * 64 + lane];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          sum[q] = fmaf((float)cur.c[q][0][g], s, sum[q]);
#pragma unroll
          for (int i = 0; i < K; ++i) {
            float m = 0.f;                               // one chain of eight adds per word
#pragma unroll
            for (int j = g * (WPL / NG); j < (g + 1) * (WPL / NG); ++j) {
              float mj = 0.f;
              const uint32_t w = cur.w[q][i][j];
              const uint32_t ev = w & 0x0f0f0f0fu, od = (w >> 4) & 0x0f0f0f0fu;
#pragma unroll
              for (int n = 0; n < 8; ++n) {
                // address bytes: 0 = lane, 1 = the nibble, 2 and 3 = upper half of the table or not
                const unsigned off = (unsigned)(n * WPL + j) * 4096u;
                const unsigned a = __builtin_amdgcn_perm((n & 1) ? od : ev, off >= 65536u ? base1 : base0,
                                                         0x03020000u | (unsigned)((4 + (n >> 1)) << 8));
                mj += *reinterpret_cast<lds_float*>(a + (off & 65535u));
              }
              m += mj;
            }
            sum[q] = fmaf((float)cur.c[q][i + 1][g], m, sum[q]);
          }
        }
      }
      if (WPL * lane >= n_word) {
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
          if (lane == 0 && r0 + q < d_out) y[r0 + q] = (passes == 1 || w0 == 0 ? 0.f : y[r0 + q]) + v;
        }
      }
      cur = nxt;
    }
  }
}

// Launch of one instance: row groups of kGemvWaves * ROWS rows over at most 256 work-groups.  Two items of
// two rows do not fit the 128 registers of a 1024-thread work-group with three planes and four groups per
// lane, or with four planes and more than one: those take their rows one at a time.
template <int K, int WPL, int NG, int ROWS_>
static int launch_gemv(hipStream_t stream, const uint32_t* planes, const _Float16* coefs, int d_out, int d_in,
                       int group, const float* x, float* y) {
  constexpr int ROWS = (K <= 2 || (K == 3 && NG <= 2) || NG == 1) ? ROWS_ : 1;
  BPDQ_HIP_TRY((bpdq_lds_limit<&gemv_planes_kernel<K, WPL, NG, ROWS>>(gemv_lds_bytes<WPL>())));
  const int nw = d_in / 32;
  // equal chunks, in whole lanes
  const int n_chunk = bpdq_ceil_div(nw, 64 * WPL);
  const int chunk_words = bpdq_ceil_div(bpdq_ceil_div(nw, n_chunk), WPL) * WPL;
  const int vec = nw % WPL == 0 && (reinterpret_cast<uintptr_t>(planes) & (4 * WPL - 1)) == 0;
  const int units = bpdq_ceil_div(d_out, kGemvWaves * ROWS);
  const int passes = bpdq_ceil_div(units, 256);
  hipLaunchKernelGGL((gemv_planes_kernel<K, WPL, NG, ROWS>), dim3(bpdq_ceil_div(units, passes)), dim3(kGemvThreads),
                     gemv_lds_bytes<WPL>(), stream, planes, coefs, d_out, d_in, group, chunk_words, passes, vec, x, y);
  BPDQ_LAUNCH_CHECK();
  return 0;
}

// Words per lane: the fewest that hold a row in one chunk, else four (a row of 112 words would keep 28
// lanes busy at four words each, and 56 at two).  Groups among a lane's words: one where a group is a
// multiple of the lane's words, two where it is two words and the lane has four, else one per word.
template <int K, int ROWS>
static int pick_gemv(hipStream_t stream, const uint32_t* planes, const _Float16* coefs, int d_out, int d_in, int group,
                     const float* x, float* y) {
  const int nw = d_in / 32, wpg = group / 32;
  if (nw <= 64) return launch_gemv<K, 1, 1, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y);
  if (nw <= 128)
    return wpg % 2 == 0 ? launch_gemv<K, 2, 1, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y)
                        : launch_gemv<K, 2, 2, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y);
  if (wpg % 4 == 0) return launch_gemv<K, 4, 1, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y);
  return wpg % 2 == 0 ? launch_gemv<K, 4, 2, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y)
                      : launch_gemv<K, 4, 4, ROWS>(stream, planes, coefs, d_out, d_in, group, x, y);
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
