// Steps 3-4 of the pass, host side: the loop over blocks and groups (paper Sec. 3.2, 3.3) with
// the schedule of the lazy block updates (Eq. 4 applied to whole blocks; App. B.3 tail form) and
// the storage helpers.  The per-group kernels live in group_sweep.h.
#include "group_sweep.h"

namespace bpdq {

// The lazy block update as a launch of its own (group sizes whose sweep kernel cannot share a CU
// with it): the same tail role, one 128 x 128 tile per work-group.
__global__ __launch_bounds__(TailGemm::kThreads) void tail_update_kernel(TailArgs ta, const float* __restrict__ U,
                                                                         int ldu, int lde, int ldw, int d_out) {
  tail_role(ta, U, ldu, lde, ldw, d_out);
}

int launch_tail_update(hipStream_t stream, TailArgs ta, const float* U, int ldu, int lde, int ldw,
                       int d_out, int n_tiles) {
  BPDQ_HIP_TRY(bpdq_lds_limit<&tail_update_kernel>(TailGemm::kLdsBytes));
  ta.first_wg = 0;
  ta.far_wgs = bpdq_ceil_div(lde, TailGemm::kTileM) * ta.far.tiles_n;
  hipLaunchKernelGGL(tail_update_kernel, dim3(n_tiles), dim3(TailGemm::kThreads), TailGemm::kLdsBytes,
                     stream, ta, U, ldu, lde, ldw, d_out);
  BPDQ_LAUNCH_CHECK();
  return 0;
}

// working copy of W with dead input channels zeroed; the first kPackWGs n_grp work-groups lay out the group
// records of the factor instead (SuLayout), beside the copy, which is bound by memory.  ones: a fit follows
template <int G>
__global__ __launch_bounds__(256) void copy_in_kernel(const float* __restrict__ W, long n, int d_in,
                                                      const unsigned char* __restrict__ dead,
                                                      float* __restrict__ Wp, const float* __restrict__ U, int ones,
                                                      float* __restrict__ rec) {
  const int n_pack = kPackWGs<G> * (d_in / G);
  if ((int)blockIdx.x < n_pack) {
    const int gi = blockIdx.x / kPackWGs<G>, part = blockIdx.x % kPackWGs<G>;
    float* r = rec + (long)gi * SuLayout<G>::record_floats();
    if (part == 0) pack_p0<G>(U, d_in, gi * G, ones != 0, r);      // the longest first
    else pack_image<G>(U, d_in, gi * G, part - 1, r);
    return;
  }
  const long stride = (long)(gridDim.x - n_pack) * 1024;
  for (long e = ((long)(blockIdx.x - n_pack) * 256 + threadIdx.x) * 4; e < n; e += stride) {
    float4 v = *reinterpret_cast<const float4*>(W + e);
    if (dead) {
      const int c = (int)(e % d_in);
      if (dead[c]) v.x = 0.f;
      if (dead[c + 1]) v.y = 0.f;
      if (dead[c + 2]) v.z = 0.f;
      if (dead[c + 3]) v.w = 0.f;
    }
    *reinterpret_cast<float4*>(Wp + e) = v;
  }
}

// ------------------------------------------------------------------ storage helpers --------
__global__ __launch_bounds__(256) void pack_planes_kernel(const unsigned char* __restrict__ codes,
                                                          int d_out, int d_in, int bits,
                                                          uint32_t* __restrict__ planes) {
  const int n_word = d_in / 32;
  const long n = (long)d_out * n_word;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
    const unsigned char* cp = codes + e * 32;
    uint32_t word[4] = {0u, 0u, 0u, 0u};
    for (int j = 0; j < 32; ++j) {
      const int code = cp[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) word[i] |= (uint32_t)((code >> i) & 1) << j;
    }
    for (int i = 0; i < bits; ++i) planes[(long)i * n + e] = word[i];
  }
}

__device__ __forceinline__ float coef_value(float c) { return c; }
__device__ __forceinline__ float coef_value(_Float16 c) { return (float)c; }

// Eq. 1 from the packed format, ((C_0 + b_1 C_1) + b_2 C_2) + ... in fp32; CT = float or half.
// Bound by the store of W_hat.  A thread owns COLS consecutive columns of ROWS rows: all its loads are in flight
// before the first value is formed, and with four columns (of one group, W_hat 16-byte aligned) a row's values
// leave as one 16-byte store.  WIDE: a work-group is 256 threads of one row block; otherwise it is blockDim.x
// threads wide and blockDim.y row blocks high, so that narrow matrices fill it too (131072 x 32, 2 planes: 23.8 us
// with one row block per work-group, 15.5 with a thread per element, now 6.7).  Rows come from a grid-stride loop: no
// division per element (one 64-bit division and a modulo per element had cost most of the kernel).
// 4096 x 4096, 2 planes, half coefficients: 14.8 us on a matrix and a buffer that are in the cache, 19.7 (3.7 TB/s) on others
// in turn.  (8192 x 8192, before it went by tiles: 303 us with one thread per element and its own division, 66 with this.)
template <typename CT, int K, int COLS, int ROWS, bool WIDE>
__global__ __launch_bounds__(256) void dequant_kernel(const uint32_t* __restrict__ planes,
                                                      const CT* __restrict__ coefs, int d_out,
                                                      int d_in, int group, float* __restrict__ W_hat) {
  const int c = (blockIdx.x * (WIDE ? 256 : blockDim.x) + threadIdx.x) * COLS;
  if (c >= d_in) return;
  const int n_word = d_in / 32, n_grp = d_in / group;
  const int sh = c & 31, gi = c / group;
  const long step = (long)gridDim.y * (WIDE ? 1 : blockDim.y) * ROWS;
  for (long r0 = (WIDE ? (long)blockIdx.y : (long)blockIdx.y * blockDim.y + threadIdx.y) * ROWS; r0 < d_out; r0 += step) {
    uint32_t w[ROWS][K];
    CT cf[ROWS][K + 1];
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
      const long r = (r0 + q < d_out) ? r0 + q : d_out - 1;      // past the end: the last row again, not stored
#pragma unroll
      for (int i = 0; i < K; ++i) w[q][i] = planes[((long)i * d_out + r) * n_word + (c >> 5)];
#pragma unroll
      for (int i = 0; i <= K; ++i) cf[q][i] = coefs[((long)i * d_out + r) * n_grp + gi];
    }
#pragma unroll
    for (int q = 0; q < ROWS; ++q) {
      if (r0 + q >= d_out) break;
      float v[COLS];
#pragma unroll
      for (int e = 0; e < COLS; ++e) {
        v[e] = coef_value(cf[q][0]);
#pragma unroll
        for (int i = 0; i < K; ++i)
          if ((w[q][i] >> (sh + e)) & 1u) v[e] = v[e] + coef_value(cf[q][i + 1]);
      }
      float* out = W_hat + (r0 + q) * d_in + c;
      if constexpr (COLS == 4) *reinterpret_cast<float4*>(out) = make_float4(v[0], v[1], v[2], v[3]);
      else *out = v[0];
    }
  }
}

// The same for large matrices whose groups hold whole plane words: a work-group stages the words and coefficients of a
// tile of kTileRows x kTileCols in LDS and forms the tile from there.  Stores alone reach 7.0 TB/s on this card
// (8192 x 8192: 38.5 us), the loads alone took 19 us and the two together 57: a thread that forms four columns of a row loads
// K words and K + 1 coefficients that its seven neighbours load too, 20 small requests for every 16 values, and they
// queue with the stores.  Staged, a row's words come as 256 consecutive bytes per plane, 4 K loads per thread and tile.
// 8192 x 8192, 2 planes, half coefficients, the same matrix into the same buffer: 62 -> 46 us (16 x 1024 tiles 49, 8 x 4096 46,
// 32 x 1024 50; a second tile's loads ahead of the stores gains nothing); matrices and buffers in turn, on another day, 66 -> 57
// (5.0 TB/s; the former then 64 -> 48).
constexpr int kTileRows = 16, kTileCols = 2048;
template <int K>
constexpr int kTileCoefs = K < 4 ? 4 : 8;           // floats a (row, group) takes in LDS

template <typename CT, int K>
__global__ __launch_bounds__(256) void dequant_tile_kernel(const uint32_t* __restrict__ planes, const CT* __restrict__ coefs,
                                                           int d_out, int d_in, int group, float* __restrict__ W_hat) {
  constexpr int kWords = kTileCols / 32, CP = kTileCoefs<K>, kLoads = K * kTileRows * kWords / 256;
  extern __shared__ uint32_t sW[];                                      // [plane][row][word]
  float* sC = reinterpret_cast<float*>(sW + K * kTileRows * kWords);    // [row][group of the tile][CP]
  const int n_word = d_in / 32, n_grp = d_in / group, tid = threadIdx.x;
  const int c0 = blockIdx.x * kTileCols, w0 = c0 / 32, g0 = c0 / group;
  const int c1 = c0 + kTileCols < d_in ? c0 + kTileCols : d_in;
  const int last_word = (c1 - 1) / 32, n_c = (c1 - 1) / group - g0 + 1, n_coef = kTileRows * n_c * (K + 1);
  const int row_tiles = (d_out + kTileRows - 1) / kTileRows;
  for (int t = blockIdx.y; t < row_tiles; t += gridDim.y) {
    const int r0 = t * kTileRows;
    auto row = [&](int r) { return (long)(r0 + r < d_out ? r0 + r : d_out - 1); };      // past the end: the last row, not stored
    uint32_t w[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = tid + 256 * u, x = e % kWords, r = e / kWords % kTileRows, i = e / kWords / kTileRows;
      w[u] = planes[((long)i * d_out + row(r)) * n_word + (w0 + x <= last_word ? w0 + x : w0)];
    }
    for (int e0 = tid; e0 < n_coef; e0 += 1024) {
      CT c[4];
      int to[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + 256 * u < n_coef ? e0 + 256 * u : e0;
        const int g = e % n_c, rr = e / n_c, r = rr % kTileRows, i = rr / kTileRows;
        c[u] = coefs[((long)i * d_out + row(r)) * n_grp + g0 + g];
        to[u] = (r * n_c + g) * CP + i;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) sC[to[u]] = coef_value(c[u]);
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) sW[tid + 256 * u] = w[u];
    __syncthreads();
    for (int q = 0; q < kTileRows && r0 + q < d_out; ++q) {
#pragma unroll
      for (int u = 0; u < kTileCols / 1024; ++u) {
        const int x = 4 * tid + 1024 * u, c = c0 + x;
        if (c >= d_in) break;
        const float* f = sC + (q * n_c + c / group - g0) * CP;
        const float4 f0 = *reinterpret_cast<const float4*>(f);
        const float cf[5] = {f0.x, f0.y, f0.z, f0.w, K < 4 ? 0.f : f[K < 4 ? 0 : 4]};
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = cf[0];
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const uint32_t word = sW[(i * kTileRows + q) * kWords + x / 32] >> (x & 31);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if ((word >> e) & 1u) v[e] = v[e] + cf[i + 1];
        }
        *reinterpret_cast<float4*>(W_hat + (long)(r0 + q) * d_in + c) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
    __syncthreads();                                                    // (the next tile's words go to the same place)
  }
}

__global__ __launch_bounds__(256) void coefs_to_fp16_kernel(const float* __restrict__ coefs, long n,
                                                            _Float16* __restrict__ out) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256)
    out[e] = (_Float16)coefs[e];                 // v_cvt_f16_f32: round to nearest even
}

// ------------------------------------------------------------------ host side --------------
static int check_params(int d_out, int d_in, const bpdq_params* p) {
  if (!p) return 1;
  if (p->bits < 1 || p->bits > 4) return 1;
  if (p->group != 32 && p->group != 64 && p->group != 128 && p->group != 256) return 1;
  if (p->group == 256 && p->bits > 3) return 1;      // 4 planes at g = 256 are not built (see header)
  if (d_in % p->group || d_in % 32) return 1;
  const int B = p->block > p->group ? p->block : p->group;
  if (p->block < 1 || B % p->group) return 1;
  if (p->refine_iters < 0 || p->refine_iters > kMaxIters) return 1;
  if (!(p->alpha >= 0.f)) return 1;
  if (p->grid != BPDQ_GRID_VARIABLE && p->grid != BPDQ_GRID_UNIFORM) return 1;
  if (p->coef_fp16 != 0 && p->coef_fp16 != 1) return 1;
  if (d_out <= 0 || d_in <= 0) return 1;
  return 0;
}

static GroupLauncher pick_group(int k, int g) {
  if (g == 256) {
    switch (k) {
      case 1: return group256_k1();
      case 2: return group256_k2();
      case 3: return group256_k3();
    }
    return nullptr;
  }
  switch (k) {
    case 1: return pick_group_k1(g);
    case 2: return pick_group_k2(g);
    case 3: return pick_group_k3(g);
    case 4: return pick_group_k4(g);
  }
  return nullptr;
}

}  // namespace bpdq

using namespace bpdq;

extern "C" int bpdq_version(void) { return 100; }

extern "C" size_t bpdq_quantize_workspace_bytes(int d_out, int d_in, const bpdq_params* p) {
  if (check_params(d_out, d_in, p)) return 0;
  return quant_layout(d_out, d_in, *p).total;
}

static int quantize_rows(const float* W, int d_out, int d_in, const float* U,
                         const unsigned char* dead, const bpdq_params* p, const SegArgs& seg,
                         uint32_t* planes, float* coefs, float* W_hat, double* grp_err,
                         int* grp_iter, void* ws, size_t ws_bytes, hipStream_t stream) {
  const QuantLayout L = quant_layout(d_out, d_in, *p);
  if (ws_bytes < L.total) return -13;
  char* base = static_cast<char*>(ws);
  float* Wp = reinterpret_cast<float*>(base + L.wp_off);
  float* Eall = reinterpret_cast<float*>(base + L.eall_off);
  GroupLauncher group = pick_group(p->bits, p->group);
  if (!group) return -6;

  const long n = (long)d_out * d_in;
  const int copy_wgs = (int)((n / 4 + 255) / 256 < 65536 ? (n / 4 + 255) / 256 : 65536);
  float* rec = reinterpret_cast<float*>(base + L.rec_off);
  const int ones = p->grid != BPDQ_GRID_UNIFORM;
  auto copy_in = [&](auto kern, int pack_wgs) {
    hipLaunchKernelGGL(kern, dim3(copy_wgs + pack_wgs * (d_in / p->group)), dim3(256), 0, stream, W, n, d_in, dead, Wp, U,
                       ones, rec);
  };
  switch (p->group) {
    case 32: copy_in(copy_in_kernel<32>, kPackWGs<32>); break;
    case 64: copy_in(copy_in_kernel<64>, kPackWGs<64>); break;
    case 128: copy_in(copy_in_kernel<128>, kPackWGs<128>); break;
    default: copy_in(copy_in_kernel<256>, kPackWGs<256>); break;
  }
  BPDQ_LAUNCH_CHECK();

  // Blocks of B columns, groups of g inside.  W' only ever receives whole-block updates, one
  // block late: the first group launch of block q carries the update of block q-1 to the columns
  // beyond block q (tail role), and every group of block q reads the updates of block q-1 and of
  // the earlier groups of its own block left-looking from the committed E*.
  // Two levels (see TailArgs): with super-blocks of SBc columns, the update of a block of
  // super-block S reaches only to the end of super-block S + 1; the columns from super-block S + 2
  // on receive ONE update of depth SBc for all of super-block S, applied during the launches of
  // super-block S + 1: its first launch takes the columns of super-block S + 2 (the per-block
  // update of that launch, from the last block of S, ends where they begin), the other launches
  // share the columns beyond (which no per-block update of super-block S + 1 reaches).  Two
  // updates of one launch thus never meet, and a column has received every earlier block's term
  // before its own block starts.
  const int g = p->group, B = L.B;
  const int SBc = B >= 1024 ? B : B * (1024 / B);
  auto make_task = [&](int k0, int Kd, long c0, long c1) {
    TailTask t{};
    c0 = c0 < d_in ? c0 : d_in;
    c1 = c1 < d_in ? c1 : d_in;
    if (c1 > c0) {
      t.Et = Eall + (long)k0 * L.lde;
      t.Kd = Kd;
      t.k0 = k0;
      t.c_begin = (int)c0;
      t.c_end = (int)c1;
      t.tiles_n = bpdq_ceil_div((int)(c1 - c0), TailGemm::kTileN);
    }
    return t;
  };
  for (int b0 = 0; b0 < d_in; b0 += B) {
    const int b1 = b0 + B < d_in ? b0 + B : d_in;
    const int kp0 = b0 > 0 ? b0 - B : 0;
    const int sb0 = b0 / SBc * SBc;                         // start of this block's super-block
    for (int s0 = b0; s0 < b1; s0 += g) {
      TailArgs ta{};
      ta.Wp = Wp;
      if (s0 == b0 && b0 > 0)     // per-block update of block q-1: to the end of the super-block after its own
        ta.near = make_task(kp0, B, b1, ((long)(kp0 / SBc) + 2) * SBc);
      if (sb0 > 0) {
        // deep update of the previous super-block [sb0 - SBc, sb0), columns from sb0 + SBc on
        const int li = (s0 - sb0) / g, n_l = SBc / g;
        const long f0 = (long)sb0 + SBc, f1 = f0 + SBc;      // the next super-block's columns
        if (li == 0) {
          ta.far = make_task(sb0 - SBc, SBc, f0, f1);
        } else if (f1 < d_in) {
          const int cols = bpdq_ceil_div(bpdq_ceil_div(d_in - (int)f1, TailGemm::kTileN), n_l - 1) * TailGemm::kTileN;
          ta.far = make_task(sb0 - SBc, SBc, f1 + (long)(li - 1) * cols, f1 + (long)li * cols);
        }
      }
      const int rc = group(stream, Wp, d_out, d_in, U, s0, kp0, ta, seg, *p, L, base, planes, coefs,
                           W_hat, grp_err, grp_iter);
      if (rc) return rc;
    }
  }
  return 0;
}

extern "C" int bpdq_quantize_layer(const float* W, int d_out, int d_in, const float* U,
                                   const unsigned char* dead, const bpdq_params* p,
                                   uint32_t* planes, float* coefs, float* W_hat, double* grp_err,
                                   int* grp_iter, void* ws, size_t ws_bytes, void* stream_) {
  if (!W || (reinterpret_cast<uintptr_t>(W) & 15)) return -1;
  if (d_out <= 0) return -2;
  if (d_in <= 0 || d_in % 32) return -3;
  if (!U || (reinterpret_cast<uintptr_t>(U) & 15)) return -4;
  if (check_params(d_out, d_in, p)) return -6;
  if (!planes) return -7;
  if (!coefs) return -8;
  if (!grp_err) return -10;
  if (!grp_iter) return -11;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) return -12;
  SegArgs seg{};
  seg.n_seg = 1;
  seg.wg_end[0] = bpdq_ceil_div(d_out, kRowsPerWG);
  return quantize_rows(W, d_out, d_in, U, dead, p, seg, planes, coefs, W_hat, grp_err, grp_iter, ws,
                       ws_bytes, static_cast<hipStream_t>(stream_));
}

extern "C" int bpdq_quantize_layers(const float* W, int d_out, int d_in, const float* U,
                                    const unsigned char* dead, const bpdq_params* p, int n_seg,
                                    const int* seg_end, uint32_t* planes, float* coefs,
                                    float* W_hat, double* grp_err, int* grp_iter, void* ws,
                                    size_t ws_bytes, void* stream_) {
  if (!W || (reinterpret_cast<uintptr_t>(W) & 15)) return -1;
  if (d_out <= 0) return -2;
  if (d_in <= 0 || d_in % 32) return -3;
  if (!U || (reinterpret_cast<uintptr_t>(U) & 15)) return -4;
  if (check_params(d_out, d_in, p)) return -6;
  if (n_seg < 1 || n_seg > kMaxSegments) return -7;
  if (!seg_end) return -8;
  SegArgs seg{};
  seg.n_seg = n_seg;
  int prev = 0;
  for (int s = 0; s < n_seg; ++s) {
    const int e = seg_end[s];
    // every layer but the last must end on a work-group boundary (16 rows)
    if (e <= prev || e > d_out || (s + 1 < n_seg && e % kRowsPerWG)) return -8;
    seg.wg_end[s] = bpdq_ceil_div(e, kRowsPerWG);
    prev = e;
  }
  if (prev != d_out) return -8;
  if (!planes) return -9;
  if (!coefs) return -10;
  if (!grp_err) return -12;
  if (!grp_iter) return -13;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) return -14;
  const int rc = quantize_rows(W, d_out, d_in, U, dead, p, seg, planes, coefs, W_hat, grp_err,
                               grp_iter, ws, ws_bytes, static_cast<hipStream_t>(stream_));
  return rc == -13 ? -15 : rc;
}

extern "C" int bpdq_block_update(const float* Et, int lde, int Kd, const float* U, int ldu, int k0,
                                 float* Wp, int ldw, int d_out, int c_begin, int c_end, void* stream_) {
  if (!Et || (reinterpret_cast<uintptr_t>(Et) & 15)) return -1;
  if (lde < d_out || lde % 4) return -2;
  if (Kd <= 0) return -3;
  if (!U || (reinterpret_cast<uintptr_t>(U) & 15)) return -4;
  if (ldu < c_end || ldu % 4) return -5;
  if (k0 < 0) return -6;
  if (!Wp) return -7;
  if (ldw < c_end) return -8;
  if (d_out <= 0) return -9;
  if (c_begin < 0 || c_begin % 4) return -10;
  if (c_end < c_begin || c_end % 4) return -11;
  if (c_end == c_begin) return 0;
  TailArgs ta{};
  ta.Wp = Wp;
  ta.near.Et = Et;
  ta.near.Kd = Kd;
  ta.near.k0 = k0;
  ta.near.c_begin = c_begin;
  ta.near.c_end = c_end;
  ta.near.tiles_n = bpdq_ceil_div(c_end - c_begin, TailGemm::kTileN);
  const int n_tiles = bpdq_ceil_div(lde, TailGemm::kTileM) * ta.near.tiles_n;
  return launch_tail_update(static_cast<hipStream_t>(stream_), ta, U, ldu, lde, ldw, d_out, n_tiles);
}

extern "C" int bpdq_pack_planes(const unsigned char* codes, int d_out, int d_in, int bits,
                                uint32_t* planes, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (!codes) return -1;
  if (d_out <= 0) return -2;
  if (d_in <= 0 || d_in % 32) return -3;
  if (bits < 1 || bits > 4) return -4;
  if (!planes) return -5;
  const long n = (long)d_out * (d_in / 32);
  const int grid = (int)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
  hipLaunchKernelGGL(pack_planes_kernel, dim3(grid), dim3(256), 0, stream, codes, d_out, d_in, bits, planes);
  BPDQ_LAUNCH_CHECK();
  return 0;
}

template <typename CT>
static int launch_dequant(const uint32_t* planes, const CT* coefs, int d_out, int d_in, int bits, int group,
                          float* W_hat, hipStream_t stream) {
  if (!planes) return -1;
  if (!coefs) return -2;
  if (d_out <= 0) return -3;
  if (d_in <= 0 || d_in % 32) return -4;
  if (bits < 1 || bits > 4) return -5;
  if (group <= 0 || d_in % group) return -6;
  if (!W_hat) return -7;
  const bool vec = group % 4 == 0 && (reinterpret_cast<uintptr_t>(W_hat) & 15) == 0;
  // Several rows per thread once one would already fill the chip (2 planes: 1024 x 1056, 270 k threads of one row, 4.8 us
  // against 4.3 with four; 256 x 1056 3.2 against 3.5; scalar stores, groups of 2: 256 x 1056 3.3 us with one row and
  // 4.0 with eight, 4096 x 8192 67 and 53).
  const int per = vec ? 4 : 1;
  const bool many = (long)d_out * d_in / per >= (vec ? 1L << 18 : 1L << 20);
  const int cols = d_in / per, rows = many ? (vec ? 4 : 8) : 1;
  int width = 256;                                       // threads along the columns: as many as there are, to a power of two
  while (width / 2 >= cols) width /= 2;
  const int row_blocks = bpdq_ceil_div(bpdq_ceil_div(d_out, rows), 256 / width);
  auto launch = [&](auto kern) -> int {
    hipLaunchKernelGGL(kern, dim3(bpdq_ceil_div(cols, width), row_blocks < 65535 ? row_blocks : 65535),
                       dim3(width, 256 / width), 0, stream, planes, coefs, d_out, d_in, group, W_hat);
    BPDQ_LAUNCH_CHECK();
    return 0;
  };
  // Tiles through LDS where there are four for every compute unit and their columns are in use: one tile of 1024 or more, or
  // seven eighths of several.  us, a thread's own loads / tiles, half coefficients; first the same matrix into the same buffer
  // again and again, then matrices and buffers in turn that nothing has touched for a gigabyte:
  //   8192 x 8192 63.6 / 48.2 and 66.4 / 57.4 at 2 planes and groups of 128, 78.5 / 60.2 and 82.3 / 65.5 at 4 and 64; 8192 x 3584
  //   25.5 / 20.9 and 34.2 / 24.5; 16384 x 1280 22.2 / 17.4 and 28.2 / 19.6; 16384 x 2048 24.0 / 23.7 and 34.2 / 28.1; 70000 x 1024,
  //   groups of 64, 69.2 / 57.5 and 69.4 / 60.2.
  // On the other side of the line: 4096 x 4096, 512 tiles, 14.8 / 13.8 and 19.7 / 14.7, but 3000 x 6016, 564, 18.1 / 20.2 and
  //   24.4 / 22.6 at 3 planes and groups of 32 (staging is a round trip to memory that only other work-groups hide, and
  //   units with three tiles wait for those with two); 9300 x 3072, the second of two tiles half full, 21.4 / 22.6 and 30.6 / 25.6;
  //   8192 x 2304, an eighth full, 16.6 / 19.2 and 22.5 / 19.6.  (The line follows the first kind.)
  // Four planes in groups of 32 fill so much LDS that a unit holds three tiles, which hides less; with 32-bit coefficients, twice
  // the bytes to stage, that costs more than the tiles save until there are 2048, unless the other kernel's blocks of 1024 columns
  // are not full: 16384 x 2048 31.0 / 35.1 and 40.5 / 43.3, 24576 x 2048 43.5 / 44.1 and 57.9 / 60.1, 32768 x 2048 85.9 / 84.1 and
  // 85.5 / 84.3; 16384 x 1280 29.4 / 23.3 and 34.1 / 26.7.  With half coefficients 16384 x 2048 31.8 / 34.5 and 41.5 / 42.4, 8192 x 4096
  // 31.2 / 33.7 and 42.6 / 41.3, 16384 x 1024 19.4 / 19.6 and 23.5 / 19.9, 20000 x 2048 37.0 / 35.8 and 50.6 / 46.7: tiles, as a program
  // that reads its layers once a pass has the second kind.
  const int col_tiles = bpdq_ceil_div(d_in, kTileCols);
  const long n_tiles = (long)bpdq_ceil_div(d_out, kTileRows) * col_tiles;
  const bool many_coefs = sizeof(CT) == 4 && bits == 4 && group == 32;
  const bool tiles = vec && group % 32 == 0 && d_in >= 1024 && (col_tiles == 1 || 8L * d_in >= 7L * col_tiles * kTileCols) &&
                     n_tiles >= (many_coefs && d_in % 1024 == 0 ? 2048 : 1024);
  auto pick = [&](auto planes_of) -> int {
    constexpr int K = decltype(planes_of)::value;
    if (tiles) {
      const int groups = (d_in < kTileCols ? d_in : kTileCols) / group + 2;
      const size_t lds = (size_t)(K * kTileRows * kTileCols / 32 + kTileRows * groups * kTileCoefs<K>) * 4;
      const int row_tiles = bpdq_ceil_div(d_out, kTileRows);
      hipLaunchKernelGGL((dequant_tile_kernel<CT, K>), dim3(col_tiles, row_tiles < 65535 ? row_tiles : 65535),
                         dim3(256), lds, stream, planes, coefs, d_out, d_in, group, W_hat);
      BPDQ_LAUNCH_CHECK();
      return 0;
    }
    if (!vec) return many ? launch(dequant_kernel<CT, K, 1, 8, false>) : launch(dequant_kernel<CT, K, 1, 1, false>);
    if (width < 256) return many ? launch(dequant_kernel<CT, K, 4, 4, false>) : launch(dequant_kernel<CT, K, 4, 1, false>);
    return many ? launch(dequant_kernel<CT, K, 4, 4, true>) : launch(dequant_kernel<CT, K, 4, 1, true>);
  };
  switch (bits) {
    case 1: return pick(std::integral_constant<int, 1>{});
    case 2: return pick(std::integral_constant<int, 2>{});
    case 3: return pick(std::integral_constant<int, 3>{});
    default: return pick(std::integral_constant<int, 4>{});
  }
}

extern "C" int bpdq_dequant(const uint32_t* planes, const float* coefs, int d_out, int d_in,
                            int bits, int group, float* W_hat, void* stream_) {
  return launch_dequant(planes, coefs, d_out, d_in, bits, group, W_hat,
                        static_cast<hipStream_t>(stream_));
}

extern "C" int bpdq_dequant_fp16(const uint32_t* planes, const uint16_t* coefs_h, int d_out,
                                 int d_in, int bits, int group, float* W_hat, void* stream_) {
  if (coefs_h && (reinterpret_cast<uintptr_t>(coefs_h) & 1)) return -2;
  return launch_dequant(planes, reinterpret_cast<const _Float16*>(coefs_h), d_out, d_in, bits, group, W_hat,
                        static_cast<hipStream_t>(stream_));
}

extern "C" int bpdq_coefs_to_fp16(const float* coefs, long n, uint16_t* out, void* stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (n < 0) return -2;
  if (n == 0) return 0;
  if (!coefs) return -1;
  if (!out || (reinterpret_cast<uintptr_t>(out) & 1)) return -3;
  const int grid = (int)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
  hipLaunchKernelGGL(coefs_to_fp16_kernel, dim3(grid), dim3(256), 0, stream, coefs, n,
                     reinterpret_cast<_Float16*>(out));
  BPDQ_LAUNCH_CHECK();
  return 0;
}
