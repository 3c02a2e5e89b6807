// fp32 linear layers C = A W^T (A [M, K], W [N, K], both K-contiguous) on v_mfma_f32_16x16x4_f32, for the fp32
// models.  The matrix instruction multiplies and accumulates in fp32, so nothing is given up against vector FMAs,
// and it asks for a quarter of their operand traffic.
//
// A wave owns 32 tokens x 32 weight rows (2 x 2 blocks of 16 x 16).  Operands go from global memory (L2) straight
// into operand layout: a lane reads 16 bytes of row lane % 16 at k = 4 (lane / 16) of a 16-wide k chunk and spends
// element s of them in matrix instruction s.  The k order inside a chunk is then 0, 4, 8, 12, 1, 5, ...; both
// operands use the same one.  No LDS and no barrier in the loop: a chunk's four loads (4 KB) stand against sixteen
// matrix instructions of 32 clocks, half of what a CU's vector-memory path moves.
//
// Which waves make a workgroup (chosen by the launcher from the number of 32 x 32 tiles, see launch_f32_t):
//   8 or 4 waves splitting K on one tile   a prompt of a few hundred tokens through a small model has 64-256 tiles; the
//                                          partial tiles are summed through LDS in wave order;
//   2 x 2 waves of 64 x 64 each            many tiles (k_gemm_f32_wide).
// One fp32 prompt of 512 tokens (hidden 256, mlp 688): 36-88 us per product on the vector ALUs, where a workgroup
// walked K alone with its staging in the open, against 6-12 us here (launch, one or two trips to L2, the sum).
// 4096 x 4096 x 4096: 2218 us on the vector ALUs, 2729 with waves of 32 x 32, 1405 (98 TFLOP/s) with 64 x 64.
//
// Folded in, each one launch less per layer: RMSNorm of the input (the operand is x * gain, the row's 1 / rms - its
// sum of squares comes from the same loads - multiplies the accumulators), RoPE of the leading segments (the two
// weight blocks of a wave are 16 rotation partners each, so a lane holds both halves of its pairs), SiLU(gate) * up
// (the blocks are 16 gate and 16 up rows), and a row list for A.
#include "common.hpp"

namespace fastav {

struct F32GemmArgs {
  const float* x;                // [M, K] input rows (row list: [n_src, K])
  const int32_t* rows;           // optional: output row r reads x row rows[r]
  const float* w[3];             // up to three [rows, K] matrices stacked along the output dimension
  int seg_end[3];                // exclusive end column of each (multiples of 32 when there are several)
  const float* w2;               // "up" matrix (SwiGLU only)
  float* c[3];                   // output of each segment, row pitch ldc elements
  int64_t ldc[3];
  int M, N, K, tiles_n;
  const float* g;                // NORM: gain [K]
  float eps;
  const int32_t* rope_pos;       // rotate the first rope_cols output columns (whole heads of dh), or rope_tab == nullptr
  const float2* rope_tab;        // [position][dh / 2] = (cos, sin)
  int dh, rope_cols;
};

// The two 16-row weight blocks of a tile and the output column each starts at (inside its segment).
struct F32Cols { int seg, n_seg, nb[2], f0; bool rope; };
template <int EPI>
__device__ __forceinline__ F32Cols f32_cols(const F32GemmArgs& a, int tile) {
  F32Cols c;
  int seg0 = 0;
  c.seg = 0;
  const int n0 = EPI == FASTAV_EPI_SWIGLU ? tile * 16 : tile * 32;
  if (EPI != FASTAV_EPI_SWIGLU) {
    if (n0 >= a.seg_end[0]) { c.seg = 1; seg0 = a.seg_end[0]; }
    if (n0 >= a.seg_end[1]) { c.seg = 2; seg0 = a.seg_end[1]; }
  }
  c.rope = EPI == FASTAV_EPI_STORE && a.rope_tab != nullptr && n0 < a.rope_cols;
  c.nb[0] = n0 - seg0;
  c.nb[1] = n0 - seg0 + 16;
  c.f0 = 0;                                             // rope: frequency index of the block's first column
  if (c.rope) {
    const int per_head = a.dh / 32, t = (n0 - seg0) / 32;
    c.f0 = (t % per_head) * 16;
    c.nb[0] = (t / per_head) * a.dh + c.f0;
    c.nb[1] = c.nb[0] + a.dh / 2;
  }
  c.n_seg = (EPI == FASTAV_EPI_SWIGLU) ? a.N : (a.seg_end[c.seg] < a.N ? a.seg_end[c.seg] : a.N) - seg0;
  return c;
}
// This lane's address in weight block j of the tile; rows past the segment repeat its last one and are not stored.
template <int EPI>
__device__ __forceinline__ const float* f32_weights(const F32GemmArgs& a, const F32Cols& c, int j, int l16, int l4) {
  const int nb = c.nb[EPI == FASTAV_EPI_SWIGLU ? 0 : j];
  const int n = nb + l16 < c.n_seg ? nb + l16 : c.n_seg - 1;
  return (EPI == FASTAV_EPI_SWIGLU ? (j ? a.w2 : a.w[0]) : a.w[c.seg]) + (int64_t)n * a.K + l4 * 4;
}
__device__ __forceinline__ const float* f32_input(const F32GemmArgs& a, int m, int l4) {
  m = m < a.M ? m : a.M - 1;
  return a.x + (int64_t)(a.rows ? a.rows[m] : m) * a.K + l4 * 4;
}

// Output of one token (row m) in the two weight blocks: element r is column nb[j] + l4 * 4 + r.
template <int EPI, bool NORM>
__device__ __forceinline__ void f32_store(const F32GemmArgs& a, const F32Cols& c, int m, int l4, f32x4_t v0, f32x4_t v1, float ss) {
  f32x4_t v[2] = {v0, v1};
  if (NORM) {
    const float r = 1.0f / sqrtf(ss / (float)a.K + a.eps);
    v[0] = v[0] * r; v[1] = v[1] * r;
  }
  if (c.rope) {
    const float2* tr = a.rope_tab + (int64_t)a.rope_pos[m] * (a.dh / 2) + c.f0 + l4 * 4;
    const f32x4_t t0 = *(const f32x4_t*)tr, t1 = *(const f32x4_t*)(tr + 2);
    const float cs[4] = {t0[0], t0[2], t1[0], t1[2]}, sn[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float x1 = v[0][r], x2 = v[1][r];
      v[0][r] = x1 * cs[r] - x2 * sn[r];
      v[1][r] = x2 * cs[r] + x1 * sn[r];
    }
  }
  if (EPI == FASTAV_EPI_SWIGLU) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[0][r] = v[0][r] / (1.0f + expf(-v[0][r])) * v[1][r];
  }
  float* const cb = a.c[c.seg];
  const int64_t ldc = a.ldc[c.seg];
  const bool vec = ldc % 4 == 0 && ((uintptr_t)cb % 16) == 0;
#pragma unroll
  for (int j = 0; j < (EPI == FASTAV_EPI_SWIGLU ? 1 : 2); ++j) {
    const int n = c.nb[j] + l4 * 4;
    float* p = cb + (int64_t)m * ldc + n;
    if (vec && n + 3 < c.n_seg) {
      if (EPI == FASTAV_EPI_RESADD) v[j] = v[j] + *(const f32x4_t*)p;
      *(f32x4_t*)p = v[j];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (n + r < c.n_seg) p[r] = (EPI == FASTAV_EPI_RESADD) ? p[r] + v[j][r] : v[j][r];
    }
  }
}

// Products of many tiles: a workgroup of 2 x 2 waves, a wave owns 64 tokens x two tiles' weight blocks (64 rows), so that a
// chunk's eight loads (8 KB) stand against 64 matrix instructions; the next chunk is requested before the present one is used.
// Sums run over K in the order of the one-tile form.
template <int EPI, bool NORM>
__global__ __launch_bounds__(256, 2) void k_gemm_f32_wide(F32GemmArgs a) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m0 = (int)blockIdx.y * 128 + (wave >> 1) * 64;
  const int tile = (int)blockIdx.x * 4 + (wave & 1) * 2;
  if (m0 >= a.M || tile >= a.tiles_n) return;
  const int n_tiles = tile + 1 < a.tiles_n ? 2 : 1;
  const F32Cols cols[2] = {f32_cols<EPI>(a, tile), f32_cols<EPI>(a, tile + n_tiles - 1)};     // an odd last tile: twice, stored once
  const float *wp[4], *xp[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) wp[j] = f32_weights<EPI>(a, cols[j >> 1], j & 1, l16, l4);
#pragma unroll
  for (int i = 0; i < 4; ++i) xp[i] = f32_input(a, m0 + i * 16 + l16, l4);
  const float* gp = NORM ? a.g + l4 * 4 : nullptr;
  f32x4_t acc[4][4];                                    // [token block][weight block]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss[4] = {0.f, 0.f, 0.f, 0.f};

  auto load = [&](f32x4_t (&xf)[4], f32x4_t (&wf)[4], f32x4_t& gf, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) xf[i] = *(const f32x4_t*)(xp[i] + k);
#pragma unroll
    for (int j = 0; j < 4; ++j) wf[j] = *(const f32x4_t*)(wp[j] + k);
    if (NORM) gf = *(const f32x4_t*)(gp + k);
  };
  auto compute = [&](f32x4_t (&xf)[4], const f32x4_t (&wf)[4], const f32x4_t& gf) __attribute__((always_inline)) {
    if (NORM) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ss[i] = fmaf(xf[i][e], xf[i][e], ss[i]);
          xf[i][e] *= gf[e];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[j][e], xf[i][e], acc[i][j], 0, 0, 0);
  };
  const int whole = a.K & ~15;
  f32x4_t x0[4], w0[4], x1[4], w1[4], g0, g1;
  int k = 0;
  if (whole > 0) {
    load(x0, w0, g0, 0);
    for (; k + 32 < whole; k += 32) {                   // both chunks of the body have one behind them
      load(x1, w1, g1, k + 16);
      compute(x0, w0, g0);
      load(x0, w0, g0, k + 32);
      compute(x1, w1, g1);
    }
    if (k + 16 < whole) {
      load(x1, w1, g1, k + 16);
      compute(x0, w0, g0);
      compute(x1, w1, g1);
    } else {
      compute(x0, w0, g0);
    }
  }
  if (whole < a.K) {                                    // K is a multiple of 4: a lane's 16 bytes are inside or outside as a whole
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) { x0[i] = z; w0[i] = z; }
    g0 = z;
    if (whole + l4 * 4 < a.K) load(x0, w0, g0, whole);
    compute(x0, w0, g0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (NORM) {                                         // the four lane groups hold different k of the same token
      ss[i] += __shfl_xor(ss[i], 16, kWave);
      ss[i] += __shfl_xor(ss[i], 32, kWave);
    }
    const int m = m0 + i * 16 + l16;
    if (m >= a.M) continue;
    f32_store<EPI, NORM>(a, cols[0], m, l4, acc[i][0], acc[i][1], ss[i]);
    if (n_tiles == 2) f32_store<EPI, NORM>(a, cols[1], m, l4, acc[i][2], acc[i][3], ss[i]);
  }
}

// One tile of 32 x 32 per workgroup, KS waves sharing its K.
template <int EPI, int KS, bool NORM>
__global__ __launch_bounds__(64 * KS) void k_gemm_f32(F32GemmArgs a) {
  constexpr int U = 4;                                  // chunks requested together: 16 loads of 16 bytes in flight
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m0 = (int)blockIdx.y * 32, tile = blockIdx.x;
  const F32Cols cols = f32_cols<EPI>(a, tile);
  const float *wp[2], *xp[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) wp[j] = f32_weights<EPI>(a, cols, j, l16, l4);
#pragma unroll
  for (int i = 0; i < 2; ++i) xp[i] = f32_input(a, m0 + i * 16 + l16, l4);
  const float* gp = NORM ? a.g + l4 * 4 : nullptr;

  f32x4_t acc[2][2];                                    // [token block][weight block]: rows = features, column = token
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss[2] = {0.f, 0.f};
  const int chunks = (a.K + 15) / 16;
  for (int c0 = wave; c0 < chunks; c0 += U * KS) {
    f32x4_t xf[U][2], wf[U][2], gf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u * KS) * 16;                 // K is a multiple of 4: a lane's 16 bytes are inside or outside as a whole
      const bool in = k + l4 * 4 < a.K;
      const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 2; ++i) xf[u][i] = in ? *(const f32x4_t*)(xp[i] + k) : z;
#pragma unroll
      for (int j = 0; j < 2; ++j) wf[u][j] = in ? *(const f32x4_t*)(wp[j] + k) : z;
      if (NORM) gf[u] = in ? *(const f32x4_t*)(gp + k) : z;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((c0 + u * KS) * 16 >= a.K) break;             // uniform
      if (NORM) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ss[i] = fmaf(xf[u][i][e], xf[u][i][e], ss[i]);
            xf[u][i][e] *= gf[u][e];
          }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[u][j][e], xf[u][i][e], acc[i][j], 0, 0, 0);
    }
  }
  if (NORM) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {                       // the four lane groups hold different k of the same token
      ss[i] += __shfl_xor(ss[i], 16, kWave);
      ss[i] += __shfl_xor(ss[i], 32, kWave);
    }
  }
  __shared__ f32x4_t red[KS][4][64];
  __shared__ float red_ss[KS][2][16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) red[wave][i * 2 + j][lane] = acc[i][j];
  if (NORM && l4 == 0) { red_ss[wave][0][l16] = ss[0]; red_ss[wave][1][l16] = ss[1]; }
  __syncthreads();
  if (wave >= 2) return;
  const int m = m0 + wave * 16 + l16;                   // wave w finishes token block w
  f32x4_t v[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    v[j] = red[0][wave * 2 + j][lane];
#pragma unroll
    for (int w = 1; w < KS; ++w) v[j] = v[j] + red[w][wave * 2 + j][lane];
  }
  float t = 0.f;
  if (NORM) {
    t = red_ss[0][wave][l16];
#pragma unroll
    for (int w = 1; w < KS; ++w) t += red_ss[w][wave][l16];
  }
  if (m < a.M) f32_store<EPI, NORM>(a, cols, m, l4, v[0], v[1], t);
}

// Sizes: 32-row tiles are counted by the grid's y, a tile lies in one segment.
bool f32_linear_takes(int64_t m, const int* seg_rows, int n_seg, int k) {
  for (int i = 0; i < n_seg; ++i)
    if (n_seg > 1 && seg_rows[i] % 32) return false;
  return k % 4 == 0 && m >= 1 && ceil_div(m, 32) <= 65535;
}
bool f32_linear_aligned(const void* x, const void* const* w, int n_seg, const void* w2) {
  uintptr_t all = (uintptr_t)x | (uintptr_t)w2;
  for (int i = 0; i < n_seg; ++i) all |= (uintptr_t)w[i];
  return all % 16 == 0;
}

// The rule (us; K = 256 / 1024 / 4096).  8 or 4 waves on a tile: 256 tiles 7.1 / 14.7 / 46 against 7.4 / 15.3 / 40, 512 tiles
// 9.0 / 25.6 / 91 against 9.3 / 26.1 / 85, 1024 tiles 14.8 / 48.7 / 178 against 14.3 / 46.6 / 172.  4 waves on a tile or waves of
// 64 x 64: 1536 tiles 20 / 70 / 257 against 24 / 79 / 288, 2048 tiles 25 / 93 / 346 against 25 / 79 / 287, 4096 tiles 46 / 184 / 705
// against 28 / 82 / 305.
template <int EPI, bool NORM>
static void launch_f32_t(const F32GemmArgs& a, hipStream_t s) {
  const int64_t tm = ceil_div(a.M, 32), tiles = tm * a.tiles_n;
  if (tiles >= 2048)
    hipLaunchKernelGGL((k_gemm_f32_wide<EPI, NORM>), dim3((unsigned)ceil_div(a.tiles_n, 4), (unsigned)ceil_div(tm, 4)), dim3(256), 0, s, a);
  else if (tiles >= 512)
    hipLaunchKernelGGL((k_gemm_f32<EPI, 4, NORM>), dim3((unsigned)a.tiles_n, (unsigned)tm), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_gemm_f32<EPI, 8, NORM>), dim3((unsigned)a.tiles_n, (unsigned)tm), dim3(512), 0, s, a);
}

// c / ldc per segment; norm_g: the input rows are RMS-normalised (x then is the fp32 residual); rope: as RopeFuse says
fastav_status_t launch_linear_f32(const float* x, const int32_t* rows, const void* const* w_seg, const int* seg_rows, int n_seg,
                                  const void* w2, float* const* c, const int64_t* ldc, int64_t m, int k, int epilogue,
                                  const float* norm_g, float eps, const RopeFuse* rope, hipStream_t s) {
  if (!f32_linear_takes(m, seg_rows, n_seg, k) || !f32_linear_aligned(x, w_seg, n_seg, w2)) return fail(FASTAV_EUNSUPPORTED, "f32 linear: unsupported shape or alignment");
  if (norm_g && (epilogue == FASTAV_EPI_RESADD || (uintptr_t)norm_g % 16)) return fail(FASTAV_EINVAL, "f32 linear: bad fused-norm arguments");
  F32GemmArgs a;
  a.x = x; a.rows = rows; a.w2 = (const float*)w2; a.M = (int)m; a.K = k; a.g = norm_g; a.eps = eps;
  int n = 0;
  a.rope_pos = nullptr; a.rope_tab = nullptr; a.dh = 0; a.rope_cols = 0;
  for (int i = 0; i < 3; ++i) {
    const int at = i < n_seg ? i : 0;
    if (i < n_seg) n += seg_rows[i];
    a.w[i] = (const float*)w_seg[at]; a.c[i] = c[at]; a.ldc[i] = ldc[at];
    a.seg_end[i] = i < n_seg ? n : 0x7FFFFFFF;
    if (rope && i == rope->n_segs - 1) a.rope_cols = n;
  }
  if (rope) {
    if (epilogue != FASTAV_EPI_STORE || (rope->head_dim != 64 && rope->head_dim != 128) || rope->n_segs < 1 || rope->n_segs > n_seg || n_seg < 2)
      return fail(FASTAV_EINVAL, "f32 linear: this product cannot take the RoPE epilogue");
    for (int i = 0; i < rope->n_segs; ++i)
      if (seg_rows[i] % rope->head_dim) return fail(FASTAV_EINVAL, "f32 linear: RoPE needs whole heads");
    a.rope_pos = rope->pos; a.rope_tab = (const float2*)rope->table; a.dh = rope->head_dim;
  }
  a.N = n;
  a.tiles_n = (int)ceil_div(n, epilogue == FASTAV_EPI_SWIGLU ? 16 : 32);
  if (epilogue == FASTAV_EPI_SWIGLU) { if (norm_g) launch_f32_t<FASTAV_EPI_SWIGLU, true>(a, s); else launch_f32_t<FASTAV_EPI_SWIGLU, false>(a, s); }
  else if (epilogue == FASTAV_EPI_RESADD) launch_f32_t<FASTAV_EPI_RESADD, false>(a, s);
  else { if (norm_g) launch_f32_t<FASTAV_EPI_STORE, true>(a, s); else launch_f32_t<FASTAV_EPI_STORE, false>(a, s); }
  return check_launch("linear_f32");
}

}  // namespace fastav
