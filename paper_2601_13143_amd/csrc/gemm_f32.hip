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
// Which waves make a workgroup (chosen by the launcher from the number of 32 x 32 tiles):
//   2 x 2 tiles, one wave each         when the tiles alone give every SIMD two waves (>= 2048 tiles);
//   one tile, 4 or 8 waves splitting K otherwise (a prompt of a few hundred tokens through a small model: 64-256
//                                      tiles); the partial tiles are summed through LDS in wave order.
// One fp32 prompt of 512 tokens (hidden 256, mlp 688): 36-88 us per product on the vector ALUs, where a workgroup
// walked K alone with its staging in the open, against 6-12 us here (launch, one or two trips to L2, the sum).
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

template <int EPI, int WM, int WN, int KS, bool NORM>
__global__ __launch_bounds__(64 * WM * WN * KS) void k_gemm_f32(F32GemmArgs a) {
  static_assert(KS == 1 || (WM == 1 && WN == 1), "waves share a tile or have one each");
  constexpr int U = 4;                                  // chunks requested together: 16 loads of 16 bytes in flight
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ks = wave % KS, wm = (wave / KS) % WM, wn = wave / (KS * WM);
  const int m0 = ((int)blockIdx.y * WM + wm) * 32;
  const int tile = (int)blockIdx.x * WN + wn;
  if (KS == 1 && (m0 >= a.M || tile >= a.tiles_n)) return;        // no barrier in this form

  // the two 16-row weight blocks and the output column each starts at (inside its segment)
  int seg = 0, seg0 = 0;
  int n0 = EPI == FASTAV_EPI_SWIGLU ? tile * 16 : tile * 32;
  if (EPI != FASTAV_EPI_SWIGLU) {
    if (n0 >= a.seg_end[0]) { seg = 1; seg0 = a.seg_end[0]; }
    if (n0 >= a.seg_end[1]) { seg = 2; seg0 = a.seg_end[1]; }
  }
  const bool rope = EPI == FASTAV_EPI_STORE && a.rope_tab != nullptr && n0 < a.rope_cols;
  int nb[2] = {n0 - seg0, n0 - seg0 + 16};
  int f0 = 0;                                           // rope: frequency index of the block's first column
  if (rope) {
    const int per_head = a.dh / 32, t = (n0 - seg0) / 32;
    f0 = (t % per_head) * 16;
    nb[0] = (t / per_head) * a.dh + f0;
    nb[1] = nb[0] + a.dh / 2;
  }
  const int n_seg = (EPI == FASTAV_EPI_SWIGLU) ? a.N : (a.seg_end[seg] < a.N ? a.seg_end[seg] : a.N) - seg0;
  const float* wp[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (EPI == FASTAV_EPI_SWIGLU) {
      const int n = nb[0] + l16 < n_seg ? nb[0] + l16 : n_seg - 1;        // clamped rows are masked at the store
      wp[j] = (j ? a.w2 : a.w[0]) + (int64_t)n * a.K + l4 * 4;
    } else {
      const int n = nb[j] + l16 < n_seg ? nb[j] + l16 : n_seg - 1;
      wp[j] = a.w[seg] + (int64_t)n * a.K + l4 * 4;
    }
  }
  const float* xp[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int m = m0 + i * 16 + l16;
    m = m < a.M ? m : a.M - 1;
    xp[i] = a.x + (int64_t)(a.rows ? a.rows[m] : m) * a.K + l4 * 4;
  }
  const float* gp = NORM ? a.g + l4 * 4 : nullptr;

  f32x4_t acc[2][2];                                    // [token block][weight block]: rows = features, column = token
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss[2] = {0.f, 0.f};
  const int chunks = (a.K + 15) / 16;
  for (int c0 = ks; c0 < chunks; c0 += U * KS) {
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
  int i_lo = 0, i_hi = 2;
  if constexpr (KS > 1) {
    __shared__ f32x4_t red[KS][4][64];
    __shared__ float red_ss[KS][2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) red[wave][i * 2 + j][lane] = acc[i][j];
    if (NORM && l4 == 0) { red_ss[wave][0][l16] = ss[0]; red_ss[wave][1][l16] = ss[1]; }
    __syncthreads();
    if (wave >= 2) return;
    i_lo = wave; i_hi = wave + 1;                       // wave w finishes token block w
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      f32x4_t s = red[0][i_lo * 2 + j][lane];
#pragma unroll
      for (int w = 1; w < KS; ++w) s = s + red[w][i_lo * 2 + j][lane];
      acc[0][j] = s; acc[1][j] = s;
    }
    if (NORM) {
      float t = red_ss[0][i_lo][l16];
#pragma unroll
      for (int w = 1; w < KS; ++w) t += red_ss[w][i_lo][l16];
      ss[0] = t; ss[1] = t;
    }
  }

  // accumulator element r: feature block column l4 * 4 + r, token l16
  float* const cb = a.c[seg];
  const int64_t ldc = a.ldc[seg];
  const bool vec = ldc % 4 == 0 && ((uintptr_t)cb % 16) == 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (i < i_lo || i >= i_hi) continue;
    const int m = m0 + i * 16 + l16;
    if (m >= a.M) continue;
    f32x4_t v[2] = {acc[i][0], acc[i][1]};
    if (NORM) {
      const float r = 1.0f / sqrtf(ss[i] / (float)a.K + a.eps);
      v[0] = v[0] * r; v[1] = v[1] * r;
    }
    if (rope) {
      const float2* tr = a.rope_tab + (int64_t)a.rope_pos[m] * (a.dh / 2) + f0 + l4 * 4;
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
#pragma unroll
    for (int j = 0; j < (EPI == FASTAV_EPI_SWIGLU ? 1 : 2); ++j) {
      const int n = nb[j] + l4 * 4;
      float* p = cb + (int64_t)m * ldc + n;
      if (vec && n + 3 < n_seg) {
        if (EPI == FASTAV_EPI_RESADD) v[j] = v[j] + *(const f32x4_t*)p;
        *(f32x4_t*)p = v[j];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n + r < n_seg) p[r] = (EPI == FASTAV_EPI_RESADD) ? p[r] + v[j][r] : v[j][r];
      }
    }
  }
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

template <int EPI, bool NORM>
static void launch_f32_t(const F32GemmArgs& a, hipStream_t s) {
  const int64_t tm = ceil_div(a.M, 32), tiles = tm * a.tiles_n;
  if (tiles >= 2048) {
    const dim3 grid((unsigned)ceil_div(a.tiles_n, 2), (unsigned)ceil_div(tm, 2));
    hipLaunchKernelGGL((k_gemm_f32<EPI, 2, 2, 1, NORM>), grid, dim3(256), 0, s, a);
  } else if (tiles >= 512) {
    hipLaunchKernelGGL((k_gemm_f32<EPI, 1, 1, 4, NORM>), dim3((unsigned)a.tiles_n, (unsigned)tm), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_gemm_f32<EPI, 1, 1, 8, NORM>), dim3((unsigned)a.tiles_n, (unsigned)tm), dim3(512), 0, s, a);
  }
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
