// One decode step on the per-layer K/V caches a pruned prefill leaves behind (Section 3.1: the paper's
// latency is the time to generate a single token, its memory saving the compacted caches).
//
// A decode step for a handful of samples is bound by streaming the weights (7B: 13 GB per step) and, far
// behind, the caches.  Two kernel families:
//
//   k_gemv_rows       one sample: a wave owns two weight rows, the input row sits in LDS.
//   k_skinny_resident, k_skinny_stream
//                     2-16 samples: weights from global memory straight into matrix-core operand layout, the batch as
//                     the other operand, partial sums of the waves through LDS.
//   Both fold in RMSNorm, RoPE and the append to the generated-token caches.
//
//   k_decode_attn    single-query grouped-query attention over [cache prefix | generated so far | the new
//                    token itself] for one (sample, KV head, key split): logits of all heads of the group on
//                    the matrix cores with the keys read from global memory in operand layout, P V on the
//                    vector units straight from the V rows.  k_decode_merge combines the splits' (max, sum, o).
#include "common.hpp"

namespace fastav {

typedef float f32x4v __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS traffic only: global loads already issued stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------------------- skinny linear
struct SkinnyArgs {
  const bf16_t* x;            // [B, K] bf16
  const bf16_t* w[3];         // up to three [rows, K] matrices stacked along the output dimension (Q | K | V)
  int seg_end[3];             // exclusive end row of each segment
  const bf16_t* w2;           // "up" matrix (SwiGLU only), same shape as w[0]
  void* y;                    // store / SwiGLU: bf16 [B, ldy]; residual: fp32 [B, ldy]
  int64_t ldy;
  int B, N, K;
  // one-row GEMV, NORM: the input is the fp32 residual stream, RMS-normalised by every workgroup for itself
  const float* xres;          // [B, K] fp32
  const bf16_t* g;            // [K] gain
  float eps;
  // matrix-core kernels, optional: x holds bf16(residual * gain) and the product is scaled with 1 / rms of its row, from
  // the row's sums of squares over 16 columns each, ss_in [K / 16][16] (the same one rounding of the input as normalising
  // first).  The residual epilogue can write both for the projection that comes next: xg_out = bf16(y * g_out) and ss_out.
  const float* ss_in;
  const bf16_t* g_out;
  bf16_t* xg_out;
  float* ss_out;              // [N / 16][16]
  // store epilogue, optional: output features below rope_rows are heads of dh features each, rotated before they are
  // stored (rotate-half pairs (i, i + dh/2)).  The one-row GEMV evaluates the angle itself (position pos[0], angle
  // pos * base^(-2i/dh)); the matrix-core kernels read rope_tab [B][dh/2] = (cos, sin) of every row's position.
  const int32_t* pos;
  const float2* rope_tab;
  int rope_rows, dh;
  double rope_coef;           // -log2(base) * 2 / dh
  // store epilogue, optional: features [app_k0, app_v0) also go to app_k + b * app_stride, those from app_v0 on to app_v:
  // the step's own key and value land in the generated-token cache without a copy launch
  bf16_t *app_k, *app_v;
  int64_t app_stride;
  int app_k0, app_v0;
};

__device__ __forceinline__ bf16_t* skinny_append_row(const SkinnyArgs& a, int b, int n) {
  if (a.app_k == nullptr || n < a.app_k0) return nullptr;
  return n < a.app_v0 ? a.app_k + b * a.app_stride + (n - a.app_k0) : a.app_v + b * a.app_stride + (n - a.app_v0);
}

// Y[b, n] = sum_k X[b, k] W[n, k] for 1 <= b <= 16 on v_mfma_f32_16x16x32_bf16, laid out for the weight stream.
//
// An item is two groups of 8 output features: neighbours; the rotation pair of a head where RoPE is fused; a gate and
// an up group for SwiGLU.  A weight load instruction covers 8 features x 128 contiguous bytes (whole lines): operand
// rows 0-7 are the features at the first 32 k of a 64-k block, rows 8-15 the same features at the second 32.  Two
// matrix instructions, one per half of the block's input, then leave the product in rows 0-7 of the first accumulator
// and rows 8-15 of the second; the other halves are discarded (the matrix cores have nothing else to do).  The eight
// waves of a workgroup take the 64-k blocks of K in turn, so that together they read 1 KB runs of a row, and their
// partial sums meet in LDS in wave order.
constexpr int kSkinnyWaves = 8;

template <bool PLAIN>
__device__ __forceinline__ void skinny_item(const SkinnyArgs& a, int epi, int item, int& n0, int& dn) {
  if (epi == FASTAV_EPI_SWIGLU) { n0 = item * 8; dn = 0; return; }
  if (!PLAIN && a.rope_rows > 0) {
    const int per_head = a.dh / 16;
    n0 = (item / per_head) * a.dh + (item % per_head) * 8;
    dn = a.dh / 2;
  } else {
    n0 = item * 16;
    dn = 8;
  }
}

// First weight elements of the item's two groups (both lie in one segment).  The segments' pointers are made values before
// one is chosen: left to the compiler the chosen one is loaded behind the comparisons, those behind the choice of rotated
// heads, and the first weight load waits for three trips to the constant cache (8 rows, 1024 x 1024 4.19 -> 3.95 us, 4096 x
// 4096 9.4 -> 9.1).  PLAIN: no segment has rotated heads.
template <int EPI, bool PLAIN = false>
__device__ __forceinline__ void skinny_rows(const SkinnyArgs& a, int item, const bf16_t*& p0, const bf16_t*& p1) {
  const bf16_t *w0 = a.w[0], *w1 = EPI == FASTAV_EPI_SWIGLU ? a.w2 : a.w[1], *w2 = a.w[2];
  int end0 = a.seg_end[0], end1 = a.seg_end[1];
  asm volatile("" : "+s"(w0), "+s"(w1) : "s"(a.x), "s"(a.y), "s"(a.B), "s"(a.K));
  if (EPI != FASTAV_EPI_SWIGLU) asm volatile("" : "+s"(w2), "+s"(end0), "+s"(end1) : "s"(a.rope_rows), "s"(a.dh));
  int n0, dn;
  skinny_item<PLAIN>(a, EPI, item, n0, dn);
  int seg0 = 0;
  p0 = w0;
  if (EPI != FASTAV_EPI_SWIGLU) {
    if (n0 >= end0) { p0 = w1; seg0 = end0; }
    if (n0 >= end1) { p0 = w2; seg0 = end1; }
  }
  p0 += (int64_t)(n0 - seg0) * a.K;
  p1 = EPI == FASTAV_EPI_SWIGLU ? w1 + (int64_t)n0 * a.K : p0 + (int64_t)dn * a.K;
}

// The sums of one item: v0, v1 = features n + f4 .. + 3 of the two groups, batch row b (lanes 0-31; the others hold copies).
template <int EPI, bool PLAIN = false>
__device__ __forceinline__ void skinny_finish(const SkinnyArgs& a, int item, int lane, f32x4v v0, f32x4v v1, f32x4v y0, f32x4v y1) {
  int n0, dn;
  skinny_item<PLAIN>(a, EPI, item, n0, dn);
  const int b = lane & 15, f4 = ((lane >> 4) & 1) * 4;
  if (lane >= 32 || b >= a.B) return;
  const int n = n0 + f4;
  if (EPI == FASTAV_EPI_RESADD) {
    float* y = (float*)a.y + (int64_t)b * a.ldy + n;
    y0 = y0 + v0;
    y1 = y1 + v1;
    *(f32x4v*)y = y0;
    *(f32x4v*)(y + dn) = y1;
    if (PLAIN || a.xg_out == nullptr) return;
    const bf16x4_t g0 = *(const bf16x4_t*)(a.g_out + n), g1 = *(const bf16x4_t*)(a.g_out + n + dn);
    bf16x4_t o0, o1;
    float ss = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      o0[r] = (bf16_t)(y0[r] * (float)g0[r]);
      o1[r] = (bf16_t)(y1[r] * (float)g1[r]);
      ss = fmaf(y0[r], y0[r], fmaf(y1[r], y1[r], ss));
    }
    *(bf16x4_t*)(a.xg_out + (int64_t)b * a.N + n) = o0;
    *(bf16x4_t*)(a.xg_out + (int64_t)b * a.N + n + dn) = o1;
    ss += __shfl_xor(ss, 16, kWave);                          // lanes b and b + 16 are both here
    if (lane < 16) a.ss_out[item * 16 + b] = ss;
    return;
  }
  bf16_t* y = (bf16_t*)a.y + (int64_t)b * a.ldy + n;
  bf16x4_t o0, o1;
  if (EPI == FASTAV_EPI_SWIGLU) {
#pragma unroll
    for (int r = 0; r < 4; ++r) o0[r] = (bf16_t)(v0[r] / (1.0f + __expf(-v0[r])) * v1[r]);
    *(bf16x4_t*)y = o0;
    return;
  }
  if (!PLAIN && n0 < a.rope_rows) {
    const f32x4v* t = (const f32x4v*)(a.rope_tab + b * (a.dh / 2) + n0 % a.dh + f4);
    const f32x4v t0 = t[0], t1 = t[1];
    const float cs[4] = {t0[0], t0[2], t1[0], t1[2]}, sn[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float lo = v0[r], hi = v1[r];
      v0[r] = lo * cs[r] - hi * sn[r];
      v1[r] = hi * cs[r] + lo * sn[r];
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) { o0[r] = (bf16_t)v0[r]; o1[r] = (bf16_t)v1[r]; }
  *(bf16x4_t*)y = o0;
  *(bf16x4_t*)(y + dn) = o1;
  if (PLAIN) return;
  if (bf16_t* p = skinny_append_row(a, b, n)) {              // both groups lie in one segment
    *(bf16x4_t*)p = o0;
    *(bf16x4_t*)(p + dn) = o1;
  }
}

// Buffer loads: base in scalar registers, one lane offset for all of a wave's loads and a scalar offset per block - with
// 64-bit lane addresses the loads in flight do not fit the registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t skinny_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, 0x00020000);
}
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
constexpr uint32_t kSkinnyOutside = 0x80000000u;            // a lane offset beyond every resource: such a load returns zero
template <typename T>
__device__ __forceinline__ T skinny_load(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
}

// Sum of the waves' partials of one group, in wave order: lanes 0-31 add the first halves, 32-63 the second.
__device__ __forceinline__ f32x4v skinny_halves(f32x4v s) {
#pragma unroll
  for (int r = 0; r < 4; ++r) s[r] += __shfl_xor(s[r], 32, kWave);
  return s;
}
__device__ __forceinline__ f32x4v skinny_sum(const f32x4v (*red)[64], int lane) {
  f32x4v s = red[0][lane];
#pragma unroll
  for (int w = 1; w < kSkinnyWaves; ++w) s = s + red[w][lane];
  return skinny_halves(s);
}
// Two groups, all reads asked for before the first addition: where a workgroup ends with its sum, two or three reads in
// flight make that a chain of LDS latencies (8 rows, 512 x 512 2.99 -> 2.89 us, 4096 x 4096 9.12 -> 9.02).
__device__ __forceinline__ void skinny_last_sums(const f32x4v (*red)[kSkinnyWaves][64], int lane, f32x4v& v0, f32x4v& v1) {
  f32x4v p[2][kSkinnyWaves];
#pragma unroll
  for (int w = 0; w < kSkinnyWaves; ++w) {
    p[0][w] = red[0][w][lane];
    p[1][w] = red[1][w][lane];
  }
  __builtin_amdgcn_sched_barrier(0);
  v0 = p[0][0];
  v1 = p[1][0];
#pragma unroll
  for (int w = 1; w < kSkinnyWaves; ++w) {
    v0 = v0 + p[0][w];
    v1 = v1 + p[1][w];
  }
  v0 = skinny_halves(v0);
  v1 = skinny_halves(v1);
}

// 1 / rms of every row from the sums of squares ss_in, into rs[16]; the caller's next barrier publishes it.  Thread =
// (row, one of 32 column ranges), partial sums in range order.
__device__ __forceinline__ void skinny_rms_part(const SkinnyArgs& a, int tid, float (*part)[16]) {
  constexpr int R = 4 * kSkinnyWaves, U = 8;                  // U loads at a time: one after the other each waits for its own
  const int b = tid & 15, q = tid >> 4, n = a.K / 16;
  float t = 0.f;
  for (int i = q; i < n; i += R * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i + R * u < n && b < a.B ? a.ss_in[(i + R * u) * 16 + b] : 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) t += v[u];
  }
  part[q][b] = t;
}
template <bool AHEAD>
__device__ __forceinline__ float skinny_rms(const SkinnyArgs& a, int b, const float (*part)[16]) {
  float p[4 * kSkinnyWaves], t = 0.f;
#pragma unroll
  for (int q = 0; q < 4 * kSkinnyWaves; ++q) p[q] = part[q][b];
  if (AHEAD) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 4 * kSkinnyWaves; ++q) t += p[q];
  return 1.0f / sqrtf(t / (float)a.K + a.eps);
}

// K <= 4096, store and SwiGLU epilogues: a workgroup stays on its CU, keeps the batch as matrix operands in registers
// (NB 64-k blocks per wave, read once) and walks the items blockIdx, + gridDim, ... with two items' weights in flight
// (128 KB each for K = 4096).
// Bound: the weight stream.  Before, every workgroup of 16 features normalised the batch into 64 KB of LDS (one
// workgroup per CU): gate/up of 14336 x 4096 at 8 rows 86 us = 2.7 TB/s, now 44 us = 5.3 TB/s; Q|K|V of 6144 x 4096 with
// its rotation and cache rows 31 + 6 + 9 us -> 16 us.
template <int EPI, int NB>
__global__ __launch_bounds__(64 * kSkinnyWaves) void k_skinny_resident(SkinnyArgs a, int items) {
  __shared__ f32x4v red[2][2][kSkinnyWaves][64];
  __shared__ float ss[4 * kSkinnyWaves][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb = a.K / 64, G = gridDim.x;
  const int b = (lane & 15) < a.B ? (lane & 15) : a.B - 1;    // padded batch rows repeat the last real one
  const int kq = (lane >> 4) * 8;
  const uint32_t woff = ((uint32_t)(lane & 7) * (uint32_t)a.K + ((lane >> 3) & 1) * 32 + kq) * 2;
  const uint32_t wbytes = 16u * (uint32_t)a.K;                // a group's 8 rows
  const __amdgpu_buffer_rsrc_t rx = skinny_rsrc(a.x, (uint32_t)(a.B * a.K) * 2u);
  const uint32_t xoff = (uint32_t)(b * a.K + kq) * 2u;

  auto load = [&](bf16x8_t (&w)[2][NB], int item) __attribute__((always_inline)) {
    const bf16_t *p0, *p1;
    skinny_rows<EPI>(a, item, p0, p1);
    const __amdgpu_buffer_rsrc_t r0 = skinny_rsrc(p0, wbytes), r1 = skinny_rsrc(p1, wbytes);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int blk = wave + kSkinnyWaves * j;                // past the end both operands are zero: an infinite weight of
      const uint32_t off = blk < kb ? woff : kSkinnyOutside;  // the last block must not meet a zero input
      w[0][j] = skinny_load<bf16x8_t>(r0, off, blk < kb ? blk * 128 : 0);
      w[1][j] = skinny_load<bf16x8_t>(r1, off, blk < kb ? blk * 128 : 0);
    }
  };
  bf16x8_t xf[NB][2], w0[2][NB], w1[2][NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int blk = wave + kSkinnyWaves * j;
#pragma unroll
    for (int h = 0; h < 2; ++h) xf[j][h] = skinny_load<bf16x8_t>(rx, blk < kb ? xoff + h * 64 : kSkinnyOutside, blk < kb ? blk * 128 : 0);
  }
  const int it0 = blockIdx.x;
  load(w0, it0);
  load(w1, it0 + G < items ? it0 + G : it0);
  if (a.ss_in != nullptr) skinny_rms_part(a, tid, ss);        // published by the first item's barrier

  int n_done = 0;
  auto compute = [&](bf16x8_t (&w)[2][NB], int item) __attribute__((always_inline)) {
    f32x4v a00 = {0.f, 0.f, 0.f, 0.f}, a01 = a00, a10 = a00, a11 = a00;   // [group][half]
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      a00 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0][j], xf[j][0], a00, 0, 0, 0);
      a01 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0][j], xf[j][1], a01, 0, 0, 0);
      a10 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1][j], xf[j][0], a10, 0, 0, 0);
      a11 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1][j], xf[j][1], a11, 0, 0, 0);
    }
    const int buf = n_done & 1;
    red[buf][0][wave][lane] = lane < 32 ? a00 : a01;
    red[buf][1][wave][lane] = lane < 32 ? a10 : a11;
    lds_barrier();                                            // two buffers: item i + 2 rewrites one behind item i + 1's barrier
    if (wave == (n_done & (kSkinnyWaves - 1))) {
      f32x4v v0 = skinny_sum(red[buf][0], lane), v1 = skinny_sum(red[buf][1], lane);
      if (a.ss_in != nullptr) {
        const float r = skinny_rms<false>(a, lane & 15, ss);
        v0 = v0 * r;
        v1 = v1 * r;
      }
      const f32x4v z = {0.f, 0.f, 0.f, 0.f};
      skinny_finish<EPI>(a, item, lane, v0, v1, z, z);
    }
    ++n_done;
  };
  int it = it0;
  for (; it + 3 * G < items; it += 2 * G) {
    compute(w0, it);
    load(w0, it + 2 * G);
    compute(w1, it + G);
    load(w1, it + 3 * G);
  }
  if (it + 2 * G < items) {
    compute(w0, it);
    load(w0, it + 2 * G);
    compute(w1, it + G);
    compute(w0, it + 2 * G);
  } else {
    compute(w0, it);
    if (it + G < items) compute(w1, it + G);
  }
}

// Any K, any epilogue, bf16 input: P items per workgroup; a wave walks its 64-k blocks C at a time with three such chunks of
// weights and input operands in flight (96 KB of weights per workgroup; the input comes from L2, once for all P items).
// The O and down projections' kernel, and that of smaller products: few items leave nothing to keep the batch resident for.  Eight rows:
// down of 4096 x 14336 33 -> 27 us = 4.4 TB/s against batches of 16 loads with a serial remainder, O of 4096 x 4096 10.2 -> 9.0.
// The stream carries nothing but what is needed, in order: loads past the end that repeat the last block cost down 5 us and
// O of 1024 x 1024 7 of 11; a load behind a run-time test makes the compiler wait for its registers.
// BRIEF: K <= 2048 and nothing folded in.  Such a product ends in 2-6 us, and code that is only jumped over and blocks that
// are only requested to read as zero show: 8 rows of 512 x 512 2.89 -> 2.61 us, of 768 x 1152 3.58 -> 3.44.
template <int EPI, int P, bool BRIEF>
__global__ __launch_bounds__(64 * kSkinnyWaves) void k_skinny_stream(SkinnyArgs a) {
  constexpr int C = 2 / P, NG = 2 * P;                        // blocks per chunk, groups of 8 weight rows
  __shared__ f32x4v red[NG][kSkinnyWaves][64];
  __shared__ float ss[EPI == FASTAV_EPI_RESADD ? 1 : 4 * kSkinnyWaves][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb = a.K / 64, item0 = blockIdx.x * P;
  const int b = (lane & 15) < a.B ? (lane & 15) : a.B - 1;
  const int kq = (lane >> 4) * 8;
  const uint32_t woff = ((uint32_t)(lane & 7) * (uint32_t)a.K + ((lane >> 3) & 1) * 32 + kq) * 2, xoff = (uint32_t)(b * a.K + kq) * 2;
  __amdgpu_buffer_rsrc_t r[NG];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const bf16_t *p0, *p1;
    skinny_rows<EPI, BRIEF>(a, item0 + p, p0, p1);
    r[2 * p] = skinny_rsrc(p0, 16u * (uint32_t)a.K);
    r[2 * p + 1] = skinny_rsrc(p1, 16u * (uint32_t)a.K);
  }
  const __amdgpu_buffer_rsrc_t rx = skinny_rsrc(a.x, (uint32_t)(a.B * a.K) * 2u);
  f32x4v y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
  static_assert(EPI != FASTAV_EPI_RESADD || P == 1, "the residual of one item is held");
  if (EPI == FASTAV_EPI_RESADD && wave == 0) {                // ahead of the stream: not waited for until the end
    const float* y = (const float*)a.y + (int64_t)b * a.ldy + item0 * 16 + ((lane >> 4) & 1) * 4;
    y0 = *(const f32x4v*)y;
    y1 = *(const f32x4v*)(y + 8);
  }
  // as 32-bit words: vectors of 16-bit elements that meet behind a branch are rebuilt from halves, which waits for them
  u32x4v w0[NG][C], w1[NG][C], w2[NG][C], x0[C][2], x1[C][2], x2[C][2];
  // n of a chunk's blocks, a number known at compile time.  Blocks past the end exist in the last chunk only: their lane
  // offset lies outside every resource, so they read as zero and touch no memory.
  auto load = [&](u32x4v (&w)[NG][C], u32x4v (&x)[C][2], int ch, bool last, int n = 2 / P) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < C && u < n; ++u) {
      const int blk = wave + kSkinnyWaves * (ch * C + u);
      const bool in = !last || blk < kb;
      const uint32_t off = in ? (uint32_t)blk * 128u : 0u, wl = in ? woff : kSkinnyOutside, xl = in ? xoff : kSkinnyOutside;
#pragma unroll
      for (int g = 0; g < NG; ++g) w[g][u] = skinny_load<u32x4v>(r[g], wl, off);
      x[u][0] = skinny_load<u32x4v>(rx, xl, off);
      x[u][1] = skinny_load<u32x4v>(rx, xl + 64, off);
    }
    __builtin_amdgcn_sched_barrier(0);                        // requested here, not next to their use
  };
  f32x4v acc[NG][2];                                          // [group][half]
#pragma unroll
  for (int g = 0; g < NG; ++g) acc[g][0] = acc[g][1] = f32x4v{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](u32x4v (&w)[NG][C], u32x4v (&x)[C][2], int n = 2 / P) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < C && u < n; ++u)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const bf16x8_t wv = __builtin_bit_cast(bf16x8_t, w[g][u]);
        acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8_t, x[u][0]), acc[g][0], 0, 0, 0);
        acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8_t, x[u][1]), acc[g][1], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // every end of the walk has a body of its own: a load behind a run-time test inside the stream costs it its depth
  const int nch = (kb + kSkinnyWaves * C - 1) / (kSkinnyWaves * C);
  const bool scaled = !BRIEF && EPI != FASTAV_EPI_RESADD && a.ss_in != nullptr;
  if (!BRIEF && nch >= 3) {
    load(w0, x0, 0, false);
    load(w1, x1, 1, false);
    load(w2, x2, 2, true);
    if (scaled) skinny_rms_part(a, tid, ss);
    int ch = 3;
    for (; ch + 2 < nch; ch += 3) {
      compute(w0, x0);
      load(w0, x0, ch, false);
      compute(w1, x1);
      load(w1, x1, ch + 1, false);
      compute(w2, x2);
      load(w2, x2, ch + 2, true);
    }
    if (ch == nch) {
      compute(w0, x0);
      compute(w1, x1);
      compute(w2, x2);
    } else if (ch + 1 == nch) {
      compute(w0, x0);
      load(w0, x0, ch, true);
      compute(w1, x1);
      compute(w2, x2);
      compute(w0, x0);
    } else {
      compute(w0, x0);
      load(w0, x0, ch, false);
      compute(w1, x1);
      load(w1, x1, ch + 1, true);
      compute(w2, x2);
      compute(w0, x0);
      compute(w1, x1);
    }
  } else if (BRIEF && kb <= kSkinnyWaves) {
    load(w0, x0, 0, true, 1);
    compute(w0, x0, 1);
  } else if (nch == 2) {
    load(w0, x0, 0, false);
    load(w1, x1, 1, true);
    if (scaled) skinny_rms_part(a, tid, ss);
    compute(w0, x0);
    compute(w1, x1);
  } else {
    load(w0, x0, 0, true);
    if (scaled) skinny_rms_part(a, tid, ss);
    compute(w0, x0);
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    f32x4v t;                                                 // by element: a choice between two array elements goes through memory
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = lane < 32 ? acc[g][0][e] : acc[g][1][e];
    red[g][wave][lane] = t;
  }
  lds_barrier();
  if (wave >= P) return;                                      // wave p finishes item p
  f32x4v v0, v1;
  skinny_last_sums(red + 2 * wave, lane, v0, v1);
  if (scaled) {
    const float f = skinny_rms<true>(a, lane & 15, ss);
    v0 = v0 * f;
    v1 = v1 * f;
  }
  skinny_finish<EPI, BRIEF>(a, item0 + wave, lane, v0, v1, y0, y1);
}

// ---------------------------------------------------------------------------------------- one-row GEMV
// Y[n] = sum_k X[k] W[n, k] for a single input row (the paper's latency case: one sample generates one token).
// With one row there is nothing for the matrix cores to reuse, so the kernel is laid out purely for the weight
// stream: a wave owns two consecutive weight rows and reads them as whole 1 KB runs (lane = 16-byte chunk), eight
// to sixteen loads in flight per lane; a workgroup's eight waves cover 16 rows = one contiguous slab.  The input
// row sits in LDS as bf16 (normalised there when NORM, rounded as k_rmsnorm rounds it), each 16-byte chunk of
// it is read once per pair of rows and multiplied with v_dot2_f32_bf16 into fp32 sums, which the wave reduces at
// the end.  K % 512 == 0.
__device__ __forceinline__ float dot8(bf16x8_t w, bf16x8_t x, float acc) {
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 0, 1), __builtin_shufflevector(x, x, 0, 1), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 2, 3), __builtin_shufflevector(x, x, 2, 3), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 4, 5), __builtin_shufflevector(x, x, 4, 5), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 6, 7), __builtin_shufflevector(x, x, 6, 7), acc, false);
  return acc;
}

template <int EPI, bool NORM, bool ROPE>
__global__ __launch_bounds__(512) void k_gemv_rows(SkinnyArgs a) {
  constexpr int NW = 8, NT = 64 * NW;
  constexpr int UB = 4;                                         // chunks per row and batch: 8 or 16 (SwiGLU) loads in flight per lane
  extern __shared__ __attribute__((aligned(16))) bf16_t xs[];   // [K] the input row
  __shared__ float wsum[NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * 16;
  // this wave's two output features: neighbours, or - where the rotation is fused - the pair (i, i + dh/2) of a
  // head, so that the wave holds both halves of the rotation (a workgroup then covers 8 + 8 features of one head)
  const bool rot = ROPE && n0 < a.rope_rows;
  int n_lo = n0 + 2 * wave, dn = 1;
  if (rot) {
    const int wph = a.dh / 16;                                  // workgroups per head
    n_lo = (blockIdx.x / wph) * a.dh + (blockIdx.x % wph) * 8 + wave;
    dn = a.dh / 2;
  }
  const bf16_t* wbase = a.w[0];
  int seg0 = 0;
  if (EPI != FASTAV_EPI_SWIGLU) {                               // both features lie in one segment (whole heads)
    if (n_lo >= a.seg_end[0]) { wbase = a.w[1]; seg0 = a.seg_end[0]; }
    if (n_lo >= a.seg_end[1]) { wbase = a.w[2]; seg0 = a.seg_end[1]; }
  }
  const int cpr = a.K / 8;                                      // 16-byte chunks per row
  const int per_lane = cpr / 64;
  const int64_t row = (int64_t)(n_lo - seg0);                   // this wave's rows: row, row + dn
  const int64_t cdn = (int64_t)dn * cpr;
  const bf16x8_t* w0 = (const bf16x8_t*)(wbase + row * a.K) + lane;
  const bf16x8_t* u0 = (EPI == FASTAV_EPI_SWIGLU) ? (const bf16x8_t*)(a.w2 + row * a.K) + lane : nullptr;
  bf16x8_t f0[UB], f1[UB], g0[UB], g1[UB];
  auto load_batch = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if (c + u < per_lane) {                                   // uniform
        f0[u] = w0[(c + u) * 64];
        f1[u] = w0[(c + u) * 64 + cdn];
        if (EPI == FASTAV_EPI_SWIGLU) { g0[u] = u0[(c + u) * 64]; g1[u] = u0[(c + u) * 64 + cdn]; }
      }
    }
  };
  load_batch(0);                                                // in flight across the prologue (its barriers wait on LDS only)
  float rc = 1.f, rs_ = 0.f;
  if (rot) {                                                    // angle in fp64, as the stand-alone rotation evaluates it
    const double ang = (double)a.pos[0] * exp2((double)(n_lo % a.dh) * a.rope_coef);
    double sd, cd;
    sincos(ang, &sd, &cd);
    rc = (float)cd; rs_ = (float)sd;
  }
  if (NORM) {
    // every thread keeps its quads of the row in registers: the row is read once
    constexpr int R1 = 4;                                       // K <= 4 * R1 * NT = 8192
    const int per_row = a.K / 4;
    f32x4v v[R1];
    bf16x4_t gv[R1];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < R1; ++it) {
      const int i = tid + it * NT;
      if (i < per_row) { v[it] = ((const f32x4v*)a.xres)[i]; gv[it] = ((const bf16x4_t*)a.g)[i]; }
    }
#pragma unroll
    for (int it = 0; it < R1; ++it)
      if (tid + it * NT < per_row) ss += v[it][0] * v[it][0] + v[it][1] * v[it][1] + v[it][2] * v[it][2] + v[it][3] * v[it][3];
    ss = wave_sum(ss);
    if (lane == 0) wsum[wave] = ss;
    lds_barrier();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += wsum[w];                // fixed order: the same value in every thread
    const float r = 1.0f / sqrtf(tot / (float)a.K + a.eps);
#pragma unroll
    for (int it = 0; it < R1; ++it) {
      const int i = tid + it * NT;
      if (i < per_row) {
        bf16x4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16_t)(v[it][e] * r * (float)gv[it][e]);
        ((bf16x4_t*)xs)[i] = o;
      }
    }
  } else {
    for (int i = tid; i < cpr; i += NT) ((bf16x8_t*)xs)[i] = ((const bf16x8_t*)a.x)[i];
  }
  lds_barrier();

  float acc0 = 0.f, acc1 = 0.f, acc0u = 0.f, acc1u = 0.f;
  for (int c = 0; c < per_lane; c += UB) {
    if (c > 0) load_batch(c);
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if (c + u < per_lane) {
        const bf16x8_t xv = ((const bf16x8_t*)xs)[(c + u) * 64 + lane];
        acc0 = dot8(f0[u], xv, acc0);
        acc1 = dot8(f1[u], xv, acc1);
        if (EPI == FASTAV_EPI_SWIGLU) { acc0u = dot8(g0[u], xv, acc0u); acc1u = dot8(g1[u], xv, acc1u); }
      }
    }
  }
  acc0 = wave_sum(acc0);
  acc1 = wave_sum(acc1);
  if (EPI == FASTAV_EPI_SWIGLU) { acc0u = wave_sum(acc0u); acc1u = wave_sum(acc1u); }
  if (lane != 0) return;
  if (EPI == FASTAV_EPI_RESADD) {
    float2* yp = (float2*)((float*)a.y + n_lo);
    float2 y = *yp;
    y.x += acc0; y.y += acc1;
    *yp = y;
  } else if (rot) {
    const bf16_t lo = (bf16_t)(acc0 * rc - acc1 * rs_), hi = (bf16_t)(acc1 * rc + acc0 * rs_);
    ((bf16_t*)a.y)[n_lo] = lo;
    ((bf16_t*)a.y)[n_lo + dn] = hi;
    if (bf16_t* p = skinny_append_row(a, 0, n_lo)) { p[0] = lo; p[dn] = hi; }
  } else {
    if (EPI == FASTAV_EPI_SWIGLU) {
      acc0 = acc0 / (1.0f + __expf(-acc0)) * acc0u;
      acc1 = acc1 / (1.0f + __expf(-acc1)) * acc1u;
    }
    bf16x2_t o;
    o[0] = (bf16_t)acc0; o[1] = (bf16_t)acc1;
    *(bf16x2_t*)((bf16_t*)a.y + n_lo) = o;
    if (EPI == FASTAV_EPI_STORE) {
      if (bf16_t* p = skinny_append_row(a, 0, n_lo)) *(bf16x2_t*)p = o;
    }
  }
}

bool gemv_rows_supported(int B, int n, int k, bool norm) {
  return B == 1 && n % 16 == 0 && k % 512 == 0 && k <= 32768 && (!norm || k <= 8192);
}
// The one-row GEMV can rotate the heads it produces (see SkinnyArgs): the caller then skips the rope launch.
bool gemv_rows_fuses_rope(int B, int n, int k, bool norm, int rope_rows, int dh) {
  return gemv_rows_supported(B, n, k, norm) && dh % 16 == 0 && rope_rows % dh == 0 && rope_rows <= n;
}

bool skinny_linear_supported(int64_t m, int n, int k, int dtype, int64_t ldy) {
  return dtype == FASTAV_BF16 && m >= 1 && m <= 16 && n % 16 == 0 && k % 128 == 0 && ldy % 4 == 0;
}

// norm_x != nullptr (one-row GEMV only): the input is rmsnorm(norm_x [1,k] fp32; gain norm_g, norm_eps) and x is ignored.
// ss_in, next (matrix-core kernels only): see SkinnyArgs.
bool skinny_norm_supported(int B, int k) { return gemv_rows_supported(B, 16, k, true); }

// Whether the store epilogue rotates the leading rope_rows features (whole heads); n must be whole heads too.  The
// one-row GEMV evaluates the angles itself, the matrix-core kernels read a table of the batch (SkinnyRope::table).
static bool skinny_fuses_rope(int B, int n, int k, bool norm, int rope_rows, int dh) {
  if (gemv_rows_supported(B, n, k, norm)) return gemv_rows_fuses_rope(B, n, k, norm, rope_rows, dh);
  return (dh == 64 || dh == 128) && rope_rows % dh == 0 && n % dh == 0 && rope_rows <= n;
}

fastav_status_t launch_skinny_linear(const void* x, const void* const* w_seg, const int* seg_rows, int n_seg,
                                     const void* w2, void* y, int64_t ldy, int B, int n, int k, int epilogue,
                                     hipStream_t s, const float* norm_x, const void* norm_g, float norm_eps,
                                     const SkinnyRope* rope, const SkinnyAppend* app, const float* ss_in, const SkinnyNext* next) {
  if (B == 0 || n == 0) return FASTAV_OK;
  if (rope && (epilogue != FASTAV_EPI_STORE || !rope->pos || !rope->table || (uintptr_t)rope->table % 16 || !skinny_fuses_rope(B, n, k, norm_x != nullptr, rope->rows, rope->head_dim)))
    return fail(FASTAV_EINVAL, "skinny linear: the fused rotation needs the store epilogue and whole heads");
  if (app && (epilogue != FASTAV_EPI_STORE || n_seg != 3 || ((uintptr_t)app->k | (uintptr_t)app->v) % 8 || app->row_stride % 4))
    return fail(FASTAV_EINVAL, "skinny linear: bad cache rows");
  if (!skinny_linear_supported(B, n, k, FASTAV_BF16, ldy)) return fail(FASTAV_EUNSUPPORTED, "skinny linear: unsupported shape");
  if (((uintptr_t)x | (uintptr_t)y | (uintptr_t)norm_x | (uintptr_t)norm_g) % 16)
    return fail(FASTAV_EINVAL, "skinny linear: x, y and the norm inputs must be 16-byte aligned");
  if (norm_x && (!norm_g || epilogue == FASTAV_EPI_RESADD || !gemv_rows_supported(B, n, k, true)))
    return fail(FASTAV_EINVAL, "skinny linear: bad fused-norm arguments");
  SkinnyArgs a;
  a.xres = norm_x; a.g = (const bf16_t*)norm_g; a.eps = norm_eps;
  a.pos = rope ? rope->pos : nullptr; a.rope_tab = rope ? (const float2*)rope->table : nullptr;
  a.rope_rows = rope ? rope->rows : 0; a.dh = rope ? rope->head_dim : 16;
  a.rope_coef = rope ? -log2((double)rope->base) * 2.0 / (double)rope->head_dim : 0.0;
  a.app_k = app ? (bf16_t*)app->k : nullptr; a.app_v = app ? (bf16_t*)app->v : nullptr; a.app_stride = app ? app->row_stride : 0;
  a.app_k0 = app ? seg_rows[0] : n; a.app_v0 = app ? seg_rows[0] + seg_rows[1] : n;
  if ((ss_in || next) && (norm_x || gemv_rows_supported(B, n, k, false))) return fail(FASTAV_EINVAL, "skinny linear: the one-row kernel normalises for itself");
  if (next && epilogue != FASTAV_EPI_RESADD) return fail(FASTAV_EINVAL, "skinny linear: the next projection's input needs the residual epilogue");
  a.ss_in = ss_in;
  a.g_out = next ? (const bf16_t*)next->g : nullptr; a.xg_out = next ? (bf16_t*)next->xg : nullptr; a.ss_out = next ? next->ss : nullptr;
  a.x = (const bf16_t*)x; a.w2 = (const bf16_t*)w2; a.y = y; a.ldy = ldy; a.B = B; a.N = n; a.K = k;
  int end = 0;
  for (int i = 0; i < 3; ++i) {
    if (i < n_seg) {
      if (seg_rows[i] % 16 || ((uintptr_t)w_seg[i] % 16)) return fail(FASTAV_EINVAL, "skinny linear: segments must be 16-row, 16-byte aligned");
      end += seg_rows[i];
      a.w[i] = (const bf16_t*)w_seg[i];
    } else {
      a.w[i] = a.w[0];
    }
    a.seg_end[i] = i < n_seg ? end : 0x7FFFFFFF;
  }
  if (end != n) return fail(FASTAV_EINVAL, "skinny linear: segments do not add up to n");
  if (epilogue == FASTAV_EPI_SWIGLU && (!w2 || ((uintptr_t)w2 % 16)))
    return fail(FASTAV_EINVAL, "skinny linear: SwiGLU needs a 16-byte aligned up matrix");
  const int kind = epilogue == FASTAV_EPI_SWIGLU ? FASTAV_PROF_LINEAR_SWIGLU
                   : (epilogue == FASTAV_EPI_RESADD ? FASTAV_PROF_LINEAR_RESADD : FASTAV_PROF_LINEAR_STORE);
  // the work figure of a decode GEMV is its weight bytes (HBM-bound), not flops
  ProfScope prof(kind, (double)n * k * 2.0 * (epilogue == FASTAV_EPI_SWIGLU ? 2.0 : 1.0), s);
  if (gemv_rows_supported(B, n, k, norm_x != nullptr)) {
    const size_t lds = (size_t)k * 2;
#define FASTAV_GEMV(EPI, NORM, ROPE)                                                                            \
  do {                                                                                                          \
    if (lds > 32 * 1024) {                                                                                      \
      hipError_t e = hipFuncSetAttribute((const void*)k_gemv_rows<EPI, NORM, ROPE>, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024); \
      if (e != hipSuccess) return fail(FASTAV_EHIP, "gemv: hipFuncSetAttribute: %s", hipGetErrorString(e));     \
    }                                                                                                           \
    hipLaunchKernelGGL((k_gemv_rows<EPI, NORM, ROPE>), dim3((unsigned)(n / 16)), dim3(512), lds, s, a);         \
  } while (0)
    if (epilogue == FASTAV_EPI_SWIGLU) { if (norm_x) FASTAV_GEMV(FASTAV_EPI_SWIGLU, true, false); else FASTAV_GEMV(FASTAV_EPI_SWIGLU, false, false); }
    else if (epilogue == FASTAV_EPI_RESADD) FASTAV_GEMV(FASTAV_EPI_RESADD, false, false);
    else if (rope) { if (norm_x) FASTAV_GEMV(FASTAV_EPI_STORE, true, true); else FASTAV_GEMV(FASTAV_EPI_STORE, false, true); }
    else { if (norm_x) FASTAV_GEMV(FASTAV_EPI_STORE, true, false); else FASTAV_GEMV(FASTAV_EPI_STORE, false, false); }
#undef FASTAV_GEMV
    return check_launch("gemv_rows");
  }
  // Items have 16 features (8 pairs for SwiGLU).  Up to 4096 columns the batch fits a workgroup's registers and 256
  // workgroups (one per CU) walk the items, more than 256 of them; longer rows, the residual epilogue and products of one item per workgroup,
  // which leave nothing to be resident for, take the streaming kernel (8 rows, resident against streaming: 256 items of
  // 4096 columns 12.8 / 9.9 us, 192 of 2048 7.7 / 6.5, 288 of 3584 12.5 / 15.4).  Two gate/up items per workgroup share
  // the input where that leaves a workgroup per CU (28672 x 8192, one against two: 4 rows 192 / 179 us, 8 rows 202 / 180,
  // 16 rows 239 / 188; 2 rows of 8192 x 8192 56.6 / 58.2).
  const int items = epilogue == FASTAV_EPI_SWIGLU ? n / 8 : n / 16;
  const int nb = (k / 64 + kSkinnyWaves - 1) / kSkinnyWaves;
  if (epilogue == FASTAV_EPI_RESADD || nb > 8 || items <= 256) {
    const bool brief = k <= 64 * kSkinnyWaves * 4 && !ss_in && !rope && !app && !next;
#define FASTAV_STREAM(EPI, P, BRIEF) hipLaunchKernelGGL((k_skinny_stream<EPI, P, BRIEF>), dim3((unsigned)(items / P)), dim3(64 * kSkinnyWaves), 0, s, a)
    if (epilogue == FASTAV_EPI_RESADD) { if (brief) FASTAV_STREAM(FASTAV_EPI_RESADD, 1, true); else FASTAV_STREAM(FASTAV_EPI_RESADD, 1, false); }
    else if (epilogue == FASTAV_EPI_STORE) { if (brief) FASTAV_STREAM(FASTAV_EPI_STORE, 1, true); else FASTAV_STREAM(FASTAV_EPI_STORE, 1, false); }
    else if (B > 4 && items >= 512) FASTAV_STREAM(FASTAV_EPI_SWIGLU, 2, false);       // n is a multiple of 16: items are even
    else if (brief) FASTAV_STREAM(FASTAV_EPI_SWIGLU, 1, true);
    else FASTAV_STREAM(FASTAV_EPI_SWIGLU, 1, false);
#undef FASTAV_STREAM
    return check_launch("skinny_stream");
  }
  const dim3 grid(256);
#define FASTAV_SKINNY(EPI, NB) hipLaunchKernelGGL((k_skinny_resident<EPI, NB>), grid, dim3(64 * kSkinnyWaves), 0, s, a, items)
#define FASTAV_SKINNY_NB(EPI) \
  do { if (nb <= 2) FASTAV_SKINNY(EPI, 2); else if (nb <= 4) FASTAV_SKINNY(EPI, 4); else if (nb <= 7) FASTAV_SKINNY(EPI, 7); else FASTAV_SKINNY(EPI, 8); } while (0)
  if (epilogue == FASTAV_EPI_SWIGLU) FASTAV_SKINNY_NB(FASTAV_EPI_SWIGLU);
  else FASTAV_SKINNY_NB(FASTAV_EPI_STORE);
#undef FASTAV_SKINNY_NB
#undef FASTAV_SKINNY
  return check_launch("skinny_resident");
}

// ---------------------------------------------------------------------------------------- decode attention
struct DecodeAttnArgs {
  const bf16_t* q;            // [B, q_stride]: the new token's rotated queries
  const bf16_t* k_self;       // [B, q_stride]: its own rotated key ...
  const bf16_t* v_self;       // ... and value (all three live in the step's QKV row)
  int64_t q_stride;
  const bf16_t* k_prefix;     // [T_l, kd] packed per sample (cu_prefix), the prefill's cache of this layer
  const bf16_t* v_prefix;
  const int32_t* cu_prefix;   // [B + 1]
  const bf16_t* k_gen;        // [B, gen_cap, kd] tokens generated before this step (gen_len of them), or null
  const bf16_t* v_gen;
  int gen_len, gen_cap;
  int Hq, Hkv, splits, chunk; // chunk = keys per split (multiple of 64)
  float scale_log2;           // log2(e) / sqrt(head_dim): logits live in the base-2 domain
  float* part;                // [B, Hkv, splits, G, DH + 2] fp32: o (unnormalised), max (base-2 domain), sum
};

// One workgroup per (key split, KV head, sample); its four waves take the split's 64-key chunks in turn.
// Per chunk a wave
//   * reads the 64 keys straight from global memory in matrix-core operand layout (lane = key row x 16-byte
//     dim chunk) and the query heads of the group as the other operand (heads padded to 16 columns): the
//     logits of all heads of the group come out of DH/32 v_mfma_f32_16x16x32_bf16 per 16 keys, lane = head,
//     four keys each;
//   * updates the running (max, sum) of every head (in-lane over its keys, two shuffles across the lane
//     groups), writes the 64 x G probabilities to LDS;
//   * accumulates P V with lane = (key subgroup, 8 output dims): a V row is one 16-byte load per lane, the
//     G probabilities of its key one broadcast LDS read, G x 8 FMAs.
// Nothing is staged through LDS but the probabilities, and the waves never wait for each other until the
// end, where their (max, sum, o) are combined and written as the split's partial; k_decode_merge combines the
// splits.  (Merging in the same launch by the workgroup that finishes last was measured: the device-scope
// release every workgroup then needs writes back its L2 and costs more than the second launch.)
template <int DH, int GP>
__global__ __launch_bounds__(256) void k_decode_attn(DecodeAttnArgs a) {
  constexpr int CK = 64;                              // keys per chunk
  constexpr int STEPS = DH / 32;                      // matrix instructions per 16-key tile
  constexpr int SEGS = DH / 8;                        // lanes (16-byte segments) per V row
  constexpr int KPI = 64 / SEGS;                      // keys one wave-wide V load covers
  constexpr int NIT = CK / KPI;
  constexpr int PD = DH + 2;
  __shared__ __attribute__((aligned(16))) float ps[4][CK][GP];
  __shared__ __attribute__((aligned(16))) float red_o[4][GP][DH];     // the four waves' outputs
  __shared__ float red_m[4][GP], red_l[4][GP];
  const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int G = a.Hq / a.Hkv;                         // <= GP (checked by the launcher)
  const int kd = a.Hkv * DH;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p0 = a.cu_prefix[b], n_pre = a.cu_prefix[b + 1] - p0;
  const int n_tot = n_pre + a.gen_len + 1;
  const int j_begin = split * a.chunk;
  const int j_end = (j_begin + a.chunk < n_tot) ? j_begin + a.chunk : n_tot;
  const int head = lane & 15, lg = lane >> 4;         // logits: lane = (head column, lane group)
  const int seg = lane % SEGS, kq = lane / SEGS;      // P V: lane = (8 output dims, key subgroup)

  // row j of the unified key list: prefix, then generated, then the token itself
  auto krow = [&](int j) __attribute__((always_inline)) -> const bf16_t* {
    if (j < n_pre) return a.k_prefix + (int64_t)(p0 + j) * kd + g * DH;
    if (j < n_pre + a.gen_len) return a.k_gen + ((int64_t)b * a.gen_cap + (j - n_pre)) * kd + g * DH;
    return a.k_self + (int64_t)b * a.q_stride + g * DH;
  };
  auto vrow = [&](int j) __attribute__((always_inline)) -> const bf16_t* {
    if (j < n_pre) return a.v_prefix + (int64_t)(p0 + j) * kd + g * DH;
    if (j < n_pre + a.gen_len) return a.v_gen + ((int64_t)b * a.gen_cap + (j - n_pre)) * kd + g * DH;
    return a.v_self + (int64_t)b * a.q_stride + g * DH;
  };

  bf16x8_t qf[STEPS];
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    bf16x8_t z = {0, 0, 0, 0, 0, 0, 0, 0};
    qf[st] = head < G ? *(const bf16x8_t*)(a.q + (int64_t)b * a.q_stride + (g * G + head) * DH + lg * 8 + 32 * st) : z;
  }
  float m_run = -INFINITY, l_part = 0.f;              // per head (column): max over all lane groups, this lane's share of the sum
  float acc[GP][8];
#pragma unroll
  for (int h = 0; h < GP; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.f;

  for (int c0 = j_begin + wave * CK; c0 < j_end; c0 += 4 * CK) {
    bf16x8_t kf[4][STEPS], vf[NIT];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      int j = c0 + t * 16 + head;                     // here `head` is the key row of the A operand
      j = j < j_end ? j : j_end - 1;                  // rows past the end repeat the last key (masked below)
      const bf16_t* kr = krow(j) + lg * 8;
#pragma unroll
      for (int st = 0; st < STEPS; ++st) kf[t][st] = *(const bf16x8_t*)(kr + 32 * st);
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      int j = c0 + it * KPI + kq;
      j = j < j_end ? j : j_end - 1;
      vf[it] = *(const bf16x8_t*)(vrow(j) + seg * 8);
    }
    f32x4v sc[4];
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4v c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < STEPS; ++st) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][st], qf[st], c, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        c[r] = (c0 + t * 16 + lg * 4 + r < j_end) ? c[r] * a.scale_log2 : -INFINITY;
        mx = fmaxf(mx, c[r]);
      }
      sc[t] = c;
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));        // finite: key c0 exists
    const float m_new = fmaxf(m_run, mx);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);      // exp2(-inf) = 0 on the first chunk
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pr = __builtin_amdgcn_exp2f(sc[t][r] - m_new);
        psum += pr;
        if (head < GP) ps[wave][t * 16 + lg * 4 + r][head] = pr;
      }
    l_part = l_part * alpha + psum;
    m_run = m_new;
    // the wave's own LDS writes are visible to its other lanes after the LDS counter wait below
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
#pragma unroll
    for (int h = 0; h < GP; ++h) {
      const float ah = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), h));          // lane h holds head h
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[h][e] *= ah;
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      float pv[GP];
#pragma unroll
      for (int h4 = 0; h4 < GP; h4 += 4) {
        const f32x4v t4 = *(const f32x4v*)&ps[wave][it * KPI + kq][h4];
        pv[h4] = t4[0]; pv[h4 + 1] = t4[1]; pv[h4 + 2] = t4[2]; pv[h4 + 3] = t4[3];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = (float)vf[it][e];
#pragma unroll
        for (int h = 0; h < GP; ++h) acc[h][e] = fmaf(pv[h], v, acc[h][e]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();                  // all reads of ps done before the next chunk rewrites it
  }

  // ---- combine inside the wave: the sum over lane groups, the outputs over key subgroups
  l_part += __shfl_xor(l_part, 16, kWave);
  l_part += __shfl_xor(l_part, 32, kWave);
#pragma unroll
  for (int h = 0; h < GP; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float v = acc[h][e];
#pragma unroll
      for (int o = SEGS; o < 64; o <<= 1) v += __shfl_xor(v, o, kWave);
      acc[h][e] = v;
    }
  if (kq == 0) {
#pragma unroll
    for (int h = 0; h < GP; ++h) {
      f32x4v lo = {acc[h][0], acc[h][1], acc[h][2], acc[h][3]}, hi = {acc[h][4], acc[h][5], acc[h][6], acc[h][7]};
      *(f32x4v*)&red_o[wave][h][seg * 8] = lo;
      *(f32x4v*)&red_o[wave][h][seg * 8 + 4] = hi;
    }
  }
  if (lane < GP) { red_m[wave][lane] = m_run; red_l[wave][lane] = l_part; }
  __syncthreads();
  // ---- combine the four waves, write the split's partial: thread = (head, dim)
  float* part = a.part + (((int64_t)b * a.Hkv + g) * a.splits + split) * (int64_t)(G * PD);
  for (int i = tid; i < G * DH; i += 256) {
    const int h = i / DH, d = i % DH;
    float M = red_m[0][h];
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, red_m[w][h]);
    float o = 0.f, l = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float mw = red_m[w][h];
      const float f = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
      o = fmaf(f, red_o[w][h][d], o);
      l = fmaf(f, red_l[w][h], l);
    }
    part[h * PD + d] = o;
    if (d == 0) { part[h * PD + DH] = M; part[h * PD + DH + 1] = l; }
  }
}

// Merge of the splits' partials: one workgroup per (query head, sample), no loop-carried waits.  Every wave
// loads the splits' (max, sum) with lane = split and gets the global max and the weights from two wave
// reductions; thread = (split group, 4 output dims) has the weighted outputs of its splits in flight at the same
// time (independent 8-byte loads, out-of-range splits clamped and weighted 0), and the groups are summed through
// LDS.  splits <= 64.
template <int DH>
__global__ __launch_bounds__(256) void k_decode_merge(const float* __restrict__ part_all, int splits, int Hq, int Hkv,
                                                      bf16_t* __restrict__ out, int64_t out_stride) {
  constexpr int PD = DH + 2;
  constexpr int QUADS = DH / 4;                       // 32 or 16 column quads
  constexpr int NSG = 256 / QUADS;                    // 8 or 16 split groups
  constexpr int NK = 64 / NSG;                        // splits per thread
  __shared__ __attribute__((aligned(16))) float red_o[NSG][DH];
  const int hq = blockIdx.x, b = blockIdx.y;
  const int G = Hq / Hkv, g = hq / G, h = hq % G;
  const int tid = threadIdx.x, lane = tid & 63;
  // partial of (split sp, head h): pall + sp * G * PD
  const float* pall = part_all + (((int64_t)b * Hkv + g) * splits * G + h) * (int64_t)PD;
  const int c = tid % QUADS, sg = tid / QUADS;
  float2 lo[NK], hi[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    int sp = sg + k * NSG;
    sp = sp < splits ? sp : splits - 1;
    // rows are PD = DH + 2 floats apart: 8-byte aligned, so two 8-byte loads per quad
    lo[k] = *(const float2*)(pall + (int64_t)sp * G * PD + c * 4);
    hi[k] = *(const float2*)(pall + (int64_t)sp * G * PD + c * 4 + 2);
  }
  const float ms = lane < splits ? pall[(int64_t)lane * G * PD + DH] : -INFINITY;   // -inf: a split past this sample's keys
  const float ls = lane < splits ? pall[(int64_t)lane * G * PD + DH + 1] : 0.f;
  const float M = wave_max(ms);                       // finite: split 0 always holds a key
  const float wgt = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ms - M);
  const float inv = 1.0f / wave_sum(wgt * ls);
  f32x4v o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int sp = sg + k * NSG;                      // < 64: lane sp of this wave holds its weight (0 beyond splits)
    const float f = __shfl(wgt, sp, kWave);
    o[0] = fmaf(f, lo[k].x, o[0]); o[1] = fmaf(f, lo[k].y, o[1]);
    o[2] = fmaf(f, hi[k].x, o[2]); o[3] = fmaf(f, hi[k].y, o[3]);
  }
  *(f32x4v*)&red_o[sg][c * 4] = o;
  __syncthreads();
  if (tid < DH) {
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < NSG; ++q) t += red_o[q][tid];
    out[(int64_t)b * out_stride + hq * DH + tid] = (bf16_t)(t * inv);
  }
}

// partials [B, Hkv, splits, G, dh + 2] fp32
size_t decode_attn_workspace_bytes(int batch, int Hq, int dh, int max_splits) {
  return align_up((size_t)batch * Hq * max_splits * (dh + 2) * sizeof(float), 256);
}

// Keys per split.  A workgroup's four waves take 64 keys each, so shares of 256 keys keep all of them at work; the sums of the
// waves meet in LDS, those of the splits in the merge.  The finest shares (about four workgroups per CU, whatever is left of them
// for a wave) are better where the loads in flight are few, or where shares of 256 end in an uneven second round.
// A layer's time in us with caches that come from HBM (hidden 512, so that attention is most of it), finest / 256 keys:
// - fewer than 192 workgroups of 256, or keys for fewer than 128: 1 x 4096 keys, 28/4 heads of 128 (68 workgroups) 25.2 / 27.5,
//   4 x 1500 (96) 33.4 / 34.8, 1 x 6000, 32/4 heads of 64 (96) 22.5 / 23.1, 12 x 310, 32/8 of 128 (192 with keys for 116) 34.6 / 35.8;
//   from 192 to 256: 4 x 3012, 28/4 of 128 40.2 / 36.1, 8 x 1988 42.6 / 37.9,
//   1 x 8132, 32/8 of 128 30.2 / 29.3, 4 x 4036, 32/4 of 64 35.6 / 29.6
// - 257 to 400, a second round of up to a half: heads of 64 2 x 2500, 16/16 27.3 / 28.6, 4 x 2244, 32/8 29.0 / 30.1, 1 x 5572,
//   16/16 24.9 / 26.3; heads of 128 take 192 keys there: 2 x 10180, 28/4 finest 39.1, 256 41.5, 192 39.1; 1 x 12228, 32/8 32.3,
//   33.0, 32.4; 2 x 5060, 32/8 38.0, 37.7, 36.4
// - beyond: 2 x 7108, 32/8 of 128 42.3 / 38.3, 8 x 6000 68.7 / 65.1, 16 x 4096 89.0 / 80.9, 8 x 16000, 16/16 of 64 132 / 113, 8 x 3524,
//   32/4 of 64 36.4 / 33.7.  Not with more than four query heads of 64 to a key head once the finest are longer than 384:
//   8 x 12300, 32/4 47.8 / 48.7, 8 x 16000 53.6 / 54.9
// - beyond 16384 keys 64 splits ask for more than 256 keys.  The fewest that do (a multiple of 64), which for small batches are
//   the finest: 1 x 16600, 32/8 of 128 37.5, with 512 keys 40.4; 2 x 20000, 28/4 46.9, 51.0; 4 x 16600, 16/16 of 64 finest 76.3,
//   fewest 71.6, 512 73.4; 8 x 16600, 32/8 136.5, 131.8, 130.8.  With more than four query heads to a key head the finest:
//   8 x 16600, 28/4 of 128 88.8, 91.2, 91.0, 32/4 of 64 54.4, 57.1, 54.7.
static int decode_attn_chunk(int batch, int Hq, int Hkv, int dh, int max_keys) {
  const int64_t groups = (int64_t)batch * Hkv, want = (1024 + groups - 1) / groups, blocks = ceil_div(max_keys, 64);
  int64_t splits = want < blocks ? want : blocks;
  if (splits > 64) splits = 64;
  const int64_t finest = ceil_div(ceil_div(max_keys, splits), 64) * 64, fewest = ceil_div(blocks, 64) * 64;   // fewest: 64 splits
  const int64_t workgroups = ceil_div(max_keys, 256) * groups;
  const bool many_heads = Hq > 4 * Hkv;
  if (workgroups < 192 || max_keys * groups < 128 * 256 || (many_heads && (fewest > 256 || (dh == 64 && finest > 384)))) return (int)finest;
  if (workgroups > 256 && workgroups <= 400 && fewest <= 192) return dh == 64 ? (int)finest : 192;
  return (int)(fewest > 256 ? fewest : 256);
}

fastav_status_t launch_decode_attention(const void* q, const void* k_self, const void* v_self, int64_t q_stride,
                                        const void* k_prefix, const void* v_prefix, const int32_t* cu_prefix,
                                        int max_prefix, const void* k_gen, const void* v_gen, int gen_len,
                                        int gen_cap, int batch, int Hq, int Hkv, int dh, float* part,
                                        size_t part_bytes, void* out, int64_t out_stride, double bytes_hint,
                                        hipStream_t s) {
  if (batch == 0) return FASTAV_OK;
  if (dh != 64 && dh != 128) return fail(FASTAV_EUNSUPPORTED, "decode attention: head_dim must be 64 or 128");
  if (Hq % Hkv || Hq / Hkv > 8) return fail(FASTAV_EUNSUPPORTED, "decode attention: at most 8 query heads per KV head");
  if (gen_len > 0 && (!k_gen || !v_gen)) return fail(FASTAV_EINVAL, "decode attention: gen_len > 0 needs the generated-token caches");
  if (q_stride % 8 || ((uintptr_t)q | (uintptr_t)k_self | (uintptr_t)v_self | (uintptr_t)k_prefix | (uintptr_t)v_prefix |
                        (uintptr_t)k_gen | (uintptr_t)v_gen) % 16 || ((Hkv * dh) % 8))
    return fail(FASTAV_EINVAL, "decode attention: operands must be 16-byte aligned");
  DecodeAttnArgs a;
  a.q = (const bf16_t*)q; a.k_self = (const bf16_t*)k_self; a.v_self = (const bf16_t*)v_self; a.q_stride = q_stride;
  a.k_prefix = (const bf16_t*)k_prefix; a.v_prefix = (const bf16_t*)v_prefix; a.cu_prefix = cu_prefix;
  a.k_gen = (const bf16_t*)k_gen; a.v_gen = (const bf16_t*)v_gen; a.gen_len = gen_len; a.gen_cap = gen_cap;
  a.Hq = Hq; a.Hkv = Hkv;
  const int max_keys = max_prefix + gen_len + 1;
  a.chunk = decode_attn_chunk(batch, Hq, Hkv, dh, max_keys);
  a.splits = (int)ceil_div(max_keys, a.chunk);          // at most 64
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
  a.part = part;
  if ((size_t)batch * Hq * a.splits * (dh + 2) * sizeof(float) > part_bytes)
    return fail(FASTAV_EINVAL, "decode attention: workspace too small");
  ProfScope prof(FASTAV_PROF_ATTENTION, bytes_hint, s);
  const dim3 grid((unsigned)a.splits, (unsigned)Hkv, (unsigned)batch);
  const int G = Hq / Hkv;
  const dim3 mgrid((unsigned)Hq, (unsigned)batch);
#define FASTAV_DECODE_ATTN(DH_, GP_)                                                                              \
  do {                                                                                                            \
    hipLaunchKernelGGL((k_decode_attn<DH_, GP_>), grid, dim3(256), 0, s, a);                                      \
    hipLaunchKernelGGL((k_decode_merge<DH_>), mgrid, dim3(256), 0, s, (const float*)part, a.splits, Hq, Hkv,      \
                       (bf16_t*)out, out_stride);                                                                 \
  } while (0)
  if (dh == 128 && G <= 4) FASTAV_DECODE_ATTN(128, 4);
  else if (dh == 128) FASTAV_DECODE_ATTN(128, 8);
  else if (G <= 4) FASTAV_DECODE_ATTN(64, 4);
  else FASTAV_DECODE_ATTN(64, 8);
#undef FASTAV_DECODE_ATTN
  return check_launch("decode_attention");
}

}  // namespace fastav
