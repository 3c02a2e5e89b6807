// Causal grouped-query attention for the fp32 models on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 accumulate, expf), with
// the last query row's logits and (max, sum) as the side output Eq. 4 is finished from.
//
// A workgroup owns 16 query rows of one head; its waves take the 16-key tiles in turn, each with a running
// (max, sum, O) of its own, and merge them through LDS at the end.  A prompt of a few hundred tokens has few query
// tiles (512 tokens x 4 heads: 128), so the keys are what is spread over the chip's waves; the longest chain of a
// wave is n / (16 waves) tiles.
//
// Products are formed transposed, S^T = K Q^T and O^T = V^T P^T, with the operands straight from global memory (L2):
//   K, Q  lane = row lane % 16, 16 bytes at dim 4 (lane / 16) of a 16-wide chunk, element s for matrix instruction s;
//   S^T   lane = query lane % 16, keys 4 (lane / 16) + r: already the second product's right operand, instruction r
//         taking the keys {r, 4 + r, 8 + r, 12 + r};
//   V^T   instruction r wants V[key 4 (lane / 16) + r][dim of row lane % 16]; rows stand for the dims 4 (lane % 16) + e,
//         so one 16-byte load feeds four instructions, and a lane ends up with 16 consecutive output dims.
// 512 tokens, 4 heads of 64: 564 us on the vector ALUs (one lane per query row, four workgroups per head and no
// second wave to hide behind) against 12.7 us; 256 tokens 284 against 8.4 us.
#include "common.hpp"

namespace fastav {

struct AttnF32Args {
  const float* q; const float* k; const float* v; float* o;
  int64_t qs, kvs, os;
  const int32_t* cu;
  int Hq, Hkv;
  float scale;
  int64_t T;
  float* last_logits; float* last_ml;
};

template <int DH, int NW>
__global__ __launch_bounds__(64 * NW) void k_attn_f32(AttnF32Args a) {
  constexpr int NC = DH / 16;                           // 16-wide chunks of the head dimension
  constexpr int NV = DH / 64;                           // 64-dim groups of a V row (16 bytes per lane each)
  __shared__ __attribute__((aligned(16))) float red_o[NW][16][DH];
  __shared__ float red_m[NW][16], red_l[NW][16];
  const int b = blockIdx.z, h = blockIdx.y;
  const int row0 = a.cu[b], n = a.cu[b + 1] - row0;
  const int n_qt = (n + 15) / 16;
  const int qt = n_qt - 1 - (int)blockIdx.x;            // the long tiles first
  if (qt < 0) return;
  const int q0 = qt * 16;
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = h / (a.Hq / a.Hkv);
  const int qi = q0 + l16 < n ? q0 + l16 : n - 1;       // rows past the sample repeat its last one and are not stored
  const bool emit = a.last_logits != nullptr && q0 + l16 == n - 1;
  const float* kb = a.k + (int64_t)row0 * a.kvs + g * DH;
  const float* vb = a.v + (int64_t)row0 * a.kvs + g * DH;

  f32x4_t qf[NC];
  {
    const float* qp = a.q + (int64_t)(row0 + qi) * a.qs + h * DH + l4 * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) qf[c] = *(const f32x4_t*)(qp + 16 * c);
  }
  f32x4_t o[NV][4];
#pragma unroll
  for (int u = 0; u < NV; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[u][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;

  auto load = [&](int kt, f32x4_t (&kf)[NC], f32x4_t (&vf)[4][NV]) __attribute__((always_inline)) {
    int key = kt * 16 + l16;
    key = key < n ? key : n - 1;                        // masked below
    const float* kp = kb + (int64_t)key * a.kvs + l4 * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *(const f32x4_t*)(kp + 16 * c);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int vk = kt * 16 + l4 * 4 + r;
      vk = vk < n ? vk : n - 1;
#pragma unroll
      for (int u = 0; u < NV; ++u) vf[r][u] = *(const f32x4_t*)(vb + (int64_t)vk * a.kvs + u * 64 + l16 * 4);
    }
  };
  // every tile up to the query tile's own has at least one key every one of its rows sees
  f32x4_t kf[2][NC], vf[2][4][NV];
  auto tile = [&](int kt, int st) __attribute__((always_inline)) {
    if (kt + NW <= qt) load(kt + NW, kf[st ^ 1], vf[st ^ 1]);
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[st][c][e], qf[c][e], s, 0, 0, 0);
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = kt * 16 + l4 * 4 + r;
      s[r] *= a.scale;
      if (emit && key < n) a.last_logits[(int64_t)h * a.T + row0 + key] = s[r];
      if (key > qi) s[r] = -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    // a wave's keys may all have the logit -inf so far (masked with the lowest value, or overflowed): the maximum then
    // stays -inf and the exponents are taken against 0, so that the terms are expf(-inf) = 0 and not expf(-inf + inf)
    const float mn = fmaxf(m, mx), ms = mn == -INFINITY ? 0.f : mn;
    const float corr = expf(m - ms);                    // the first tile: expf(-inf) = 0
    m = mn;
    l *= corr;
#pragma unroll
    for (int r = 0; r < 4; ++r) { s[r] = expf(s[r] - ms); l += s[r]; }
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[u][e] = o[u][e] * corr;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[u][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[st][r][u][e], s[r], o[u][e], 0, 0, 0);
      }
  };
  if (wave <= qt) load(wave, kf[0], vf[0]);
  for (int kt = wave; kt <= qt; kt += 2 * NW) {
    tile(kt, 0);
    if (kt + NW <= qt) tile(kt + NW, 1);
  }
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);

  // o[u][e][r] is dim 64 u + 16 l4 + 4 r + e of query l16
#pragma unroll
  for (int u = 0; u < NV; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4_t t = {o[u][0][r], o[u][1][r], o[u][2][r], o[u][3][r]};
      *(f32x4_t*)&red_o[wave][l16][u * 64 + l4 * 16 + r * 4] = t;
    }
  if (l4 == 0) { red_m[wave][l16] = m; red_l[wave][l16] = l; }
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * DH / 4; i += 64 * NW) {
    const int row = i / (DH / 4), d = (i % (DH / 4)) * 4;
    if (q0 + row >= n) continue;
    float M = red_m[0][row];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, red_m[w][row]);
    const float Ms = M == -INFINITY ? 0.f : M;          // every logit of the row -inf: M = -inf, L = 0
    f32x4_t t = {0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = expf(red_m[w][row] - Ms);         // a wave without tiles, or without a finite logit: expf(-inf) = 0
      t = t + *(const f32x4_t*)&red_o[w][row][d] * f;
      L = fmaf(f, red_l[w][row], L);
    }
    *(f32x4_t*)(a.o + (int64_t)(row0 + q0 + row) * a.os + h * DH + d) = t * (1.0f / L);
    if (a.last_ml != nullptr && d == 0 && q0 + row == n - 1) {
      a.last_ml[((int64_t)b * a.Hq + h) * 2] = M;
      a.last_ml[((int64_t)b * a.Hq + h) * 2 + 1] = L;
    }
  }
}

bool f32_attention_supported(const void* q, int64_t q_stride, const void* k, const void* v, int64_t kv_stride, const void* o,
                             int64_t o_stride, int batch, int Hq, int dh) {
  return (dh == 64 || dh == 128) && (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) % 16) == 0 &&
         ((q_stride | kv_stride | o_stride) % 4) == 0 && batch <= 65535 && Hq <= 65535;
}

fastav_status_t launch_attention_f32(const void* q, int64_t q_stride, const void* k, const void* v, int64_t kv_stride, void* o,
                                     int64_t o_stride, const int32_t* cu, int batch, int64_t T, int max_seqlen, int Hq, int Hkv,
                                     int dh, float* last_logits, float* last_ml, hipStream_t s) {
  if (batch == 0 || max_seqlen == 0) return FASTAV_OK;
  AttnF32Args a = {(const float*)q, (const float*)k, (const float*)v, (float*)o, q_stride, kv_stride, o_stride, cu, Hq, Hkv,
                   1.0f / sqrtf((float)dh), T, last_logits, last_ml};
  const dim3 grid((unsigned)ceil_div(max_seqlen, 16), (unsigned)Hq, (unsigned)batch);
  if (dh == 128) hipLaunchKernelGGL((k_attn_f32<128, 4>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_attn_f32<64, 8>), grid, dim3(512), 0, s, a);
  return check_launch("attention_f32");
}

}  // namespace fastav
