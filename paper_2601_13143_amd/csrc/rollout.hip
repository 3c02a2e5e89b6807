// Attention rollout (Eq. 2-3 of the paper): the offline analysis that tells FastAV where to prune globally.
//
//   A^l  = mean over heads of the causal attention weights of layer l        (k_attn_rowstats + k_attn_map, k_attn_map_short)
//   R^l  = (alpha A^l + (1 - alpha) I) R^{l-1}                               (k_rollout_step)
//
// The head-mean map is formed without ever holding a per-head n x n map, from every query row's softmax (max, 1 / sum)
// per head.  A rollout has those from the layer's own attention launch; its last layer, whose attention nobody needs, and
// a direct call make them in a pass of their own, which streams K through the matrix cores (S^T = K Q^T tiles, running max
// and sum per lane, like the prefill attention but with no values).  The map then recomputes each tile of logits for every
// head, turns it into probabilities and accumulates the mean in registers, so A is written exactly once (bf16, the operand
// type of the step that consumes it): 64 x 64 tiles whose rows of Q and K pass through LDS, or for short prompts 32 x 64
// tiles read straight from memory in operand layout, as the statistics are.
//
// The rollout is kept transposed, RT = (R^l)^T: RT_new = RT (alpha A + (1 - alpha) I)^T = alpha (RT A^T) + (1 - alpha) RT, so
// that both operands are read along their rows.  RT is carried in fp32 with a bf16 copy as the matrix operand.
#include "common.hpp"

namespace fastav {

struct MapArgs {
  const bf16_t* q; const bf16_t* k;
  int64_t qs, ks;               // row strides in elements
  int n, Hq, Hkv;
  float scale_log2;             // log2(e) / sqrt(head_dim)
  float2* stats;                // [Hq][n]: a row's maximum (log2 domain) and the reciprocal of its sum of exp2
  bf16_t* a_out;                // [n, ld]; columns up to n_cols are written
  int64_t ld; int n_cols;
  bool lower;                   // tiles above the diagonal are not written
  bool lines;                   // rows of a_out lie at 16-byte addresses
};

// Q operand (B of S^T = K Q^T): lane = query l32, k-chunk hf of k-step s.  K operand (A): lane = key l32.
template <int DH>
__device__ __forceinline__ void load_q_frags(const MapArgs& a, int qrow, int h, int hf, bf16x8_t (&qf)[DH / 16]) {
  const bf16_t* qp = a.q + (int64_t)qrow * a.qs + h * DH + hf * 8;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) qf[s] = *(const bf16x8_t*)(qp + 16 * s);
}
template <int DH>
__device__ __forceinline__ void load_k_frags(const MapArgs& a, int krow, int g, int hf, bf16x8_t (&kf)[DH / 16]) {
  const bf16_t* kp = a.k + (int64_t)krow * a.ks + g * DH + hf * 8;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) kf[s] = *(const bf16x8_t*)(kp + 16 * s);
}

// The statistics read their operands straight from global memory in operand layout; at one wave per SIMD each key block
// waited for its own loads, so a query tile's keys are dealt over the eight waves of a workgroup, whose results meet in LDS,
// and the next block's operands are requested before the present one is used: 2048 tokens, 32 heads of 128: 117 -> 58 us
// (82 with the workgroups of one head together).
constexpr int kStatWaves = 8;

// grid (Hq, query tiles of 64, the longest first: one head's rows lie at the pitch of the fused Q|K|V rows, often all in one
// L2 channel, so the workgroups that run together take different heads); wave w takes key blocks w, w + 8, .. of 32 keys for all 64 query rows
// (a key fragment then serves two products).
template <int DH>
__global__ __launch_bounds__(kStatWaves * 64) void k_attn_rowstats(MapArgs a) {
  constexpr int NS = DH / 16;
  __shared__ float2 part[kStatWaves][64];
  const int h = blockIdx.x, g = h / (a.Hq / a.Hkv);
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int q0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * 64;
  bf16x8_t qf[2][NS];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int qi = q0 + qb * 32 + l32;
    load_q_frags<DH>(a, qi < a.n ? qi : a.n - 1, h, hf, qf[qb]);
  }
  const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};
  const int n_blocks = (((q0 + 64 < a.n) ? q0 + 64 : a.n) + 31) / 32;      // key blocks the tile can see
  bf16x8_t kn[NS];
  {
    const int key = wave * 32 + l32;
    load_k_frags<DH>(a, key < a.n ? key : a.n - 1, g, hf, kn);
  }
  for (int kb = wave; kb < n_blocks; kb += kStatWaves) {
    bf16x8_t kf[NS];
#pragma unroll
    for (int st = 0; st < NS; ++st) kf[st] = kn[st];
    {
      const int key = (kb + kStatWaves) * 32 + l32;      // past the last block: a valid row, unused
      load_k_frags<DH>(a, key < a.n ? key : a.n - 1, g, hf, kn);
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      f32x16_t s = zero16;
#pragma unroll
      for (int st = 0; st < NS; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], qf[qb][st], s, 0, 0, 0);
      // s[r] = (key kb*32 + (r/4)*8 + hf*4 + r%4, query q0 + qb*32 + l32)
      const int qi = q0 + qb * 32 + l32;
      float x[16], mx = m[qb];
      if (kb * 32 + 31 <= q0 + qb * 32) {               // every key is visible to every row of the block
#pragma unroll
        for (int r = 0; r < 16; ++r) { x[r] = s[r] * a.scale_log2; mx = fmaxf(mx, x[r]); }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kk = kb * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
          x[r] = (kk <= qi && kk < a.n) ? s[r] * a.scale_log2 : -INFINITY;
          mx = fmaxf(mx, x[r]);
        }
      }
      const float ms = (mx == -INFINITY) ? 0.f : mx;
      float add = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) add += __builtin_amdgcn_exp2f(x[r] - ms);
      l[qb] = l[qb] * __builtin_amdgcn_exp2f(m[qb] - ms) + add;
      m[qb] = mx;
    }
  }
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    // the lane 32 away holds the other half of this query's keys
    const float m2 = __shfl_xor(m[qb], 32, kWave), l2 = __shfl_xor(l[qb], 32, kWave);
    const float mt = fmaxf(m[qb], m2), ms = (mt == -INFINITY) ? 0.f : mt;
    const float lt = l[qb] * __builtin_amdgcn_exp2f(m[qb] - ms) + l2 * __builtin_amdgcn_exp2f(m2 - ms);
    if (hf == 0) part[wave][qb * 32 + l32] = make_float2(mt, lt);
  }
  __syncthreads();
  const int qi = q0 + (int)threadIdx.x;
  if (threadIdx.x < 64 && qi < a.n) {
    float mt = -INFINITY, lt = 0.f;
#pragma unroll
    for (int w = 0; w < kStatWaves; ++w) mt = fmaxf(mt, part[w][threadIdx.x].x);      // key 0 is always visible: mt is finite
#pragma unroll
    for (int w = 0; w < kStatWaves; ++w) lt += part[w][threadIdx.x].y * __builtin_amdgcn_exp2f(part[w][threadIdx.x].x - mt);
    a.stats[(int64_t)h * a.n + qi] = make_float2(mt, 1.0f / lt);
  }
}

// A workgroup makes one 64 x 64 tile of A = mean over heads of exp2(logit - max) / sum: four 32 x 32 blocks, each by HG waves
// that share out the heads.
//
// Bound by the vector ALU: a logit costs two FMAs and one v_exp_f32 (24 clocks a wave), 12 us for 2048 tokens and 32 heads, the
// matrix instructions 9.  What it spent its time on were the query rows: read straight from global memory in operand
// layout, the 32 rows of a load lie in 32 cache lines at one offset, which one bank of the vector cache serves one after the
// other (a row pitch 16 bytes off the line size alone made the map a third faster).  So the rows of the next heads are
// copied to LDS in whole lines while the present ones are computed, and the keys of a group of query heads on the same way,
// from where they go to registers.  A block's 16 sums, its keys and a head's rows are 128 registers and a stage of both halves 32 KB: two workgroups
// of eight waves (HG = 2) on a CU, 512 of the 528 tiles of 2048 tokens at once; the last 16, on the diagonal and shorter, follow
// as CUs come free.  Up to 256 tiles a workgroup has a CU to itself and takes sixteen waves (HG = 4), which halves its chain.
// 2048 tokens, 32 / 8 heads of 128, inside a rollout: 94 -> 49 us; 3600 tokens alone 205 -> 85.
// Order: the tiles below the diagonal, in a contiguous run per XCD (block id % 8) which shares the query rows in its L2; then
// the tiles on the diagonal, which are three quarters of one; then, where the caller wants them, the zeros above it.
__device__ __forceinline__ void map_tile(int b, int nt, int& I, int& J) {
  const int below = nt * (nt - 1) / 2;
  const bool zeros = b >= below + nt;
  if (b >= below && !zeros) { I = J = b - below; return; }
  if (zeros) b -= below + nt;
  else {
    const int q = below / 8, r = below % 8, x = b % 8;
    b = x * q + (x < r ? x : r) + b / 8;
  }
  int i = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)b)) * 0.5f);     // row i holds tiles i (i - 1) / 2 .. + i - 1
  while (i * (i - 1) / 2 > b) --i;
  while ((i + 1) * i / 2 <= b) ++i;
  const int j = b - i * (i - 1) / 2;
  I = zeros ? j : i; J = zeros ? i : j;
}
template <int DH, int HG>
__global__ __launch_bounds__(HG * 256, 4) void k_attn_map(MapArgs a) {
  constexpr int NS = DH / 16, DCH = DH / 8, RPI = 64 / DCH;       // k-steps; 16-byte chunks of a row; rows a copy instruction fills
  constexpr int TILE = 64 * DCH, NCP = 64 / RPI / 4;              // chunks of a head's 64 rows; copy instructions per wave
  extern __shared__ bf16x8_t map_lds[];                           // [stage][share of the heads][TILE]; at the end the blocks' sums
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int w4 = wave & 3, qb = w4 & 1, kb = w4 >> 1, hg = wave >> 2;
  int I, J;
  map_tile((int)blockIdx.x, (a.n + 63) / 64, I, J);
  const int q0 = I * 64, j0 = J * 64;
  f32x4_t v[4];                                                   // the block's sums: keys kb * 32 + r4 * 8 + hf * 4 .. + 3 of row l32
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) v[r4] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (J <= I) {
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const bool live = J < I || kb <= qb;                          // the upper block of a diagonal tile stays zero
    const int qr = q0 + qb * 32 + l32 < a.n ? q0 + qb * 32 + l32 : a.n - 1;
    const int G = a.Hq / a.Hkv;
    const int h0 = a.Hq * hg / HG, h1 = a.Hq * (hg + 1) / HG;
    // a copy instruction fills rows RPI (4 i + w4) .. of a buffer in lane order; the chunk a slot holds is swizzled on the global
    // side so that the 16 rows an operand read takes at a time lie in 16 slots of the 64 banks
    auto swz = [](int row, int c) { return DH == 128 ? (c ^ (row & 15)) : (c ^ ((row >> 1) & 7)); };
    const uint32_t buf = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(map_lds + hg * TILE);
    uint32_t qoff[NCP], koff[NCP];
#pragma unroll
    for (int i = 0; i < NCP; ++i) {
      const int row = (4 * i + w4) * RPI + lane / DCH;
      const uint32_t chunk = (uint32_t)swz(row, lane % DCH) * 16u;
      qoff[i] = (uint32_t)(q0 + row < a.n ? row : a.n - 1 - q0) * (uint32_t)a.qs * 2u + chunk;
      koff[i] = (uint32_t)(j0 + row < a.n ? row : a.n - 1 - j0) * (uint32_t)a.ks * 2u + chunk;
    }
    const bf16_t* qbase = a.q + (int64_t)q0 * a.qs;
    const bf16_t* kbase = a.k + (int64_t)j0 * a.ks;
    // What a half goes through: the keys of a group, then its query heads one by one, through one pair of buffers.
    int h = h0, g = -1, now = 0;                        // the next head to copy, the group whose keys are on their way; 1 = keys, 2 = a head
    float2 sn = make_float2(0.f, 0.f);
    auto copy_next = [&](int st) __attribute__((always_inline)) -> int {
      if (h >= h1) return 0;
      const uint32_t dst = buf + (uint32_t)(st * HG * TILE * 16) + (uint32_t)(w4 * RPI * DCH * 16);
      if (h / G != g) {
        g = h / G;
#pragma unroll
        for (int i = 0; i < NCP; ++i) lds_copy16(kbase + g * DH, koff[i], dst + (uint32_t)(4 * i * RPI * DCH * 16));
        return 1;
      }
#pragma unroll
      for (int i = 0; i < NCP; ++i) lds_copy16(qbase + h * DH, qoff[i], dst + (uint32_t)(4 * i * RPI * DCH * 16));
      sn = a.stats[(int64_t)h * a.n + qr];
      ++h;
      return 2;
    };
    auto items = [&](int lo, int hi) { return hi > lo ? hi - lo + (hi - 1) / G - lo / G + 1 : 0; };
    int steps = 0;
#pragma unroll
    for (int p = 0; p < HG; ++p) {
      const int c = items(a.Hq * p / HG, a.Hq * (p + 1) / HG);
      steps = c > steps ? c : steps;
    }
    bf16x8_t kf[NS];
#pragma unroll
    for (int st = 0; st < NS; ++st) kf[st] = bf16x8_t{};
    now = copy_next(0);
    for (int i = 0; i < steps; ++i) {
      __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0): this wave's part of the rows has landed
      asm volatile("" : : : "memory");
      __syncthreads();                                  // the others' parts too, and everybody is done with the other stage
      const float m = sn.x, inv_l = sn.y;
      const int item = now;
      now = copy_next((i + 1) & 1);
      const bf16x8_t* rows = map_lds + ((i & 1) * HG + hg) * TILE;
      if (item == 1) {
#pragma unroll
        for (int st = 0; st < NS; ++st) kf[st] = rows[(kb * 32 + l32) * DCH + swz(kb * 32 + l32, 2 * st + hf)];
      } else if (item == 2 && live) {
        f32x16_t s = zero16;
#pragma unroll
        for (int st = 0; st < NS; ++st)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], rows[(qb * 32 + l32) * DCH + swz(qb * 32 + l32, 2 * st + hf)], s, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r >> 2][r & 3] += __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -m)) * inv_l;
      }
    }
    // the shares of the heads meet in LDS
    __syncthreads();
    f32x4_t* part = (f32x4_t*)map_lds + w4 * 256 + lane;
    if (hg > 0)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) part[(hg - 1) * 1024 + r4 * 64] = v[r4];
    __syncthreads();
    if (hg == 0)
#pragma unroll
      for (int p = 0; p < HG - 1; ++p)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) v[r4] += part[p * 1024 + r4 * 64];
  }
  // the tile as bf16 in LDS behind the sums, rows 16 bytes longer than a line, and from there in whole lines to memory
  bf16_t* tile = (bf16_t*)((char*)map_lds + (HG - 1) * 16384);
  if (hg == 0) {
    const float inv_h = 1.0f / (float)a.Hq;
    const int row = qb * 32 + l32, qi = q0 + row;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int col = kb * 32 + r4 * 8 + hf * 4;
      bf16x4_t o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)((j0 + col + e <= qi) ? v[r4][e] * inv_h : 0.f);
      *(bf16x4_t*)(tile + row * 72 + col) = o;
    }
  }
  __syncthreads();
  const int row = (int)threadIdx.x >> 3, col = ((int)threadIdx.x & 7) * 8;
  if (row >= 64 || q0 + row >= a.n) return;
  const bf16x8_t o = *(const bf16x8_t*)(tile + row * 72 + col);
  bf16_t* dst = a.a_out + (int64_t)(q0 + row) * a.ld + j0 + col;
  // n_cols is a multiple of 4; a pitch that is no multiple of 8, or a base off a 16-byte boundary, leaves rows at 8-byte addresses
  if (a.lines && j0 + col + 8 <= a.n_cols) *(bf16x8_t*)dst = o;
  else {
    if (j0 + col + 4 <= a.n_cols) *(bf16x4_t*)dst = bf16x4_t{o[0], o[1], o[2], o[3]};
    if (j0 + col + 8 <= a.n_cols) *(bf16x4_t*)(dst + 4) = bf16x4_t{o[4], o[5], o[6], o[7]};
  }
}

// The map of a short prompt: a workgroup makes 32 rows x 64 keys, wave w sums heads [w Hq / 8, (w + 1) Hq / 8) with the operands
// read straight from memory in operand layout, by 64-bit addresses.  Bound by latency: there is no copy to wait for and no
// barrier until the waves' sums meet, and twice as many workgroups as of 64 x 64 tiles.
// grid (query tiles of 32, key tiles of 64)
constexpr int kMapWaves = 8;
template <int DH>
__global__ __launch_bounds__(kMapWaves * 64) void k_attn_map_short(MapArgs a) {
  constexpr int NS = DH / 16;
  __shared__ f32x4_t part[kMapWaves][8][64];            // [wave][16-byte piece kb * 4 + r4][lane]
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int q0 = (int)blockIdx.x * 32, j0 = (int)blockIdx.y * 64;
  const bool visible = j0 <= q0 + 31;                   // else the tile lies above the diagonal: zeros
  if (!visible && a.lower) return;
  if (visible) {
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int qr = q0 + l32 < a.n ? q0 + l32 : a.n - 1;
    const int G = a.Hq / a.Hkv;
    const int h0 = a.Hq * wave / kMapWaves, h1 = a.Hq * (wave + 1) / kMapWaves;
    float acc[2][16];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[kb][r] = 0.f;
    bf16x8_t kf[2][NS], qn[NS];
    float2 sn = make_float2(0.f, 0.f);
    int g_of = -1;
    if (h0 < h1) {
      load_q_frags<DH>(a, qr, h0, hf, qn);
      sn = a.stats[(int64_t)h0 * a.n + qr];
    }
    for (int h = h0; h < h1; ++h) {
      bf16x8_t qf[NS];
#pragma unroll
      for (int st = 0; st < NS; ++st) qf[st] = qn[st];
      const float m = sn.x, inv_l = sn.y;
      if (h / G != g_of) {
        g_of = h / G;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const int key = j0 + kb * 32 + l32;
          load_k_frags<DH>(a, key < a.n ? key : a.n - 1, g_of, hf, kf[kb]);
        }
      }
      const int hn = h + 1 < h1 ? h + 1 : h;
      load_q_frags<DH>(a, qr, hn, hf, qn);
      sn = a.stats[(int64_t)hn * a.n + qr];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        f32x16_t s = zero16;
#pragma unroll
        for (int st = 0; st < NS; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb][st], qf[st], s, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kb][r] += __builtin_amdgcn_exp2f(fmaf(s[r], a.scale_log2, -m)) * inv_l;
      }
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        part[wave][kb * 4 + r4][lane] = f32x4_t{acc[kb][4 * r4], acc[kb][4 * r4 + 1], acc[kb][4 * r4 + 2], acc[kb][4 * r4 + 3]};
  }
  __syncthreads();
  // wave w finishes piece w: keys j0 + (w / 4) * 32 + (w % 4) * 8 + hf * 4 .. + 3 of row q0 + l32
  const int qi = q0 + l32;
  if (qi >= a.n) return;
  f32x4_t v = {0.f, 0.f, 0.f, 0.f};
  if (visible)
#pragma unroll
    for (int w = 0; w < kMapWaves; ++w) v += part[w][wave][lane];
  const float inv_h = 1.0f / (float)a.Hq;
  const int key0 = j0 + (wave >> 2) * 32 + (wave & 3) * 8 + hf * 4;
  bf16x4_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (bf16_t)((key0 + e <= qi) ? v[e] * inv_h : 0.f);
  if (key0 < a.n_cols) *(bf16x4_t*)(a.a_out + (int64_t)qi * a.ld + key0) = o;      // n_cols is a multiple of 4
}

template <int DH, int HG>
static fastav_status_t launch_map(const MapArgs& a, unsigned tiles, hipStream_t s) {
  // two stages of the rows per share; the sums and the bf16 tile at the end need less (16 KB a share but the first, 9 KB)
  constexpr int shmem = 2 * HG * 64 * DH * 2 > (HG - 1) * 16384 + 9216 ? 2 * HG * 64 * DH * 2 : (HG - 1) * 16384 + 9216;
  if constexpr (shmem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k_attn_map<DH, HG>, hipFuncAttributeMaxDynamicSharedMemorySize, shmem);
    if (e != hipSuccess) return fail(FASTAV_EHIP, "attention map: hipFuncSetAttribute: %s", hipGetErrorString(e));
  }
  hipLaunchKernelGGL((k_attn_map<DH, HG>), dim3(tiles), dim3(HG * 256), shmem, s, a);
  return check_launch("attention_map");
}

// Which of the two: the short form's time goes with the rows it reads (32 per head, 64 per key head and wave), that of the
// 64 x 64 tiles with their chain of copies (a quarter of the heads and of the key heads).  So heads of 64 are short up to 896
// tokens, heads of 128 up to 832 where there are fewer heads than waves or many to a key head.  fastav_attention_map with its
// statistics, us, short / tiles:
//   tokens            256          512          832          896          960
//   16/16 of 64    14.0 / 17.3  15.1 / 18.2  17.5 / 19.6  18.8 / 19.8  24.5 / 20.5
//   64/8  of 64    18.5 / 27.3  22.7 / 31.4  30.7 / 38.0  33.0 / 39.8  45.0 / 41.6
//   1/1   of 64     8.6 / 10.7   9.7 / 11.8  11.7 / 12.9  12.7 / 13.1  13.4 / 13.6
//   4/2   of 128   13.7 / 15.7  15.6 / 17.5  19.1 / 19.7  20.7 / 20.1  23.2 / 21.1
//   32/8  of 128   23.1 / 25.4  25.1 / 27.4  35.5 / 36.5  37.3 / 37.1  50.2 / 39.0
//   28/4  of 128   22.5 / 23.5  24.5 / 25.5  33.2 / 32.8  36.0 / 34.2  47.7 / 35.2
//   8/2   of 128   17.2 / 16.9  19.2 / 18.9  22.5 / 21.1  24.2 / 21.4  30.5 / 22.5
//   16/16 of 128   22.7 / 22.3  24.7 / 24.1  28.6 / 27.1  30.4 / 27.5  42.1 / 28.8
//   32/32 of 128   33.4 / 30.7  36.4 / 34.3  45.8 / 43.2  47.5 / 43.5  71.2 / 45.4
// Inside a rollout (a layer with all its launches, 512 tokens): 16/16 of 64 68.5 / 72.0, 32/8 of 128 162.7 / 165.5.
static bool map_is_short(int n, int Hq, int Hkv, int dh) {
  return dh == 64 ? n <= 896 : n <= 832 && (Hq < kMapWaves || (Hq >= 24 && Hq >= 4 * Hkv));
}

size_t attention_map_stats_bytes(int n, int Hq) { return align_up((size_t)n * Hq * 2 * sizeof(float), 256); }

fastav_status_t launch_attention_map(const void* q, int64_t q_stride, const void* k, int64_t k_stride, int n, int Hq,
                                     int Hkv, int dh, float2* stats, bool have_stats, void* a_out, int64_t ld, bool lower, hipStream_t s) {
  if (n == 0) return FASTAV_OK;
  if (dh != 64 && dh != 128) return fail(FASTAV_EUNSUPPORTED, "attention map: head_dim must be 64 or 128");
  if (q_stride % 8 || k_stride % 8 || (((uintptr_t)q | (uintptr_t)k) % 16) || n % 4 || ((uintptr_t)a_out % 8))
    return fail(FASTAV_EINVAL, "attention map: q, k must be 16-byte aligned with strides of 8 elements, n a multiple of 4");
  MapArgs a;
  a.q = (const bf16_t*)q; a.k = (const bf16_t*)k; a.qs = q_stride; a.ks = k_stride; a.n = n; a.Hq = Hq; a.Hkv = Hkv;
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
  a.stats = stats; a.a_out = (bf16_t*)a_out; a.ld = ld; a.n_cols = lower ? (n + 63) / 64 * 64 : n;
  a.lower = lower;
  a.lines = ld % 8 == 0 && (uintptr_t)a_out % 16 == 0;
  // the causal Q K^T products: once for the statistics, once for the map
  ProfScope prof(FASTAV_PROF_ATTENTION, (have_stats ? 1.0 : 2.0) * 2.0 * Hq * dh * (double)n * ((double)n + 1.0) * 0.5, s);
  const dim3 g1((unsigned)Hq, (unsigned)ceil_div(n, 64));
  if (!have_stats) {
    if (dh == 128) hipLaunchKernelGGL(k_attn_rowstats<128>, g1, dim3(kStatWaves * 64), 0, s, a);
    else hipLaunchKernelGGL(k_attn_rowstats<64>, g1, dim3(kStatWaves * 64), 0, s, a);
  }
  // the 64 x 64 tiles address the rows of a tile by 32-bit byte offsets from its first
  const bool wide = q_stride >= (1 << 25) || k_stride >= (1 << 25);
  if (wide || map_is_short(n, Hq, Hkv, dh)) {
    const dim3 g2((unsigned)ceil_div(n, 32), (unsigned)ceil_div(n, 64));
    if (dh == 128) hipLaunchKernelGGL(k_attn_map_short<128>, g2, dim3(kMapWaves * 64), 0, s, a);
    else hipLaunchKernelGGL(k_attn_map_short<64>, g2, dim3(kMapWaves * 64), 0, s, a);
    return check_launch("attention_map");
  }
  const unsigned nt = (unsigned)ceil_div(n, 64), below = nt * (nt + 1) / 2, g2 = lower ? below : nt * nt;
  const bool few = below <= 256;
  if (dh == 128) return few ? launch_map<128, 4>(a, g2, s) : launch_map<128, 2>(a, g2, s);
  return few ? launch_map<64, 4>(a, g2, s) : launch_map<64, 2>(a, g2, s);
}

// ---------------------------------------------------------------------------------------- rollout step
// rt [n][n] = I; its bf16 copy [ld][ld], zero beyond n
__global__ void k_rollout_init(float* __restrict__ rt, bf16_t* __restrict__ rt16, int n, int ld) {
  const int64_t total = (int64_t)ld * ld;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(i / ld), col = (int)(i % ld);
    const float v = (row == col && row < n) ? 1.f : 0.f;
    if (row < n && col < n) rt[(int64_t)row * n + col] = v;
    rt16[i] = (bf16_t)v;
  }
}

// RT <- alpha (RT A^T) + (1 - alpha) RT in one launch.  R and A are lower triangular, so RT is upper triangular: tile (I, J) of the
// product has J >= I and needs columns 64 I .. 64 J + 63 of RT's rows and A's rows only, a sixth of the n^3 of the full product.
//
// A workgroup makes a 64 x 64 tile, the longest sums first; its four waves take every fourth 64-wide slice of K for the
// whole tile, each through a 16 KB buffer of its own that is filled with the next slice (whole 128-byte lines) while
// the products of the present one run from registers: no barrier before the four sums meet in LDS.  What bounds it
// is the chain of the longest tiles (8 slices a wave at 2048 tokens, a copy's latency each) and 2 x 8 MB of operands into every L2.
// It reads RT and A rounded to bf16, adds in fp32, and writes RT and the next step's copy of it.  A row of A beyond n is
// uninitialised: it only meets columns that are not stored.
// 2048 tokens: 17 us, where the full product, the sum of its K shares and two elementwise passes took 55.
constexpr int kStepPiece = 66;                          // 16-byte words between the pieces of a sum: 16 rows' or columns' pieces in 16 slots
__global__ __launch_bounds__(256, 2) void k_rollout_step(float* __restrict__ rt, const bf16_t* __restrict__ rt16, const bf16_t* __restrict__ a16,
                                                         bf16_t* __restrict__ rt16_next, int n, int ld, float alpha) {
  extern __shared__ f32x4_t step_lds[];                 // [wave][16 * kStepPiece]; the first 16 KB of each are the wave's operand buffer
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // tiles at distance d = J - I from the diagonal, nt - d of them, d descending
  const int nt = ld / 64, b = (int)blockIdx.x;
  int t = (int)((sqrtf(1.0f + 8.0f * (float)b) - 1.0f) * 0.5f);
  while (t * (t + 1) / 2 > b) --t;
  while ((t + 1) * (t + 2) / 2 <= b) ++t;
  const int I = b - t * (t + 1) / 2, J = I + nt - 1 - t;
  const int i0 = I * 64, j0 = J * 64, slices = J - I + 1;

  // this thread's outputs: rows i0 + it * 16 + tid / 16, four columns from j0 + 4 (tid % 16); requested before the products
  const int orow = (int)threadIdx.x >> 4, oc = (int)threadIdx.x & 15;
  f32x4_t old[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int i = i0 + it * 16 + orow, j = j0 + 4 * oc;
    old[it] = (i < n && j < n) ? *(const f32x4_t*)(rt + (int64_t)i * n + j) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // operand buffer: 64 rows of A, then 64 rows of RT, 8 chunks of 16 bytes a row; the swizzle (on the global side) spreads the
  // 16 rows an operand read takes at a time over 16 slots
  auto swz = [](int row, int c) { return c ^ ((row >> 1) & 7); };
  const bf16x8_t* mine = (const bf16x8_t*)(step_lds + wave * 16 * kStepPiece);
  const uint32_t buf = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)mine;
  uint32_t voff[2];                                     // rows 8 i + lane / 8: the swizzle repeats every 16 rows
#pragma unroll
  for (int i = 0; i < 2; ++i) voff[i] = (uint32_t)(8 * i + lane / 8) * (uint32_t)ld * 2u + (uint32_t)swz(8 * i + lane / 8, lane & 7) * 16u;
  auto copy_slice = [&](int s) __attribute__((always_inline)) {
    const bf16_t* pa = a16 + (int64_t)j0 * ld + i0 + s * 64;
    const bf16_t* pr = rt16 + (int64_t)i0 * ld + i0 + s * 64;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      lds_copy16(pa + (int64_t)(i >> 1) * 16 * ld, voff[i & 1], buf + (uint32_t)i * 1024u);
      lds_copy16(pr + (int64_t)(i >> 1) * 16 * ld, voff[i & 1], buf + 8192u + (uint32_t)i * 1024u);
    }
  };
  f32x16_t acc[2][2];                                   // [ib][jb]: row i0 + 32 ib + l32, columns j0 + 32 jb + (r / 4) * 8 + hf * 4 + r % 4
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ib][jb][r] = 0.f;
  if (wave < slices) copy_slice(wave);
  for (int s = wave; s < slices; s += 4) {
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): the slice has landed
    asm volatile("" : : : "memory");
    bf16x8_t fa[2][4], fr[2][4];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int row = rb * 32 + l32;
        fa[rb][ks] = mine[row * 8 + swz(row, 2 * ks + hf)];
        fr[rb][ks] = mine[512 + row * 8 + swz(row, 2 * ks + hf)];
      }
    __builtin_amdgcn_s_waitcnt(0xC07F);                 // lgkmcnt(0): and is in registers
    asm volatile("" : : : "memory");
    if (s + 4 < slices) copy_slice(s + 4);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
          acc[ib][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[jb][ks], fr[ib][ks], acc[ib][jb], 0, 0, 0);
  }
  f32x4_t* part = step_lds + wave * 16 * kStepPiece;
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        part[((ib * 2 + jb) * 4 + r4) * kStepPiece + hf * 33 + l32] =
            f32x4_t{acc[ib][jb][4 * r4], acc[ib][jb][4 * r4 + 1], acc[ib][jb][4 * r4 + 2], acc[ib][jb][4 * r4 + 3]};
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int row = it * 16 + orow, i = i0 + row, j = j0 + 4 * oc;
    const int at = ((row >> 5) * 8 + (oc >> 1)) * kStepPiece + (oc & 1) * 33 + (row & 31);
    f32x4_t v = step_lds[at];
#pragma unroll
    for (int w = 1; w < 4; ++w) v += step_lds[w * 16 * kStepPiece + at];
    v = v * alpha + old[it] * (1.0f - alpha);
    if (j >= n) v = f32x4_t{0.f, 0.f, 0.f, 0.f};        // columns beyond n feed the next step's sums
    if (i >= n) continue;
    if (j < n) *(f32x4_t*)(rt + (int64_t)i * n + j) = v;
    *(bf16x4_t*)(rt16_next + (int64_t)i * ld + j) = bf16x4_t{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
  }
}

__global__ void k_iota(int32_t* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i;
}
fastav_status_t launch_iota(int32_t* p, int n, hipStream_t s) {
  if (n == 0) return FASTAV_OK;
  hipLaunchKernelGGL(k_iota, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s, p, n);
  return check_launch("iota");
}

int64_t rollout_pitch(int64_t n) { return (n + 63) / 64 * 64; }
fastav_status_t launch_rollout_init(float* rt, void* rt16, int n, hipStream_t s) {
  if (n == 0) return FASTAV_OK;
  hipLaunchKernelGGL(k_rollout_init, dim3(2048), dim3(256), 0, s, rt, (bf16_t*)rt16, n, (int)rollout_pitch(n));
  return check_launch("rollout_init");
}

// rt fp32 [n, n]; rt16 (its bf16 copy), a16 and rt16_next (the copy of the result) bf16 at rollout_pitch(n), a16's tiles at and
// below the diagonal written with zeros beyond n.  alpha = 0: every factor is the identity, nothing is launched.
fastav_status_t launch_rollout_step(float* rt, const void* rt16, const void* a16, void* rt16_next, int n, float alpha, hipStream_t s) {
  if (n == 0 || alpha == 0.f) return FASTAV_OK;
  if (n % 4) return fail(FASTAV_EINVAL, "rollout: n must be a multiple of 4");
  const int ld = (int)rollout_pitch(n), nt = ld / 64;
  constexpr int shmem = 4 * 16 * kStepPiece * 16;
  ProfScope prof(FASTAV_PROF_LINEAR_RESADD, (double)n * n * n / 3.0, s);
  hipError_t e = hipFuncSetAttribute((const void*)k_rollout_step, hipFuncAttributeMaxDynamicSharedMemorySize, shmem);
  if (e != hipSuccess) return fail(FASTAV_EHIP, "rollout: hipFuncSetAttribute: %s", hipGetErrorString(e));
  hipLaunchKernelGGL(k_rollout_step, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), shmem, s, rt, (const bf16_t*)rt16, (const bf16_t*)a16,
                     (bf16_t*)rt16_next, n, ld, alpha);
  return check_launch("rollout_step");
}

// ---- rollout threshold -> cut-off position (Section 2.2, Global pruning) -------------------------------------
// influence[j] = (1/n) sum_i R[i][j]: the mean of row j of the transposed product.  One wave per row.
__global__ __launch_bounds__(256) void k_rollout_influence(const float* __restrict__ rt, int n, float* __restrict__ influence) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const f32x4_t* p = (const f32x4_t*)(rt + (int64_t)row * n);
  float s0 = 0.f, s1 = 0.f;
  int i = lane;
  for (; i + 64 < n / 4; i += 128) {
    const f32x4_t a = p[i], b = p[i + 64];
    s0 += (a[0] + a[1]) + (a[2] + a[3]);
    s1 += (b[0] + b[1]) + (b[2] + b[3]);
  }
  if (i < n / 4) { const f32x4_t a = p[i]; s0 += (a[0] + a[1]) + (a[2] + a[3]); }
  float t = s0 + s1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, kWave);
  if (lane == 0) influence[row] = t / (float)n;
}
// cutoff = 1 + the last unprotected position whose influence reaches `threshold` uniform shares (influence * n >=
// threshold, in fp32), 0 if there is none.  One workgroup.
__global__ __launch_bounds__(1024) void k_rollout_cutoff(const float* __restrict__ influence, const uint8_t* __restrict__ prot,
                                                         int n, float threshold, int32_t* __restrict__ cutoff) {
  __shared__ int wave_best[16];
  int best = 0;
  for (int j = threadIdx.x; j < n; j += 1024)
    if (!prot[j] && influence[j] * (float)n >= threshold) best = j + 1;     // j ascends: the last hit stays
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { const int t = __shfl_xor(best, o, kWave); best = t > best ? t : best; }
  if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    int b = 0;
    for (int w = 0; w < 16; ++w) b = wave_best[w] > b ? wave_best[w] : b;
    cutoff[0] = b;
  }
}
fastav_status_t launch_rollout_cutoff(const float* rt, int n, const uint8_t* prot, float threshold, float* influence,
                                      int32_t* cutoff, hipStream_t s) {
  if (n % 4) return fail(FASTAV_EINVAL, "rollout: n must be a multiple of 4");
  if (n > 0) hipLaunchKernelGGL(k_rollout_influence, dim3((unsigned)ceil_div(n, 4)), dim3(256), 0, s, rt, n, influence);
  hipLaunchKernelGGL(k_rollout_cutoff, dim3(1), dim3(1024), 0, s, (const float*)influence, prot, n, threshold, cutoff);
  return check_launch("rollout_cutoff");
}

}  // namespace fastav
