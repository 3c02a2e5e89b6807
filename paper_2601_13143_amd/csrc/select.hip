// Top-k selection and compaction for the prune step (Section 2.2, "Fine pruning" / Eq. 4: the lowest-scoring
// share P of the tokens goes; global pruning keeps the earliest positions instead; the other strategies of
// Tables 2-3 - top attentive, top informative, random - are further orders of the same kernel).
//
//   k_select  one 1024-thread workgroup per sample.  The sample's order-preserving 32-bit keys live in LDS;
//             four 8-bit MSB-first radix passes (LDS histograms in eight copies, so that the narrow exponent range
//             of softmax scores does not serialise on one counter) find the k-th largest key; ties at
//             the threshold go to the lowest indices; one workgroup scan (two where the keys do not fit in
//             LDS) turns the keep flags into the ascending list of kept rows.  The positional orders need no
//             radix pass: all candidates tie, and the tie rule by rank in row order is the selection.
//             Integer work only, so the result is exact.
//   k_gather  dst[r] = src[keep_idx[r]] for several tensors in one launch, 16 bytes per lane.
#include "common.hpp"

namespace fastav {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelLdsKeys = 32768;          // samples up to this length keep their keys in LDS (128 KB)
constexpr int kSelMaxHeads = 128;           // most query heads the fused Eq. 4 finish holds (max, 1/sum) for

// fp32 -> unsigned key, larger key = better.  NaN ranks as -inf; -0.0 equals +0.0.
__device__ __forceinline__ uint32_t score_key(float s) {
  if (s != s) s = -INFINITY;
  if (s == 0.0f) s = 0.0f;
  const uint32_t u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over a wave, all lanes active: rows of 16 by shifts, then lane 15 of a row into the next row and lane
// 31 into the upper half.  In the vector ALU; through LDS (shuffles) it is a chain of six round trips.
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // row_bcast 15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // row_bcast 31 into rows 2 and 3
  return v;
}

// Exclusive prefix sum over the workgroup.  wave_tot must not be in use: a caller that scans twice takes two arrays.
__device__ __forceinline__ int block_exclusive_scan(int v, int* wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = wave_inclusive_sum(v);
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) base += w < wave ? wave_tot[w] : 0;
  return base + inc - v;
}

// 32-bit avalanche mix (xor-shift 16, multiply, xor-shift 13, multiply, xor-shift 16): the finishing step of the
// published MurmurHash3 hash, a bijection on 32-bit words.
__host__ __device__ __forceinline__ uint32_t mix32(uint32_t h) {
  h ^= h >> 16; h *= 0x85EBCA6Bu;
  h ^= h >> 13; h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}
constexpr uint32_t kGolden = 0x9E3779B9u;

uint32_t select_random_key(uint32_t seed, int layer) { return mix32(seed + kGolden * (uint32_t)(layer + 1)); }

// Key of candidate j (unprotected row) of sample b under the rule's order; never 0.
// Random order: the draw is the top 24 bits of mix32(mix32(key + G (b + 1)) + position id) as a fraction in
// [0, 1), ranked like a score, so that a token's draw does not depend on what was pruned before it.
__device__ __forceinline__ uint32_t cand_key_of(const SelectRule& r, float score, uint32_t sample_key, int row0, int n, int j) {
  switch (r.order) {
    case kSelHighScore: return score_key(score);
    case kSelLowScore: return score_key(-score);
    case kSelEarliest:
    case kSelLatest: return 1u;                                         // positional orders: decided by candidate rank, below
    default: {
      const uint32_t p = r.pos ? (uint32_t)r.pos[row0 + j] : (uint32_t)j;
      return score_key((float)(mix32(sample_key + p) >> 8) * 0x1p-24f);
    }
  }
}
__device__ __forceinline__ uint32_t cand_key(const SelectRule& r, const float* scores, uint32_t sample_key, int row0,
                                             int n, int j) {
  const bool by_score = r.order == kSelHighScore || r.order == kSelLowScore;
  return cand_key_of(r, by_score ? scores[row0 + j] : 0.f, sample_key, row0, n, j);
}

// Bound: latency - one workgroup per sample, so a chain of trips to memory and of barriers (1229 to 2248 rows and 28 to 32
// heads, kernel time in a prefill of one prompt: 16.7 -> 10.4 us; 2048 rows of given scores 12.3 -> 7.4).  Hence: the loads of the score
// finish run two steps ahead and start before the first barrier; the first digit is counted as the keys are made; a radix
// pass is two barriers, with the other histogram cleared meanwhile; and no loop is unrolled further than its loads ask for,
// because a prefill comes here once a layer and what it does not find in the instruction cache it waits for.
constexpr int kHistCopies = 8, kHistPitch = 256 + 4;       // copies by lane % 8, a digit's in different banks: scores share few top digits
template <bool KEYS_IN_LDS>
__global__ __launch_bounds__(kSelThreads) void k_select(const float* __restrict__ scores,
                                                        const uint8_t* __restrict__ prot,
                                                        const int32_t* __restrict__ cu,
                                                        const int32_t* __restrict__ cu_out,
                                                        int32_t* __restrict__ keep_idx, SelectRule rule, SelectBounds bounds) {
  extern __shared__ __align__(16) uint32_t keys[];                      // [n] when KEYS_IN_LDS; key 0 = protected (never a candidate)
  __shared__ __align__(16) int hist[2][kHistCopies][kHistPitch];
  __shared__ int wave_prot[kSelWaves], wave_a[kSelWaves], wave_b[kSelWaves];
  __shared__ uint32_t sh_prefix;
  __shared__ int sh_need;

  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool given = bounds.batch > 0;                    // prefix sums in the kernel arguments
  if (given && b == 0)
    for (int i = tid; i <= bounds.batch; i += kSelThreads) bounds.cu_out_dev[i] = bounds.cu_out[i];
  const int row0 = given ? bounds.cu[b] : cu[b], n = (given ? bounds.cu[b + 1] : cu[b + 1]) - row0;
  const int out0 = given ? bounds.cu_out[b] : cu_out[b], k_keep = (given ? bounds.cu_out[b + 1] : cu_out[b + 1]) - out0;
  if (n <= 0) return;
  const uint32_t sample_key = mix32(rule.key + kGolden * (uint32_t)(b + 1));
  const bool positional = rule.order == kSelEarliest || rule.order == kSelLatest;

  auto clear_hist = [&](int buf, int first, int threads) __attribute__((always_inline)) {
    for (int i = first; i < kHistCopies * kHistPitch / 4; i += threads) ((int4*)&hist[buf][0][0])[i] = int4{0, 0, 0, 0};
  };
  auto count_digit = [&](int buf, uint32_t digit) __attribute__((always_inline)) { atomicAdd(&hist[buf][lane % kHistCopies][digit], 1); };
  // one row: its key to LDS and into the first histogram; returns the wave's count of protected rows (all lanes are here)
  auto put_key = [&](int j, bool p, float score) __attribute__((always_inline)) -> int {
    if (j < n && KEYS_IN_LDS) {
      const uint32_t key = p ? 0u : cand_key_of(rule, score, sample_key, row0, n, j);
      keys[j] = key;
      if (key != 0u && !positional) count_digit(0, key >> 24);
    }
    return __popcll(__ballot(j < n && p));
  };

  // ---- load keys, count protected rows.  With the attention side output at hand (rule.logits: the last query
  // row's scaled logits per head, rule.ml: that row's (max, sum of exp) per head) Eq. 4 is finished right here -
  // s_j = 1/Hq sum_h exp(L[h][j] - m_h) / l_h, the terms added in head order exactly as k_score_finalize adds them
  // - and goes straight into the key array (and to rule.scores_out for the caller), which saves a launch per prune.
  int my_prot = 0;                                        // of the wave
  clear_hist(0, tid, kSelThreads);
  if (KEYS_IN_LDS && rule.logits != nullptr) {
    __shared__ float sh_ml[2 * kSelMaxHeads];
    for (int h = tid; h < rule.n_heads; h += kSelThreads) {
      const float* pm = rule.ml + ((int64_t)b * rule.n_heads + h) * 2;
      sh_ml[2 * h] = pm[0]; sh_ml[2 * h + 1] = 1.0f / pm[1];
    }
    // A step is sixteen heads of one row per lane; two steps are in flight (the planes of the heads are T floats apart, so
    // every load is a trip to L2 or beyond, and one workgroup has to cover the whole sample).
    constexpr int HB = 16;
    const int H = rule.n_heads, nb = (H + HB - 1) / HB;
    const int rounds = wave * 64 < n ? (n - wave * 64 + kSelThreads - 1) / kSelThreads : 0;
    float cur[HB], nxt[HB];
    bool p_cur = false, p_nxt = false;
    int q_ask = 0, h_ask = 0;                             // the next step to ask for
    auto ask = [&](float (&g)[HB], bool& p) __attribute__((always_inline)) {
      if (q_ask < rounds) {                               // wave-uniform
        int j = q_ask * kSelThreads + tid;
        j = j < n ? j : n - 1;
        const float* lp = rule.logits + row0 + j;
#pragma unroll
        for (int u = 0; u < HB; ++u) g[u] = lp[(int64_t)(h_ask + u < H ? h_ask + u : H - 1) * rule.T];
        p = prot[row0 + j] != 0;
        h_ask += HB;
        if (h_ask >= H) { h_ask = 0; ++q_ask; }
      }
    };
    ask(cur, p_cur);
    ask(nxt, p_nxt);
    __syncthreads();
    float sc = 0.f;
    int h0 = 0, q = 0;
#pragma nounroll
    for (int st = 0; st < rounds * nb; ++st) {
#pragma unroll
      for (int u = 0; u < HB; ++u)
        if (h0 + u < H) sc = fmaf(expf(cur[u] - sh_ml[2 * (h0 + u)]), sh_ml[2 * (h0 + u) + 1], sc);
      h0 += HB;
      if (h0 >= H) {
        const int j = q * kSelThreads + tid;
        sc = sc / (float)H;
        if (rule.scores_out && j < n) rule.scores_out[row0 + j] = sc;
        my_prot += put_key(j, p_cur, sc);
        sc = 0.f;
        h0 = 0;
        ++q;
      }
#pragma unroll
      for (int u = 0; u < HB; ++u) cur[u] = nxt[u];
      p_cur = p_nxt;
      ask(nxt, p_nxt);
    }
  } else {
    __syncthreads();
    const bool by_score = rule.order == kSelHighScore || rule.order == kSelLowScore;
    constexpr int U = 4;                                  // rows asked for at a time
    for (int j0 = wave * 64; j0 < n; j0 += U * kSelThreads) {
      bool p[U];
      float sc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int j = j0 + u * kSelThreads + lane;
        j = j < n ? j : n - 1;
        p[u] = prot[row0 + j] != 0;
        sc[u] = KEYS_IN_LDS && by_score ? scores[row0 + j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) my_prot += put_key(j0 + u * kSelThreads + lane, p[u], sc[u]);
    }
  }
  auto key_at = [&](int j) __attribute__((always_inline)) -> uint32_t {
    if (KEYS_IN_LDS) return keys[j];
    return prot[row0 + j] ? 0u : cand_key(rule, scores, sample_key, row0, n, j);
  };
  if (!KEYS_IN_LDS && !positional)
    for (int j = tid; j < n; j += kSelThreads) {
      const uint32_t key = key_at(j);
      if (key != 0u) count_digit(0, key >> 24);
    }
  if (lane == 0) wave_prot[wave] = my_prot;
  __syncthreads();
  int n_prot = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) n_prot += wave_prot[w];
  int need = k_keep - n_prot;                             // candidates to keep
  if (need < 0) need = 0;
  const int n_cand = n - n_prot;
  if (need > n_cand) need = n_cand;

  // ---- threshold: a row is kept if it is protected (key 0), if its key > prefix, or if its key == prefix and its rank among
  // such rows, in row order, lies in [eq_lo, eq_lo + need_eq).
  uint32_t prefix = need == 0 ? 0xFFFFFFFFu : 0u;         // no key reaches 0xFFFFFFFF; every candidate's exceeds 0 (need == n_cand)
  int need_eq = 0, eq_lo = 0;
  if (need > 0 && need < n_cand) {
    need_eq = need;
    if (positional) {
      // every candidate carries the same key: the first (earliest) or the last (latest) `need` of them in row order are
      // kept by the rank rule alone, no pass over the keys is needed
      prefix = 1u;
      eq_lo = rule.order == kSelLatest ? n_cand - need : 0;
    } else {
      // radix select of the largest `need` keys, a digit of eight bits at a time from the top
      uint32_t mask = 0;
#pragma nounroll
      for (int shift = 24; shift >= 0; shift -= 8) {
        const int buf = (shift >> 3) & 1 ? 0 : 1;
        if (shift < 24) {
          for (int j = tid; j < n; j += kSelThreads) {
            const uint32_t key = key_at(j);
            if (key != 0u && (key & mask) == prefix) count_digit(buf, (key >> shift) & 255u);
          }
          __syncthreads();
        }
        if (wave == 0) {
          // lane owns digits 252 - 4 lane .. + 3, so that lanes count from the top digit down
          int4 c = {0, 0, 0, 0};
#pragma unroll
          for (int w = 0; w < kHistCopies; ++w) {
            const int4 t = *(const int4*)&hist[buf][w][252 - 4 * lane];
            c.x += t.x; c.y += t.y; c.z += t.z; c.w += t.w;
          }
          const int mine = c.x + c.y + c.z + c.w, inc = wave_inclusive_sum(mine);
          int above = inc - mine;                           // keys with a digit of a lower lane
          // the lane whose range crosses need_eq finds the digit
          if (above < need_eq && need_eq <= inc) {
            int d = 3;
            if (above + c.w < need_eq) { above += c.w; d = 2;
              if (above + c.z < need_eq) { above += c.z; d = 1;
                if (above + c.y < need_eq) { above += c.y; d = 0; } } }
            sh_prefix = prefix | ((uint32_t)(252 - 4 * lane + d) << shift);
            sh_need = need_eq - above;                     // still to take among keys with this digit
          }
        } else {
          clear_hist(buf ^ 1, tid - 64, kSelThreads - 64);  // last read two barriers ago
        }
        __syncthreads();
        prefix = sh_prefix;
        need_eq = sh_need;
        mask |= 255u << shift;
      }
    }
  }

  // ---- flags and ordered output.  Thread t owns the contiguous rows [t*per, (t+1)*per).
  if constexpr (KEYS_IN_LDS) {
    // 16 bytes per read.  `per` is an odd number of such pieces: every thread starts on a 16-byte boundary and a wave's lanes
    // read 16 different slots (at an even number they meet in a few banks, all of them in two at 32 rows a thread: 33 samples of
    // 16384 / 30000 / 32768 rows by position 18.9 / 39.5 / 42.3 -> 16.5 / 26.5 / 27.6 us, by score 23.9 / 49.0 / 52.5 ->
    // 22.2 / 35.2 / 36.8).  One scan carries both running counts: the rows kept for sure (protected, or above the threshold) in
    // the low half and the rows equal to the threshold in the high half - either total is at most kSelLdsKeys = 2^15, so the
    // halves do not run into each other.
    static_assert(kSelLdsKeys <= 32768, "packed scan");
    const int per = 4 * ((n + 4 * kSelThreads - 1) / (4 * kSelThreads) | 1);
    const int j_lo = tid * per, j_hi = j_lo + per < n ? j_lo + per : n;
    auto read4 = [&](uint32_t (&k4)[4], int j) __attribute__((always_inline)) {
      if (j + 3 < n) {
        const uint4 v = *(const uint4*)(keys + j);
        k4[0] = v.x; k4[1] = v.y; k4[2] = v.z; k4[3] = v.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) k4[e] = j + e < n ? keys[j + e] : 0u;
      }
    };
    uint32_t counts = 0;
#pragma nounroll
    for (int j = j_lo; j < j_hi; j += 4) {
      uint32_t k4[4];
      read4(k4, j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j + e < n) counts += k4[e] == 0u || k4[e] > prefix ? 1u : k4[e] == prefix ? 0x10000u : 0u;
    }
    const uint32_t before = (uint32_t)block_exclusive_scan((int)counts, wave_a);
    const int eq_before = (int)(before >> 16), sure_before = (int)(before & 0xFFFFu);
    const int eq_kept_before = eq_before - eq_lo < 0 ? 0 : (eq_before - eq_lo < need_eq ? eq_before - eq_lo : need_eq);
    int e_rank = eq_before, o = sure_before + eq_kept_before;
#pragma nounroll
    for (int j = j_lo; j < j_hi; j += 4) {
      uint32_t k4[4];
      read4(k4, j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bool keep = k4[e] == 0u || k4[e] > prefix;
        if (!keep && k4[e] == prefix) { keep = e_rank >= eq_lo && e_rank < eq_lo + need_eq; ++e_rank; }
        if (j + e < n && keep) {
          if (o < k_keep) keep_idx[out0 + o] = row0 + j + e;   // o < k_keep always unless k_keep < #protected
          ++o;
        }
      }
    }
  } else {
    const int per = (n + kSelThreads - 1) / kSelThreads;
    const int j_lo = tid * per, j_hi = (j_lo + per < n) ? j_lo + per : n;
    auto keeps = [&](uint32_t key, int& e) __attribute__((always_inline)) -> bool {
      if (key == 0u || key > prefix) return true;
      if (key == prefix) { const bool kp = e >= eq_lo && e < eq_lo + need_eq; ++e; return kp; }
      return false;
    };
    int eq_cnt = 0;
    for (int j = j_lo; j < j_hi; ++j) {
      const uint32_t key = key_at(j);
      eq_cnt += (key != 0u && key == prefix) ? 1 : 0;
    }
    const int eq_before = block_exclusive_scan(eq_cnt, wave_a);
    int keep_cnt = 0;
    {
      int e = eq_before;
      for (int j = j_lo; j < j_hi; ++j) keep_cnt += keeps(key_at(j), e) ? 1 : 0;
    }
    const int keep_before = block_exclusive_scan(keep_cnt, wave_b);
    int e = eq_before, o = keep_before;
    for (int j = j_lo; j < j_hi; ++j) {
      if (keeps(key_at(j), e)) {
        if (o < k_keep) keep_idx[out0 + o] = row0 + j;     // o < k_keep always unless k_keep < #protected
        ++o;
      }
    }
  }
}

// Every sample whose keys fit LDS has its score finished here.  That is a launch less, worth 1 to 4 us up to about 1000 rows;
// beyond, one workgroup reading all heads' logits costs more than the launch saves, now that the selection on given scores
// is short.  A prune of one prompt in a prefill, separate launches against this one, us:
//   rows             331   512  1024  1350  1700  2048  3000  4096  8192  16384
//    8 heads of 128 +3.9  +3.1  +1.6  +0.9  +0.2  -0.5  -3.2  -4.5   -13    -32
//   28              +2.4  +2.7  +1.1  -1.6  -3.6  -4.8   -11   -15   -34    -86
//   32              +3.1  +3.0  +0.7  -3.1  -3.5  -5.5   -11   -15   -39    -93
//   64              +3.8  +3.8  -0.6  -5.3  -8.4   -13   -23   -36   -87   -260
// The line is not drawn there: it is where the kernel's LDS ends.
bool select_fuses_score(int max_seqlen, int n_heads) { return max_seqlen <= kSelLdsKeys && n_heads >= 1 && n_heads <= kSelMaxHeads; }

fastav_status_t launch_select(const float* scores, const uint8_t* prot, const int32_t* cu, const int32_t* cu_out,
                              int batch, int max_seqlen, int32_t* keep_idx, double bytes_hint, hipStream_t s,
                              SelectRule rule, const SelectBounds& bounds) {
  if (batch == 0 || (max_seqlen == 0 && bounds.batch == 0)) return FASTAV_OK;
  if ((rule.order == kSelHighScore || rule.order == kSelLowScore) && !scores && !rule.logits) return fail(FASTAV_EINVAL, "select: this order needs scores");
  if (rule.logits && (max_seqlen > kSelLdsKeys || rule.n_heads > kSelMaxHeads || rule.n_heads < 1 || !rule.ml))
    return fail(FASTAV_EUNSUPPORTED, "select: the fused score finish needs samples of at most %d rows and at most %d heads", kSelLdsKeys, kSelMaxHeads);
  ProfScope prof(FASTAV_PROF_SELECT, bytes_hint, s);
  if (max_seqlen <= kSelLdsKeys) {
    const size_t shmem = (size_t)max_seqlen * sizeof(uint32_t);
    if (shmem > 32 * 1024) {   // beyond the default dynamic-LDS limit: opt in (per device, so set on every such launch)
      hipError_t e = hipFuncSetAttribute((const void*)k_select<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         kSelLdsKeys * (int)sizeof(uint32_t));
      if (e != hipSuccess) return fail(FASTAV_EHIP, "select: hipFuncSetAttribute: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(k_select<true>, dim3((unsigned)batch), dim3(kSelThreads), shmem, s, scores, prot, cu, cu_out, keep_idx, rule, bounds);
  } else {
    hipLaunchKernelGGL(k_select<false>, dim3((unsigned)batch), dim3(kSelThreads), 0, s, scores, prot, cu, cu_out, keep_idx, rule, bounds);
  }
  return check_launch("select");
}

// ---------------------------------------------------------------------------------------- gather
struct GatherArgs {
  const char* src[FASTAV_MAX_GATHER_TENSORS];
  char* dst[FASTAV_MAX_GATHER_TENSORS];
  int64_t row_bytes[FASTAV_MAX_GATHER_TENSORS];
  int64_t src_stride[FASTAV_MAX_GATHER_TENSORS];
  int64_t dst_stride[FASTAV_MAX_GATHER_TENSORS];   // bytes between destination rows (row_bytes when packed)
};

// grid (row groups, tensor).  Rows whose size and addresses are multiples of 16 bytes move as uint4 with
// the workgroup's lanes laid along the row; anything else moves bytewise.  idx == nullptr copies rows in
// place order (a strided copy).
__global__ __launch_bounds__(256) void k_gather(GatherArgs a, const int32_t* __restrict__ idx, int64_t n_rows,
                                                int rows_per_block) {
  const int t = blockIdx.y;
  const int64_t rb = a.row_bytes[t];
  const int64_t ss = a.src_stride[t], ds = a.dst_stride[t];
  const char* src = a.src[t];
  char* dst = a.dst[t];
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const bool vec = ((rb | ss | ds) % 16 == 0) && (((uintptr_t)src | (uintptr_t)dst) % 16 == 0);
  if (vec) {
    const int64_t v_per_row = rb / 16;
    const int64_t total = v_per_row * rows_per_block;
    for (int64_t i = threadIdx.x; i < total; i += 256) {
      const int64_t r = r0 + i / v_per_row, c = i % v_per_row;
      if (r >= n_rows) break;
      const int64_t sr = idx ? (int64_t)idx[r] : r;
      ((uint4*)(dst + r * ds))[c] = ((const uint4*)(src + sr * ss))[c];
    }
  } else {
    const int64_t total = rb * rows_per_block;
    for (int64_t i = threadIdx.x; i < total; i += 256) {
      const int64_t r = r0 + i / rb, c = i % rb;
      if (r >= n_rows) break;
      const int64_t sr = idx ? (int64_t)idx[r] : r;
      dst[r * ds + c] = src[sr * ss + c];
    }
  }
}

static fastav_status_t gather_impl(const GatherArgs& a, int n_tensors, const int32_t* keep_idx, int64_t n_rows,
                                   int prof_kind, hipStream_t s) {
  if (n_rows == 0 || n_tensors == 0) return FASTAV_OK;
  double bytes = keep_idx ? 4.0 * n_rows : 0.0;
  for (int i = 0; i < n_tensors; ++i) bytes += 2.0 * a.row_bytes[i] * n_rows;
  ProfScope prof(prof_kind, bytes, s);
  // aim at >= 4 KB of payload per workgroup, judged by the widest tensor
  int64_t widest = 1;
  for (int i = 0; i < n_tensors; ++i) widest = a.row_bytes[i] > widest ? a.row_bytes[i] : widest;
  int rows_per_block = (int)(4096 / widest);
  if (rows_per_block < 1) rows_per_block = 1;
  if (rows_per_block > 64) rows_per_block = 64;
  dim3 grid((unsigned)ceil_div(n_rows, rows_per_block), (unsigned)n_tensors);
  hipLaunchKernelGGL(k_gather, grid, dim3(256), 0, s, a, keep_idx, n_rows, rows_per_block);
  return check_launch("gather");
}

fastav_status_t launch_gather(const GatherTensor* t, int n_tensors, const int32_t* keep_idx, int64_t n_rows,
                              hipStream_t s) {
  if (n_tensors > FASTAV_MAX_GATHER_TENSORS) return fail(FASTAV_EINVAL, "gather: too many tensors");
  GatherArgs a;
  int m = 0;
  for (int i = 0; i < n_tensors; ++i) {
    if (t[i].row_bytes == 0) continue;
    a.src[m] = (const char*)t[i].src; a.dst[m] = (char*)t[i].dst;
    a.row_bytes[m] = t[i].row_bytes; a.src_stride[m] = t[i].src_stride_bytes ? t[i].src_stride_bytes : t[i].row_bytes;
    a.dst_stride[m] = t[i].row_bytes; ++m;
  }
  for (int i = m; i < FASTAV_MAX_GATHER_TENSORS; ++i) { a.src[i] = nullptr; a.dst[i] = nullptr; a.row_bytes[i] = 0; a.src_stride[i] = 0; a.dst_stride[i] = 0; }
  // without an index this is a plain copy (KV-cache write), timed apart from the prune-step gathers
  return gather_impl(a, m, keep_idx, n_rows, keep_idx ? FASTAV_PROF_GATHER : FASTAV_PROF_OTHER, s);
}

fastav_status_t launch_copy_rows(const void* src, int64_t src_row_bytes_stride, void* dst, int64_t row_bytes,
                                 int64_t rows, const int32_t* idx, hipStream_t s, int64_t dst_row_bytes_stride) {
  GatherArgs a;
  for (int i = 0; i < FASTAV_MAX_GATHER_TENSORS; ++i) { a.src[i] = nullptr; a.dst[i] = nullptr; a.row_bytes[i] = 0; a.src_stride[i] = 0; a.dst_stride[i] = 0; }
  a.src[0] = (const char*)src; a.dst[0] = (char*)dst; a.row_bytes[0] = row_bytes; a.src_stride[0] = src_row_bytes_stride;
  a.dst_stride[0] = dst_row_bytes_stride ? dst_row_bytes_stride : row_bytes;
  // plain row copies (KV-cache writes, outputs) are not part of a prune step: they are timed as "other"
  return gather_impl(a, 1, idx, rows, idx ? FASTAV_PROF_GATHER : FASTAV_PROF_OTHER, s);
}

}  // namespace fastav
