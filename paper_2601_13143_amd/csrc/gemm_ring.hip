// bf16 linear layers of few rows (a short prompt, or the layers behind the prunes): C = A W^T with A [M, K], W [N, K].
//
// Bound: the weights' way from HBM, until about 200 rows; beyond, LDS and the stage's barrier (331 rows of 18944 x 3584
// gate/up, tiles of 384 x 160: 13 operand reads to 30 matrix instructions; a third slot for the weights' stages changes
// nothing, so it is not their latency).  So a workgroup keeps a deep ring of stages (64 of K) in flight instead of the two of the large
// tiles, its rows are cut to a multiple of 64 close to M, and its columns or its share of K are cut so that one round of
// workgroups covers the chip.
//
// A stage's operands travel to LDS with asynchronous 16-byte-per-lane copies, 8 rows x 128 contiguous bytes each, into
// slot (stage mod NS); the one barrier of a stage publishes stage t and frees the slot of stage t-1, which takes the
// copies of stage t + NS - 1 (t + NS where the next k-step's operands are read ahead).  A wave owns TM blocks of 16 rows and all BN columns of the tile; with KS = 2 the two k-steps of a stage
// go to two waves (the second wave of a SIMD covers the first one's LDS reads), whose sums meet in LDS at the end.
// A wave that spans all columns holds every pair the epilogues need in one lane: gate and up (the tile's weight rows
// alternate 16 gate, 16 up) and the two halves of a rotated head.
#include "gemm_mfma.hpp"

namespace fastav {

// Weight row (column of the product) that tile column c of the tile at n0 holds.  A 64-column tile of a projection with
// rotated heads of 128 takes 32 columns of either half of the head, [32 h, 32 h + 32) and 64 columns further on.
__device__ __forceinline__ int ring_col(int n0, int c, bool half_heads) {
  if (!half_heads) return n0 + c;
  return (n0 & ~127) + 32 * ((n0 >> 6) & 1) + (c & 31) + ((c & 32) << 1);
}

template <int BM, int BN, int TM, int KS, int NS, int EPI, bool ROT>
__global__ __launch_bounds__(BM / (16 * TM) * KS * 64) void k_gemm_ring(GemmArgs g) {
  constexpr int WM = BM / (16 * TM), NW = WM * KS;
  constexpr int TN = BN / 16;
  constexpr int GROUPS = (BM + BN) / 8;                 // 8-row copy instructions per stage
  constexpr int D = (GROUPS + NW - 1) / NW;             // of the first `FULL` waves; the others issue D - 1
  constexpr int FULL = GROUPS - (D - 1) * NW;
  constexpr int SLOT = (BM + BN) * 128;                 // bytes
  static_assert(KS == 1 || KS == 2, "a stage has two k-steps");
  extern __shared__ bf16x8_t lds[];

  // ---- tile: every XCD owns a contiguous run of (K share, tile column, tile row), rows innermost: the tile rows that
  // read one weight panel, and the tile columns that read one activation panel, meet in its L2
  const int tiles = g.tiles_m * g.tiles_n, nblk = tiles * g.splits;
  int pid = blockIdx.x;
  {
    const int per = nblk / 8, rem = nblk % 8, xcd = pid % 8, idx = pid / 8;
    pid = xcd * per + (xcd < rem ? xcd : rem) + idx;
  }
  const int split = pid / tiles, tile = pid - split * tiles;
  const int tile_n = tile / g.tiles_m, tile_m = tile - tile_n * g.tiles_m;
  const int m0 = tile_m * BM;
  const int n0 = tile_n * (EPI == FASTAV_EPI_SWIGLU ? BN / 2 : BN);

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wk = wave / WM;
  const int K = g.K;
  const int kt_all = K / 64;
  const int kt0 = (int)((int64_t)kt_all * split / g.splits);
  const int KT = (int)((int64_t)kt_all * (split + 1) / g.splits) - kt0;

  // Where this workgroup starts its walk of K (launch_ring).
  const int rot = ROT ? (int)((int64_t)tile_n * KT / g.tiles_n) : 0;

  const bf16_t* wbase = g.W[0];
  int seg_start = 0, seg = 0;
  if (EPI == FASTAV_EPI_STORE) {
    if (n0 >= g.seg_end[0]) { wbase = g.W[1]; seg_start = g.seg_end[0]; seg = 1; }
    if (n0 >= g.seg_end[1]) { wbase = g.W[2]; seg_start = g.seg_end[1]; seg = 2; }
  }
  const bool rope = EPI == FASTAV_EPI_STORE && g.rope_tab != nullptr && seg < g.rope_segs;
  const bool half_heads = rope && g.rope_dh == 128;
  const int nb = n0 - seg_start;

  // ---- this wave's copies: instruction c covers rows [8 (c NW + wave), +8) of the slot (A's rows, then B's)
  const int drow = lane >> 3, dpos = lane & 7;
  const int nd = wave < FULL ? D : D - 1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  u32x4_t rs[D];
  uint32_t vo[D];
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const int r0 = (c * NW + wave) * 8;
    const int row = r0 + drow;
    const bf16_t* base;
    int64_t src;
    if (r0 < BM) {
      const int grow = m0 + row < g.M ? m0 + row : g.M - 1;        // clamped rows are not stored
      base = g.A;
      src = g.a_rows ? g.a_rows[grow] : grow;
    } else {
      const int b0 = r0 - BM, b = b0 + drow;
      if (EPI == FASTAV_EPI_SWIGLU) {
        const int blk = b0 >> 4;                                   // 8 rows lie inside one block of 16
        const int j = n0 + (blk >> 1) * 16 + (b & 15);
        base = (blk & 1) ? g.W2 : g.W[0];
        src = j < g.N ? j : g.N - 1;
      } else {
        base = wbase;
        const int j = ring_col(nb, b, half_heads);
        src = seg_start + j < g.N ? j : g.N - 1 - seg_start;
      }
    }
    rs[c] = make_rsrc(base + kt0 * 64);
    vo[c] = ((uint32_t)src * (uint32_t)K + (uint32_t)(dpos ^ ((row >> 1) & 7)) * 8u) * 2u;
  }
  auto copies = [&](int t, int slot) __attribute__((always_inline)) {   // past the last stage: the last one again, unread
    int at = (t < KT ? t : KT - 1) + rot;
    if (ROT && at >= KT) at -= KT;
    const uint32_t so = (uint32_t)(at * 128);
    const uint32_t dst = lds0 + (uint32_t)slot * SLOT + (uint32_t)wave * 1024u;
#pragma unroll
    for (int c = 0; c < D; ++c)
      if (c < D - 1 || FULL == NW || nd == D) dma16_buf(rs[c], vo[c], so, dst + (uint32_t)(c * NW) * 1024u);
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int frow = lane & 15, fch = lane >> 4;

  auto read_step = [&](int slot, int ks, bf16x8_t (&af)[TM], bf16x8_t (&bf)[TN]) __attribute__((always_inline)) {
    const bf16x8_t* sl = lds + slot * (SLOT / 16);
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = sl[swz8(wm * 16 * TM + frow, ks * 4 + fch) + i * 128];
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[j] = sl[BM * 8 + swz8(frow, ks * 4 + fch) + j * 128];
  };
  auto multiply = [&](const bf16x8_t (&af)[TM], const bf16x8_t (&bf)[TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
  };
  // PIPED: the operands of a k-step are read while the one before it is multiplied, a read behind every few matrix instructions;
  // stage t's barrier publishes stage t + 1 and, every wave having read stage t, frees its slot for stage t + NS.  With a wave per
  // SIMD and two k-steps a stage the reads stood alone at the head of each: gate/up of 200 rows 83 -> 71 (3584 x 37888) and
  // 75 -> 65 us, 331 rows 106 -> 102, down of 200 rows 48 -> 46 and 44 -> 42.  Projections of up to 128-row tiles gain where
  // the weights' stream leaves room (82 rows, Q|K|V 20.5 -> 18.2 and 23.0 -> 20.2); the other tiles of two k-steps to two waves
  // have no registers for a second set of operands (192 x 160 spills: 66 -> 180 us) or lose a percent.
  constexpr bool PIPED = KS == 1 || (EPI == FASTAV_EPI_STORE && TN == 4 && BM <= 128);
  auto interleave = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < TM + TN; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN / (TM + TN), 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(TM * TN >= TM + TN, "at least one matrix instruction to a read");
  int slot = 0;
  auto next_stage = [&](int t) __attribute__((always_inline)) {
    // stage t + 1 has landed when only the copies of the NS - 2 stages behind it are in flight
    if (FULL == NW || nd == D) dma_wait_keep<(NS - 2) * D>(); else dma_wait_keep<(NS - 2) * (D - 1)>();
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    __syncthreads();
    copies(t + NS, slot);
    slot = slot + 1 == NS ? 0 : slot + 1;
  };
  bf16x8_t a0[TM], b0[TN], a1[TM], b1[TN];
  if constexpr (PIPED) {
#pragma unroll
    for (int t = 0; t < NS; ++t) copies(t, t);
    if (FULL == NW || nd == D) dma_wait_keep<(NS - 1) * D>(); else dma_wait_keep<(NS - 1) * (D - 1)>();
    __syncthreads();
    read_step(0, wk, a0, b0);
  }
  if constexpr (KS == 1) {
#pragma unroll 1
    for (int t = 0; t < KT; ++t) {
      read_step(slot, 1, a1, b1);
      multiply(a0, b0);
      interleave();
      next_stage(t);
      read_step(slot, 0, a0, b0);                                  // behind the last stage: a repeated one, not multiplied
      multiply(a1, b1);
      interleave();
    }
  } else if constexpr (PIPED) {
    int t = 0;
#pragma unroll 1
    for (; t + 1 < KT; t += 2) {
      next_stage(t);
      read_step(slot, wk, a1, b1);
      multiply(a0, b0);
      interleave();
      next_stage(t + 1);
      read_step(slot, wk, a0, b0);
      multiply(a1, b1);
      interleave();
    }
    if (t < KT) multiply(a0, b0);
  } else {
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) copies(t, t);
    int fill = NS - 1;
#pragma unroll 1
    for (int t = 0; t < KT; ++t) {
      // stage t has landed when only the copies of the NS - 2 stages behind it are in flight
      if (FULL == NW || nd == D) dma_wait_keep<(NS - 2) * D>(); else dma_wait_keep<(NS - 2) * (D - 1)>();
      asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");         // and stage t - 1 has been read
      __syncthreads();
      copies(t + NS - 1, fill);
      read_step(slot, wk, a0, b0);
      multiply(a0, b0);
      slot = slot + 1 == NS ? 0 : slot + 1;
      fill = fill + 1 == NS ? 0 : fill + 1;
    }
  }

  if constexpr (KS == 2) {
    static_assert(WM * TM * TN * 1024 <= NS * SLOT, "the second k-step's sums fit LDS");
    dma_wait_keep<0>();
    __syncthreads();
    f32x4_t* x = (f32x4_t*)lds + wm * (TM * TN * 64) + lane;
    if (wk == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) x[(i * TN + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (wk == 1) return;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += x[(i * TN + j) * 64];
  } else {
    dma_wait_keep<0>();
  }

  // ---- epilogue.  A quad is columns 4 (lane / 16) .. of the 16-column block, row lane % 16 of the 16-row block
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const int mr = lane & 15, c4 = (lane >> 4) * 4;
  auto put_bf16 = [&](bf16_t* p, const float (&v)[4]) __attribute__((always_inline)) {
    if (g.vec_ok) {
      *(u32x2_t*)p = u32x2_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = (bf16_t)v[r];
    }
  };
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = m0 + wm * 16 * TM + i * 16 + mr;
    if (row >= g.M) continue;
    if constexpr (EPI == FASTAV_EPI_SWIGLU) {
      bf16_t* C = (bf16_t*)g.C + (int64_t)row * g.ldc + n0 + c4;
#pragma unroll
      for (int p = 0; p < TN / 2; ++p) {
        if (n0 + p * 16 >= g.N) break;                             // N is a multiple of 16
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float gt = acc[i][2 * p][r];
          v[r] = gt / (1.0f + __expf(-gt)) * acc[i][2 * p + 1][r];
        }
        put_bf16(C + p * 16, v);
      }
    } else if constexpr (EPI == FASTAV_EPI_STORE) {
      bf16_t* C = g.seg_out ? (bf16_t*)g.Cs[seg] + (int64_t)row * g.ldcs[seg] : (bf16_t*)g.C + (int64_t)row * g.ldc + seg_start;
      if (rope) {
        static_assert(TN == 4, "a tile is 64 columns: 32 of either half of a head");
        const int half = g.rope_dh >> 1;
        const float2* tr = g.rope_tab + (int64_t)g.rope_pos[row] * half + (half_heads ? 32 * ((nb >> 6) & 1) : 0) + c4;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4_t t01 = *(const f32x4_t*)(tr + j * 16), t23 = *(const f32x4_t*)(tr + j * 16 + 2);
          const float cs[4] = {t01[0], t01[2], t23[0], t23[2]}, sn[4] = {t01[1], t01[3], t23[1], t23[3]};
          float v1[4], v2[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x1 = acc[i][j][r], x2 = acc[i][j + 2][r];
            v1[r] = x1 * cs[r] - x2 * sn[r];
            v2[r] = x2 * cs[r] + x1 * sn[r];
          }
          put_bf16(C + ring_col(nb, j * 16, half_heads) + c4, v1);
          put_bf16(C + ring_col(nb, j * 16 + 32, half_heads) + c4, v2);
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
          put_bf16(C + nb + j * 16 + c4, v);
        }
      }
    } else {
      float* C = EPI == kEpiPartial ? g.partial + ((int64_t)split * g.M + row) * g.N + n0 + c4 : (float*)g.C + (int64_t)row * g.ldc + n0 + c4;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if (g.vec_ok) {
          f32x4_t v = acc[i][j];
          if (EPI == FASTAV_EPI_RESADD) v += *(const f32x4_t*)(C + j * 16);
          *(f32x4_t*)(C + j * 16) = v;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (EPI == FASTAV_EPI_RESADD) C[j * 16 + r] += acc[i][j][r];
            else C[j * 16 + r] = acc[i][j][r];
          }
        }
      }
    }
  }
}

template <int BM, int BN, int TM, int KS, int NS, int EPI, bool ROT>
static fastav_status_t launch_ring(const GemmArgs& g, hipStream_t s) {
  constexpr int shmem = NS * (BM + BN) * 128;
  hipError_t e = hipFuncSetAttribute((const void*)k_gemm_ring<BM, BN, TM, KS, NS, EPI, ROT>, hipFuncAttributeMaxDynamicSharedMemorySize, shmem);
  if (e != hipSuccess) return fail(FASTAV_EHIP, "gemm: hipFuncSetAttribute: %s", hipGetErrorString(e));
  hipLaunchKernelGGL((k_gemm_ring<BM, BN, TM, KS, NS, EPI, ROT>), dim3((unsigned)(g.tiles_m * g.tiles_n * g.splits)), dim3(BM / (16 * TM) * KS * 64), shmem, s, g);
  return check_launch("gemm_ring");
}
template <int BM, int BN, int TM, int KS, int NS, int EPI>
static fastav_status_t launch_ring(GemmArgs g, int splits, hipStream_t s) {
  constexpr int OUT_BN = EPI == FASTAV_EPI_SWIGLU ? BN / 2 : BN;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.N + OUT_BN - 1) / OUT_BN;
  g.splits = splits;
  // Gate and up rows at a pitch of whole 4 KB, every workgroup at the same k: the rows then meet in a few memory channels, so
  // each tile column starts its walk of K elsewhere, evenly over K.  us, all at the same k / spread, 17 / 48 / 82 / 117 / 166 / 256
  // rows of 28672 x 4096: 52.5 / 51.5 / 48.9 / 52.2 / 61.4 / 68 -> 43.9 / 44.3 / 47.2 / 50.3 / 58.8 / 67; 48 rows of
  // 16384 x 2048 16.5 -> 15.0; five stages further a column instead: 64 rows of 28672 x 4096 45.5 -> 47.0, spread 44.5.  Rows of
  // other pitches, the other products and the large tiles gain nothing.  Not with several tile rows: they share a panel of
  // weights in L2 while they walk it together (each workgroup elsewhere: 8192 x 8192, 300 rows 62 -> 103, 2048 x 4096, 576 rows
  // 24 -> 27; each tile column elsewhere: 24.7).
  if constexpr (EPI == FASTAV_EPI_SWIGLU)
    if (g.K % 2048 == 0 && g.tiles_m == 1) return launch_ring<BM, BN, TM, KS, NS, EPI, true>(g, s);
  return launch_ring<BM, BN, TM, KS, NS, EPI, false>(g, s);
}

// Weights of fewer elements stay with the large tiles: there is little to gain (1024 x 1024 and 1536 x 1024, 48 to 500 rows,
// 10-12 us -> 8-12).  From the line on: 4096 -> 1024 columns 23-25 -> 11-18, 2048 x 2048 21-24 -> 9-19.
constexpr int64_t kRingMinWeights = (int64_t)4 << 20;

// Tile and split of a product.  bm = 0: not a product for this kernel.
struct RingPlan { int bm, bn, splits; };

// The rules (us, large-tile kernel -> this one; weights cold, K / N of 3584 / 4608 .. 37888 and 4096 / 6144 .. 28672;
// a split product counts the sum of its partial tiles, which the next RMSNorm or the reduce launch does):
// - 64-column tiles with the fewest rows that still make one round of 256 workgroups.  Q|K|V: 82 rows 33 -> 18 and
//   38 -> 21, 232 rows 34 -> 26 and 39 -> 29, 331 rows 33 -> 23 and 38 -> 35; a second round loses (331 rows in 288
//   tiles of 128: 38 -> 50).  Of 192 rows: a single tile row (more than 128 columns of tiles) only up to 144 rows (9216
//   columns, 129 / 144 / 160 / 192 rows: K = 5120 47 -> 48, 48 -> 50, 49 -> 53, 50 -> 56, K = 8192 71 -> 66, 72 -> 68,
//   72 -> 69, 74 -> 75), and several tile rows only from 32 stages on (16 stages: 12 -> 13; 32: 21 -> 19).
// - gate/up: one tile row of up to 256 rows, 128 or 160 columns, whichever gives one round.  82 rows 76 -> 57 and
//   49 -> 44, 165 rows 98 -> 64 and 68 -> 56, 232 rows 98 -> 79 and 76 -> 66.  Up to 384 rows it pays only where the
//   256 x 256 tiles need a second round (257 / 300 / 331 / 384 rows of 18944 x 3584: 122 -> 101, 123 -> 99, 124 -> 101,
//   128 -> 104; 16512 x 2048 77-79 -> 61-66, 20480 x 5120 178-189 -> 147-156; in one round they win, 89 against 95),
//   and not with half of the CUs idle (200 rows, 6144 gate/up columns in 96 tiles: 24 -> 34).
// - residual products, K shared out over one round of workgroups: 128 columns where a share then keeps 16 stages or
//   more (down, 82 rows 49 + 4.7 -> 29 + 4.9 and 39 + 4.6 -> 26 + 4.8, 232 rows 54 + 6 -> 40 + 7 and 44 + 7 -> 35 + 7),
//   else 64 columns and fewer, longer shares (O, 116 rows 17 + 4.6 -> 11 + 4 and
//   18 + 4.4 -> 13 + 4, 331 rows 19 + 7 -> 18 + 4 and 25 + 9 -> 20 + 5).  Not: more than 48 tile columns of 128 and 193 rows
//   or more (8192 x 12288, 224 rows: 72 -> 74) or long shares (8192 x 28672, 112 stages, 100 / 160 / 192 rows: 120 -> 113,
//   126 -> 132, 132 -> 142); 193-256 rows whose 64-column tiles leave no second share (5120 x 5120: 33 -> 40).
// - the same beyond 256 rows: several tile rows of 128 x 128 where two shares or more keep 24 to 47 stages, fewer by as much as
//   CUs stay idle, else of 192 x 128 where they keep 16 to 31 (with the sum of the partial tiles, 331 / 460 / 576 rows:
//   4096 x 4096 33 / 38 / - -> 30 / 31 / -, 1024 x 16384 52 / 54 / 53 -> 27 / 29 / 34, 2560 x 6912 32 / 35 / 39 -> 26 / 32 / 36,
//   2048 x 8192 35 / 36 / 39 -> 27 / 30 / 35, 4608 x 4608 35 / - / - -> 32 / - / -, 3584 x 3584 - / 30 / 36 -> - / 28 / 31; idle
//   CUs: 40 stages on 192 of them, 4096 x 5120, 34 -> 35 at 331 rows, and on all of them 38 -> 33 at 400).  Where the
//   64-column tiles are the alternative and not the large ones, 192 x 128 needs two and a half times their shares (300-560 rows,
//   shares of both: 4096 x 2048 1 / 2 21.0 -> 25.3, 5120 x 2560 1 / 2 25.6 -> 30.3, 2304 x 4096 2 / 4 23.9 -> 25.2,
//   1152 x 9216 4 / 9 24.7 -> 25.5, 512 x 18944 10 / 16 23.6 -> 26.6; 2048 x 5632 2 / 5 29.3 -> 27.0, 3072 x 4608 1 / 3 a
//   fifth faster): as many workgroups and no more, which write twice the partial tiles.  128 x 128 needs more shares than theirs
//   or nine tenths of the CUs (4096 x 3584 2 / 2 on 192 CUs 23.8 -> 25.0, 1792 x 4608 3 / 3 on 210 22.8 -> 23.4).  Longer shares
//   gain less and less (192 x 128, 331 rows: 4096 x 14336, 56 stages, 64 -> 59 to 62; 8192 x 8192, 64 stages, 68 -> 69;
//   3584 x 18944, 74 stages, 69 -> 69 to 74), one share nothing (4096 x 4096, 576 rows: 41 -> 42), and shorter ones lose to
//   64-column tiles (2048 x 2048, 8 stages: 16.1 -> 16.7).
// - without room for the partial tiles, 64-row tiles and 128 x 64 win all the same (4096 x 14336, 64 rows: 122 -> 74;
//   4096 x 4096, 100 rows 41 -> 29, 224 rows 41 -> 30), the others do not (160 rows 39 -> 36 and 49 -> 52; 128 columns:
//   4096 x 14336, 224 rows 131 -> 193); those leave unless half of their shares find room.
static RingPlan ring_plan(int m, int n, int k, int epilogue, size_t room) {
  const RingPlan no = {0, 0, 0};
  if (m > 576) return no;                               // three tiles of 192 rows
  const int rows[4] = {64, 128, 192, 256};
  int one = 0;                                          // fewest rows that make a single tile row
  for (int i = 3; i >= 0; --i)
    if (m <= rows[i]) one = rows[i];
  auto tiles = [&](int bm, int cols, int bn) { return (int64_t)((m + bm - 1) / bm) * ((cols + bn - 1) / bn); };
  if (epilogue == FASTAV_EPI_RESADD) {
    auto cut = [&](RingPlan p) {                        // to the shares whose partial tiles find room
      const int64_t fits = (int64_t)(room / ((size_t)m * n * sizeof(float)));
      if (p.splits > fits) {
        if (!(p.bm == 64 || (p.bm == 128 && p.bn == 64)) && fits * 2 < p.splits) return no;
        p.splits = fits < 1 ? 1 : (int)fits;
      }
      return p;
    };
    auto narrow = [&]() -> RingPlan {                   // 64-column tiles
      const int bm = m <= 64 ? 64 : m <= 128 ? 128 : m <= 192 ? 192 : m <= 256 ? 128 : 192;
      const int64_t t64 = tiles(bm, n, 64);
      if (t64 > kNumCUs || (m > 192 && m <= 256 && t64 > kNumCUs / 2)) return no;
      int splits = (int)(kNumCUs / t64);
      if (splits > k / 64 / 8) splits = k / 64 / 8;     // a share is at least 8 stages
      if (splits > 16) splits = 16;
      return {bm, 64, splits < 1 ? 1 : splits};
    };
    const int64_t t128 = tiles(one ? one : 256, n, 128);
    const bool long_k = t128 <= kNumCUs && (k / 64) / (kNumCUs / t128) >= 16;
    if (one == 0) {
      const RingPlan other = long_k ? no : narrow();
      for (int bm = 128; bm <= 192; bm += 64) {
        const int64_t t = tiles(bm, n, 128), fill = kNumCUs / t;
        const int splits = (int)(fill < 16 ? fill : 16);
        const int stages = splits >= 2 ? k / 64 / splits : 0;
        if (!(bm == 128 ? stages >= 24 && stages * kNumCUs < 48 * t * splits : stages >= 16 && stages < 32)) continue;
        if (other.bm != 0 && (bm == 128 ? splits <= other.splits && t * splits < 224 : 2 * splits < 5 * other.splits)) continue;
        const RingPlan wide = cut({bm, 128, splits});
        if (wide.bm != 0) return wide;                  // else, without the room, as before these tiles
        break;
      }
      return other.bm == 0 ? no : cut(other);
    }
    if (long_k && one > 64) {
      const RingPlan p = {one, 128, kNumCUs / t128 < 16 ? (int)(kNumCUs / t128) : 16};
      return t128 > 48 && (m > 192 || (m > 128 && (k / 64) / p.splits >= 64)) ? no : cut(p);
    }
    const RingPlan p = narrow();
    return p.bm == 0 ? no : cut(p);
  }
  const int cols = epilogue == FASTAV_EPI_SWIGLU ? 2 * n : n;
  for (int i = 0; i < 3; ++i) {
    if (tiles(rows[i], cols, 64) > kNumCUs) continue;
    if (rows[i] == 192 && (m <= 192 ? m > 144 : k < 32 * 64)) break;
    return {rows[i], 64, 1};
  }
  if (epilogue != FASTAV_EPI_SWIGLU) return no;
  if (tiles(256, cols, 128) < kNumCUs * 5 / 8) return no;
  if (one != 0 && tiles(one, cols, 128) <= kNumCUs) return {one, 128, 1};
  if (one != 0 && tiles(one, cols, 160) <= kNumCUs) return {one, 160, 1};
  if (m <= 384 && tiles(384, cols, 160) <= kNumCUs && tiles(256, cols, 256) > kNumCUs) return {384, 160, 1};
  return no;
}

// Scratch for partial tiles, of which only whole, aligned rows of the residual can be completed.
static size_t ring_room(const GemmArgs& g, const void* scratch, size_t scratch_bytes) {
  return scratch == nullptr || (uintptr_t)scratch % 16 != 0 || g.ldc % 4 != 0 || (uintptr_t)g.C % 16 != 0 ? 0 : scratch_bytes;
}

static bool ring_sizes(int64_t m, int64_t n, int64_t k) {
  if (n * k < kRingMinWeights) return false;
  // the copies address rows by 32-bit byte offsets from the start of a matrix
  return n * k * 2 < ((int64_t)1 << 32) && m * k * 2 < ((int64_t)1 << 32);
}

bool ring_linear_takes(const GemmArgs& g, int n_seg, int epilogue, const void* scratch, size_t scratch_bytes) {
  if (!ring_sizes(g.M, g.N, g.K)) return false;
  for (int i = 0, prev = 0; epilogue == FASTAV_EPI_STORE && i < n_seg; prev = g.seg_end[i++])
    if ((g.seg_end[i] - prev) % 128) return false;
  return ring_plan(g.M, g.N, g.K, epilogue, ring_room(g, scratch, scratch_bytes)).bm != 0;
}

// The plan of a product with one weight matrix, for fastav_linear_plan.
bool ring_linear_plan(int64_t m, int n, int k, int epilogue, size_t room, fastav_linear_plan_t* out) {
  if (m > 0x7FFFFFFF || !ring_sizes(m, n, k) || (epilogue == FASTAV_EPI_STORE && n % 128)) return false;
  const RingPlan p = ring_plan((int)m, n, k, epilogue, room);
  if (p.bm == 0) return false;
  out->tile_rows = p.bm; out->tile_cols = p.bn; out->splits = p.splits;
  return true;
}

// Ring depths: all of LDS, or half of it where two workgroups share a CU (64 x 64 tiles).
template <int EPI>
static fastav_status_t launch_plan(const RingPlan& p, const GemmArgs& g, hipStream_t s) {
  const int key = p.bm * 1000 + p.bn;
  switch (key) {
    case 64064: return launch_ring<64, 64, 2, 2, 5, EPI>(g, p.splits, s);
    case 128064: return launch_ring<128, 64, 2, 2, 6, EPI>(g, p.splits, s);
    case 192064: return launch_ring<192, 64, 2, 2, 5, EPI>(g, p.splits, s);
    default: break;
  }
  if constexpr (EPI != FASTAV_EPI_STORE) {
    switch (key) {
      case 128128: return launch_ring<128, 128, 2, 2, 4, EPI>(g, p.splits, s);
      case 192128: return launch_ring<192, 128, 2, 2, 4, EPI>(g, p.splits, s);
      case 256128: return launch_ring<256, 128, 2, 1, 3, EPI>(g, p.splits, s);
      default: break;
    }
  }
  if constexpr (EPI == FASTAV_EPI_SWIGLU) {
    switch (key) {
      case 64128: return launch_ring<64, 128, 2, 2, 3, EPI>(g, p.splits, s);
      case 64160: return launch_ring<64, 160, 2, 2, 5, EPI>(g, p.splits, s);
      case 128160: return launch_ring<128, 160, 2, 2, 4, EPI>(g, p.splits, s);
      case 192160: return launch_ring<192, 160, 2, 2, 3, EPI>(g, p.splits, s);
      case 256160: return launch_ring<256, 160, 2, 1, 3, EPI>(g, p.splits, s);
      case 384160: return launch_ring<384, 160, 3, 1, 2, EPI>(g, p.splits, s);
      default: break;
    }
  }
  return fail(FASTAV_EINVAL, "gemm: no %d x %d ring tile", p.bm, p.bn);
}

fastav_status_t launch_linear_ring(GemmArgs& g, int epilogue, void* scratch, size_t scratch_bytes, hipStream_t s, SplitKPending* pend) {
  const RingPlan p = ring_plan(g.M, g.N, g.K, epilogue, ring_room(g, scratch, scratch_bytes));
  if (epilogue == FASTAV_EPI_STORE) return launch_plan<FASTAV_EPI_STORE>(p, g, s);
  if (epilogue == FASTAV_EPI_SWIGLU) return launch_plan<FASTAV_EPI_SWIGLU>(p, g, s);
  // the partial tiles are added to the residual in split order
  if (p.splits == 1) return launch_plan<FASTAV_EPI_RESADD>(p, g, s);
  GemmArgs gp = g;
  gp.partial = (float*)scratch;
  gp.vec_ok = 1;
  fastav_status_t st = launch_plan<kEpiPartial>(p, gp, s);
  if (st != FASTAV_OK) return st;
  SplitKPending sum;
  sum.partial = (const float*)scratch; sum.splits = p.splits; sum.M = g.M; sum.N = g.N;
  if (pend != nullptr && g.ldc == g.N) { *pend = sum; return FASTAV_OK; }
  return launch_splitk_reduce((float*)g.C, g.ldc, sum, s);
}

}  // namespace fastav
