// What the two bf16 matrix-core products share: the argument block, the asynchronous global -> LDS copy and the LDS
// row layout.
#pragma once
#include "common.hpp"

namespace fastav {

struct GemmArgs {
  const bf16_t* A;
  const bf16_t* W[3];
  int seg_end[3];          // exclusive end column of each segment
  const bf16_t* W2;        // "up" matrix (SwiGLU only)
  void* C;
  int64_t ldc;
  int M, N, K;             // N = output columns
  int tiles_m, tiles_n;
  int band;                // tile columns per band of the tile order (1 = column-major)
  int n_off;               // first output column of this launch (a launch may cover a range of tile columns)
  int splits;              // split-K: blockIdx.y picks a K range and writes an fp32 partial tile to `partial`
  float* partial;          // [splits][M][N] fp32 (split-K only)
  void* Cs[3];             // plain-store epilogue with seg_out: segment i of the output columns goes to its own matrix
  int64_t ldcs[3];         //   Cs[i] (row pitch ldcs[i] elements) instead of columns of C
  int seg_out;
  int vec_ok;              // the output (C, or `partial`) takes 16-byte accesses: base and row pitch are multiples of 16 bytes
  // plain-store epilogue, optional: rotate-half RoPE on the output columns of the first `rope_segs` segments (whole
  // heads of rope_dh = 64 or 128 columns) before the one rounding to bf16: row r is rotated by the angles of position
  // rope_pos[r], taken from rope_tab [position][rope_dh / 2] = (cos, sin)
  const int32_t* rope_pos;
  const float2* rope_tab;
  int rope_dh, rope_segs;
  // optional: output row r is computed from row a_rows[r] of A (a row gather folded into the operand copies)
  const int32_t* a_rows;
};

constexpr int kNumCUs = 256;
constexpr int kEpiPartial = 100;   // internal epilogue: plain fp32 store of a split-K partial
constexpr int kEpiResAtomic = 101; // internal epilogue: residual update through fire-and-forget hardware adds

// Asynchronous 16-byte-per-lane global -> LDS copy as a buffer load: a 128-bit resource (base, no stride, no bounds
// of interest) in SGPRs, a 32-bit lane offset and a scalar byte offset that advances along K; lane l's data lands
// at lds_byte_addr + 16 l.  Completion is tracked by vmcnt (copies complete in issue order).
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x4_t make_rsrc(const void* base) {
  const uint64_t u = (uint64_t)(uintptr_t)base;
  u32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)u);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32) & 0xFFFFu);
  r[2] = 0xFFFFFFFFu;                                  // num_records: the whole address range after base
  r[3] = 0x00020000u;                                  // raw buffer, 32-bit data format
  return r;
}
__device__ __forceinline__ void dma16_buf(u32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %3\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" : : "v"(voff), "s"(rsrc), "s"(soff), "s"(lds_byte_addr) : "memory");
}
template <int N> __device__ __forceinline__ void dma_wait_keep() {   // until at most N copies are in flight
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

__device__ __forceinline__ int swz8(int row, int chunk) { return row * 8 + (chunk ^ ((row >> 1) & 7)); }   // 16-byte units

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2_t t = {(bf16_t)a, (bf16_t)b};
  return __builtin_bit_cast(uint32_t, t);
}

// Products of few rows (gemm_ring.hip): whether this one runs there, and its launch.
bool ring_linear_takes(const GemmArgs& g, int n_seg, int epilogue, const void* scratch, size_t scratch_bytes);
fastav_status_t launch_linear_ring(GemmArgs& g, int epilogue, void* scratch, size_t scratch_bytes, hipStream_t s, SplitKPending* pend);

}  // namespace fastav
