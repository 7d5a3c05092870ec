// Internal declarations shared by the translation units of libtokenring (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "divisor.h"
#include "tokenring.h"

namespace tr {

constexpr int kMaxRefs = 32;   // references of later segments that workgroups of fewer than 256 rows keep in LDS
constexpr int kMaxRefsTrio = 8;   // the same where three of them share a compute unit
constexpr int kMaxParts = 16;  // parts the keys of one partitioned attention launch are cut into at most

// Shapes of an attention workgroup: row groups of 32 Query rows x key groups.
constexpr int kShape8x1 = 0, kShape4x1 = 1, kShape4x2 = 2, kShape2x2 = 3, kShapeTrio = 4;   // kShapeTrio: 2 x 2 at D 64, three to a compute unit
constexpr int shape_rows(int shape) { return shape == kShape8x1 ? 256 : shape >= kShape2x2 ? 64 : 128; }
constexpr int shape_key_groups(int shape) { return shape >= kShape4x2 ? 2 : 1; }
constexpr int shape_per_unit(int shape, int D) { return shape == kShapeTrio ? 3 : shape != kShape4x1 ? 1 : D == 64 ? 3 : 2; }   // workgroups that share a compute unit

// Arguments of the block-attention kernel: raw pointers, element strides, sizes.
struct AttnParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  void* out;    // bf16 or fp32, [B,Hq,Sq,D]
  float* lse;   // [B,Hq,Sq]
  int64_t q_sb, q_sh, q_ss;
  int64_t k_sb, k_sh, k_ss;
  int64_t v_sb, v_sh, v_ss;
  int64_t o_sb, o_sh, o_ss;
  int64_t l_sb, l_sh, l_ss;
  int B, Hq, Hkv, Sq, Sk;
  int causal;     // 0: every key visible; 1: key c visible to query r iff c <= r + causal_off
  int causal_off; // q_pos0 - k_pos0, clamped so that r + causal_off cannot overflow
  float scale;    // softmax scale (natural units)
  int shape;      // of a workgroup, kShape8x1 ...
  int bm;         // its Query rows
  int n_qtiles;   // ceil(Sq / bm)
  int xcd_map;    // 1: place all query tiles of a K/V head on one XCD (grid x = batch*head, y = query tile); 2: the same with grid x = XCD + 8 * query tile, y = head within the XCD
  int gq;         // query heads per K/V head (Hq / Hkv)
  int gq_log2;    // log2(gq) if gq is a power of two, else -1
  // Chunk form (n_chunks > 0): q, out, lse and k, v are chunk 0 of n_chunks chunks that lie one behind the other
  // along S; the launch covers Query chunks chunk_begin .. chunk_end - 1.
  int n_chunks, chunk_begin, chunk_end;
  int chunk_bf16; // 1: every block after a Query chunk's first is rounded to bf16 before its Update
  int renew;      // keys (a multiple of 32) after which a row's exponent reference is taken anew; 0: never
  int renew_log2; // log2 of the keys (at least 128) to whose next multiple that may wait
  // Partitioned form (n_parts > 0), see the kernel: n_qtiles then counts the tiles of the row space
  // (one head's Sq rows, or with pack the gq * Sq rows of a K/V head's group).
  int n_parts;    // parts of the keys, part_keys (a multiple of 128) each; 0: the plain form
  int part_keys;
  int pack;       // 1: a row space holds every query head of a K/V head
  int units;      // B * Hkv * n_parts
  int members;    // row tiles that read one unit's keys
  int part_rows;  // rows of a scratch slot
  float* part_out;       // [row tile][part][part_rows][D], if n_parts > 1
  float* part_lse;       // [row tile][part][part_rows]
  Divisor by_members, by_parts, by_hkv, by_qtiles, by_sq, by_part_keys, by_renew;   // of the sizes of those names; set by launch_block_attn
};

// Arguments of the merge kernel.
struct MergeParams {
  float* acc_out;
  float* acc_lse;
  const void* blk_out;  // fp32 or bf16
  const float* blk_lse;
  int64_t ao_sb, ao_sh, ao_ss;
  int64_t al_sb, al_sh, al_ss;
  int64_t bo_sb, bo_sh, bo_ss;
  int64_t bl_sb, bl_sh, bl_ss;
  int B, H, S, D;
  int contiguous;  // 1: all four tensors are dense [B*H*S, D] / [B*H*S]
};

// Arguments of the n-ary merge kernel: up to kMergeNMax partial results with common strides.
constexpr int kMergeNMax = 16;
struct MergeNParams {
  float* out;        // fp32 [B,H,S,D], written (read as one more partial if accumulate)
  float* lse;        // fp32 [B,H,S]
  const void* blk_out[kMergeNMax];   // fp32 or bf16
  const float* blk_lse[kMergeNMax];
  int64_t o_sb, o_sh, o_ss;
  int64_t l_sb, l_sh, l_ss;
  int64_t bo_sb, bo_sh, bo_ss;
  int64_t bl_sb, bl_sh, bl_ss;
  int B, H, S, D;
  int n;           // number of partials
  int accumulate;  // 1: the old contents of out / lse take part as a further partial
  int contiguous;  // 1: every tensor is dense [B*H*S, D] / [B*H*S]
};

// Launchers (defined next to their kernels). They only enqueue; errors come back as hipError_t.
// epilogue: 0 = bf16 block_out, 1 = fp32 block_out, 2 = merge into the fp32 accumulators p.out / p.lse
// fold_done: event that a launch in parts carries on its fold (may be NULL)
hipError_t launch_block_attn(AttnParams& p, int D, int epilogue, hipStream_t stream, hipEvent_t fold_done = nullptr);
hipError_t launch_merge(const MergeParams& p, bool blk_bf16, hipStream_t stream);
hipError_t launch_merge_n(const MergeNParams& p, bool blk_bf16, hipStream_t stream);

// Events armed by tr_time_next_kernel for the calling thread; the next launch consumes them.
struct TimingEvents { hipEvent_t start, stop; };
TimingEvents take_timing_events();

#if defined(__HIPCC__)
// Every kernel of the library is launched through here.  With armed events the dispatch itself
// carries them, so they hold the kernel's own begin and end timestamps (no queue gaps).
template <typename Kernel, typename... Args>
inline hipError_t launch_kernel(Kernel kernel, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, Args... args) {
  const TimingEvents ev = take_timing_events();
  if (ev.start != nullptr || ev.stop != nullptr) hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, ev.start, ev.stop, 0, args...);
  else hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, args...);
  return hipGetLastError();
}
#endif

#if defined(__HIPCC__)
// The Update of Sec. 3.1 for one row, shared by the merge kernel and the fused attention
// epilogue:  lse' = max + log1p(exp(-|lse - block_lse|)),  w = exp(block_lse - lse')
// (= sigmoid(block_lse - lse)),  out' = out + w (block_out - out).  The identity element
// (out = 0, lse = -inf) on either side is handled exactly and never produces NaN.
typedef float tr_f32x4 __attribute__((ext_vector_type(4)));
struct UpdatePlan {
  int mode;  // 0: blend with weight w (meaningless otherwise); 1: both empty -> 0; 2: empty accumulator -> block; 3: empty block -> keep
  float w, new_lse;
};
__device__ __forceinline__ UpdatePlan plan_update(float lse_acc, float lse_blk) {
  // Straight-line: a chain of these (the parts of one row) then costs the latency of its logarithms only,
  // and no lane waits for another's case.
  UpdatePlan r;
  const float m = fmaxf(lse_acc, lse_blk);
  const bool acc_empty = lse_acc == -INFINITY, blk_empty = lse_blk == -INFINITY;   // an empty accumulator's out may be uninitialised
  const float both = m + log1pf(expf(-fabsf(lse_acc - lse_blk)));
  r.mode = m == -INFINITY ? 1 : (acc_empty ? 2 : (blk_empty ? 3 : 0));
  r.new_lse = m == -INFINITY ? m : (acc_empty ? lse_blk : (blk_empty ? lse_acc : both));
  r.w = expf(lse_blk - r.new_lse);
  return r;
}
// Branch-free: the blend is evaluated for every lane and bit masks made from the plan's case pick
// the result among blend, block, accumulator and zero, so whatever NaN or Inf an uninitialised
// side holds never reaches it and no lane waits for another's case.
__device__ __forceinline__ tr_f32x4 apply_update(const UpdatePlan& pl, tr_f32x4 acc, tr_f32x4 blk) {
  const unsigned m_blend = pl.mode == 0 ? 0xffffffffu : 0u;
  const unsigned m_blk = pl.mode == 2 ? 0xffffffffu : 0u;
  const unsigned m_acc = pl.mode == 3 ? 0xffffffffu : 0u;
  tr_f32x4 o;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const float a = acc[i], y = blk[i];   // scalars: a bit cast must not be applied to a vector element directly
    const float blend = __builtin_fmaf(pl.w, y - a, a);
    const unsigned bits = (m_blend & __builtin_bit_cast(unsigned, blend)) | (m_blk & __builtin_bit_cast(unsigned, y)) |
                          (m_acc & __builtin_bit_cast(unsigned, a));
    o[i] = __builtin_bit_cast(float, bits);
  }
  return o;
}
#endif

}  // namespace tr
