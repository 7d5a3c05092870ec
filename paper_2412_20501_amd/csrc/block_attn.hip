// Host side of the block attention kernel (block_attn_kernel.h): grids and shapes of the launches, and the fold of a
// launch whose keys are cut into parts.
#include "block_attn_kernel.h"

namespace tr {

#define TR_SHAPE(D, R, G) extern template hipError_t launch_attn_shape<D, R, G>(const AttnParams&, int, dim3, hipStream_t);
TR_SHAPE(64, 8, 1) TR_SHAPE(64, 4, 2) TR_SHAPE(64, 2, 2) TR_SHAPE(64, 4, 1)
TR_SHAPE(128, 8, 1) TR_SHAPE(128, 4, 2) TR_SHAPE(128, 2, 2) TR_SHAPE(128, 4, 1)
#undef TR_SHAPE

namespace {

// Fold of a partitioned launch: the Update of Sec. 3.1 over the parts of a row at once, out = sum of exp(lse_i - lse)
// out_i; with kEpiMerge that block then takes one Update onto the accumulators.  Weighted and not blended part by part,
// so that an infinite value of V stays infinite (a blend would subtract it from itself), and a row with a NaN weight in
// any part is the block that one pass over the keys gives: out = NaN, lse = -inf.  A kernel of its own, because whoever finishes last would otherwise read all
// parts of a row tile through one compute unit and pay for cache write-backs between the XCDs first:
// 16 rows x 4 heads in 16 parts of 1024 keys 50 -> 30 us, 500 rows x 32 heads in 4 parts 119 -> 106 us (whole call).
// A thread owns 16 bytes of a row; lse values and pieces of all its parts (MAXP at most) are requested before
// the log-sum-exp starts.
constexpr int kFoldThreads = 256;
template <int D, int EPI, int MAXP>
__global__ void __launch_bounds__(kFoldThreads) fold_parts_kernel(const AttnParams p) {
  constexpr int CPRF = D / 4;
  const int group = (int)blockIdx.x, kv = divide(p.by_members, group), m = group - kv * p.members;
  const int b = divide(p.by_hkv, kv), hk = kv - b * p.Hkv;
  const int head0 = p.pack ? 0 : divide(p.by_qtiles, m);
  const int q0 = (p.n_qtiles - 1 - (m - head0 * p.n_qtiles)) * p.bm, n_tile = min(p.bm, part_rows_total(p) - q0);
  const int r = (int)blockIdx.y * (kFoldThreads / CPRF) + (int)threadIdx.x / CPRF, cc = (int)threadIdx.x % CPRF;
  if (r >= n_tile) return;
  int lo, hi;
  pos_span(p, q0, p.bm, lo, hi);
  const int n_live = live_parts(p, hi);
  if (n_live == 1) return;   // written by the attention kernel

  const int head = divide(p.by_sq, q0 + r), pos = q0 + r - head * p.Sq, hq = hk * p.gq + head0 + head;
  const int64_t l_at = (int64_t)b * p.l_sb + (int64_t)hq * p.l_sh + (int64_t)pos * p.l_ss;
  const int64_t o_at = (int64_t)b * p.o_sb + (int64_t)hq * p.o_sh + (int64_t)pos * p.o_ss + 4 * cc;
  const int64_t slot_row = (int64_t)group * p.n_parts * p.part_rows + r;
  float ls[MAXP];
  f32x4 y[MAXP];
#pragma unroll
  for (int i = 0; i < MAXP; i++) ls[i] = p.part_lse[slot_row + (int64_t)min(i, n_live - 1) * p.part_rows];
#pragma unroll
  for (int i = 0; i < MAXP; i++)
    y[i] = *reinterpret_cast<const f32x4*>(p.part_out + (slot_row + (int64_t)min(i, n_live - 1) * p.part_rows) * D + 4 * cc);
  float acc = -INFINITY;
  f32x4 held = {0.f, 0.f, 0.f, 0.f};
  if (EPI == kEpiMerge) {
    acc = p.lse[l_at];
    held = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.out) + o_at);
  }
  float top = -INFINITY, total = 0.f;
  bool not_a_number = false;
#pragma unroll
  for (int i = 0; i < MAXP; i++)
    if (i < n_live) {
      top = fmaxf(top, ls[i]);
      not_a_number |= ls[i] != ls[i];
    }
#pragma unroll
  for (int i = 0; i < MAXP; i++)
    if (i < n_live) {
      ls[i] = ls[i] == -INFINITY ? -1.f : expf(ls[i] - top);   // -1: an empty part, whose values are not looked at
      total += fmaxf(ls[i], 0.f);
    }
  const float inv = total > 0.f ? 1.f / total : 0.f;
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < MAXP; i++)
    if (i < n_live) {
      const float w = ls[i] * inv;
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] = ls[i] >= 0.f ? __builtin_fmaf(w, y[i][e], x[e]) : x[e];
    }
  float lse = not_a_number || !(total > 0.f) ? -INFINITY : top + logf(total);
  if (not_a_number) x = f32x4{1.f, 1.f, 1.f, 1.f} * __builtin_nanf("");
  if (EPI == kEpiMerge) {
    const UpdatePlan pl = plan_update(acc, lse);
    lse = pl.new_lse;
    x = apply_update(pl, held, x);
  }
  if (EPI == kEpiBf16) {
    bf16x4 ob;
#pragma unroll
    for (int e = 0; e < 4; e++) ob[e] = (__bf16)x[e];
    *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + o_at) = ob;
  } else {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.out) + o_at) = x;
  }
  if (cc == 0) p.lse[l_at] = lse;   // a row lies within one wave, so every thread of it has read the old value
}

template <int D, int EPI>
hipError_t launch_fold_typed(const AttnParams& p, dim3 grid, hipStream_t stream, hipEvent_t done) {
  if (p.n_parts <= 4) hipExtLaunchKernelGGL((fold_parts_kernel<D, EPI, 4>), grid, dim3(kFoldThreads), 0, stream, nullptr, done, 0, p);
  else if (p.n_parts <= 8) hipExtLaunchKernelGGL((fold_parts_kernel<D, EPI, 8>), grid, dim3(kFoldThreads), 0, stream, nullptr, done, 0, p);
  else hipExtLaunchKernelGGL((fold_parts_kernel<D, EPI, kMaxParts>), grid, dim3(kFoldThreads), 0, stream, nullptr, done, 0, p);
  return hipGetLastError();
}
template <int D>
hipError_t launch_fold(const AttnParams& p, int epilogue, hipStream_t stream, hipEvent_t done) {
  constexpr int rows = kFoldThreads / (D / 4);   // rows one block folds
  const int tile_rows = p.part_rows < p.bm ? p.part_rows : p.bm;
  const dim3 grid((unsigned)(p.B * p.Hkv * p.members), (unsigned)((tile_rows + rows - 1) / rows));
  if (epilogue == kEpiBf16) return launch_fold_typed<D, kEpiBf16>(p, grid, stream, done);
  if (epilogue == kEpiF32) return launch_fold_typed<D, kEpiF32>(p, grid, stream, done);
  return launch_fold_typed<D, kEpiMerge>(p, grid, stream, done);
}

template <int D>
hipError_t launch_attn(const AttnParams& p, int epilogue, dim3 grid, hipStream_t stream) {
  switch (p.shape) {
    case kShapeTrio:
      if (D != 64) return hipErrorInvalidValue;
      [[fallthrough]];
    case kShape2x2: return launch_attn_shape<D, 2, 2>(p, epilogue, grid, stream);
    case kShape4x2: return launch_attn_shape<D, 4, 2>(p, epilogue, grid, stream);
    case kShape4x1: return launch_attn_shape<D, 4, 1>(p, epilogue, grid, stream);
    default: return launch_attn_shape<D, 8, 1>(p, epilogue, grid, stream);
  }
}

}  // namespace

hipError_t launch_block_attn(AttnParams& p, int D, int epilogue, hipStream_t stream, hipEvent_t fold_done) {
  const int64_t nbh = (int64_t)p.B * p.Hq;
  if (nbh * p.n_qtiles == 0) return hipSuccess;
  if (p.n_qtiles > 65535 || p.bm != shape_rows(p.shape)) return hipErrorInvalidValue;   // grid y limit
  dim3 grid((unsigned)nbh, (unsigned)p.n_qtiles);
  if (p.xcd_map == 2) grid = dim3(8u * (unsigned)p.n_qtiles, (unsigned)(nbh / 8));
  if (p.n_parts > 0) {
    if ((int64_t)p.units * p.members == 0) return hipSuccess;
    grid = dim3((unsigned)(((int64_t)p.units * p.members + 7) / 8 * 8));
  } else if (p.n_chunks > 0) {
    grid = dim3((unsigned)nbh, (unsigned)((p.chunk_end - p.chunk_begin) * p.n_qtiles));
    if (grid.y > 65535 || epilogue != kEpiMerge) return hipErrorInvalidValue;
  }
  if (p.n_parts > 0) {
    p.by_qtiles = make_divisor(p.n_qtiles);
    p.by_members = make_divisor(p.members);
    p.by_parts = make_divisor(p.n_parts);
    p.by_hkv = make_divisor(p.Hkv);
    p.by_sq = make_divisor(p.Sq);
    p.by_part_keys = make_divisor(p.part_keys);
  }
  if (p.renew > 0) p.by_renew = make_divisor(p.renew);
  const hipError_t e = D == 128 ? launch_attn<128>(p, epilogue, grid, stream) : launch_attn<64>(p, epilogue, grid, stream);
  if (e != hipSuccess || p.n_parts <= 1) return e;
  return D == 128 ? launch_fold<128>(p, epilogue, stream, fold_done) : launch_fold<64>(p, epilogue, stream, fold_done);
}

}  // namespace tr
