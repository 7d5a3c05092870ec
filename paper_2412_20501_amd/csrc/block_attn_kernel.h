// Blockwise attention step for gfx950 (CDNA4): block_out, block_lse <- Attention(Q, K, V)
// of TokenRing's Algorithm 1 (Sec. 3.2), one Query chunk against one K/V chunk.
//
// Formulation.  Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16:
// the A operand is a 32-key x 16-d slice of the K tile read from LDS, the B operand a
// 16-d x 32-query slice of Q^T held in registers for the whole kernel.  In the MFMA
// accumulator layout lane (q = lane%32, half = lane/32) then owns, for ONE query, the
// 16 keys {8g + 4*half + r} of a 32-key sub-tile: the softmax is in-lane.  The
// exponentiated sub-tile P^T, rounded to bf16, is already in the B-operand layout of the
// second product O^T = V^T P^T; its A operand (32 d x 16 keys of V^T) comes from the
// row-major V tile in LDS through the transposing read ds_read_b64_tr_b16, with the key
// order inside each 16-key step permuted to match the accumulator layout of P^T (a
// contraction index may be permuted freely as long as both operands agree).  The O^T
// accumulator again has one query per lane, so rescaling and the final 1/l need no
// cross-lane traffic.
//
// Pipeline.  A lone wave issues vector-ALU instructions far below the SIMD's rate and cannot
// hide its softmax behind another wave's MFMAs, so MFMA and softmax work are interleaved
// INSIDE every wave, one 32-key sub-tile apart: step j runs, as one instruction stream,
//     MFMA : O += V_{j-1}^T P_{j-1}      and      S_{j+1} = K_{j+1} Q^T
//     VALU : P_j = exp2((S_j - m_ref) * scale*log2e), row sums
// with no dependency between the two halves.  Two such waves per SIMD fill each other's
// gaps.  A workgroup has 8 waves of 32 query rows (256 rows); K/V tiles of 16 KiB (64 keys
// = two sub-tiles at D = 128, 128 keys = four at D = 64) go straight from global memory into
// 4-deep LDS rings (global_load_lds), the K tile with a 16-byte XOR swizzle and the V tile
// with a 32-byte XOR swizzle that make the ds_read_b128 and the transposing reads
// bank-conflict free.  One workgroup barrier per tile hands ring slots over.
//
// Few rows.  Where 256-row workgroups would leave compute units idle, a workgroup has R = 4 or 2 row groups and G = 2 key
// groups: sub-tile j of the keys belongs to key group j mod G, every wave keeps a running softmax of its own share, and the
// shares are added up in LDS at the end.  What bounds such a launch is the length of one workgroup; two waves a row group halve
// it, and 4 x 32 or 2 x 32 rows make two or four times as many workgroups of it.  Per tile of 64 keys at D = 128 (an otherwise idle chip)
// 1.1 us with R x G = 8 x 1, 0.59 with 4 x 2, 0.47 with 2 x 2 (four waves; alone on its SIMD a wave takes 1.6 times
// a shared SIMD's time).  4 x 1024 rows on 1024 keys 25.6 -> 15.0 us, 1 x 8192 rows 144 -> 67, at D = 64 105 -> 45.
// 2 x 4 measured 5 - 14 % less than 2 x 2 from 4096 keys on and 1 us more below (D = 64); at D = 128 its tiles leave room for two.
//
// Small workgroups.  Shape 4 x 1 is the 256-row workgroup's work in halves, two to a compute unit at D = 128 and three at
// D = 64 (158 VGPRs): one's loads, epilogue and waits at barriers run beside another's products, and a launch ends more evenly.
// What it costs is twice the K/V traffic from L2 into LDS for the same rows.  us, 8 x 1 -> 4 x 1: 512 heads of 256 rows on as many keys
// 41.8 -> 35.4, at D 64 26.2 -> 19.6; 48 heads of 3000 225 -> 207, at D 64 145 -> 121; 64 of 2048 125.3 -> 126.7, at D 64 77.0 -> 73.8; 32 of
// 24576 7720 -> 8015, at D 64 4847 -> 4721; bf16 blocks of 6008 rows in 4 chunks, 16 heads 167 -> 157.
//
// Trio (D = 64).  Shape 2 x 2 with rings of three tiles of 64 keys: 50 KiB of LDS (with references 52) and 154 VGPRs (with renewals 168), three workgroups a compute
// unit.  For launches of 1 to 1.5 workgroups of 128 rows a compute unit, where two of those on some units set the time.  The same bits as 2 x 2.  What bounds it is the vector
// ALU, as in 4 x 1 (0.28 us a step and SIMD, 0.25 there), and K/V traffic, twice 4 x 1's.  us, the shape that would be chosen without it -> trio, under the causal rule:
// 24 heads of 1777 rows 20.3 -> 17.4, 32 of 1024 13.6 -> 11.3, 8 of 4096 36.2 -> 28.8; alone on its unit it is slower than 2 x 2 with rings of four tiles of 128 keys (16 heads of 512 7.4 and 7.7).
#pragma once
#include <type_traits>

#include <atomic>

#include "tr_internal.h"

namespace tr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Shapes of a workgroup: R row groups of 32 Query rows, G key groups; one wave for each pair.
// Keys per LDS tile: 16 KiB of K (and of V) either way, so a tile is 2 sub-tiles of 32 keys at
// D = 128 and 4 at D = 64, where a sub-tile carries half the MFMA work per barrier otherwise.  Shape 4 x 1: half of that, so
// that two (D = 64, with rings of three: three) workgroups share a compute unit.
// Ring depth (tiles) NS of K and of V: three where three workgroups are to share a compute unit.
constexpr int ring_depth(int D, int R, int G) { return D == 64 && R == 4 && G == 1 ? 3 : 4; }
template <int D, int R, int G, int NS>
constexpr int tile_keys() { return (D == 64 ? 128 : 64) / ((R == 4 && G == 1) || NS == 3 ? 2 : 1); }
constexpr int kEpiBf16 = 0, kEpiF32 = 1, kEpiMerge = 2;
constexpr int kPlain = 0, kPart = 1, kChunks = 2, kSegments = 3, kPartSegments = 4;   // forms of the kernel, see there
constexpr bool in_segments(int form) { return form == kSegments || form == kPartSegments; }

// Exchange between the two 32-lane halves of a wave with v_permlane32_swap, which swaps the
// upper half of its first operand with the lower half of its second: fed (x, x) it leaves
// x[lane%32] in the first and x[32 + lane%32] in the second register, in every lane.
// Written as inline asm: at -O3 the compiler folds the second result of the corresponding
// builtin into the first, which silently drops the other half's contribution.  The s_nop
// covers the VALU-write -> permlane-swap hazard the assembler does not see inside asm.
__device__ __forceinline__ void half_pair(float x, float& lo, float& hi) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  lo = a;
  hi = b;
}
__device__ __forceinline__ float half_swap_max(float x) {
  float lo, hi;
  half_pair(x, lo, hi);
  return fmaxf(lo, hi);
}
__device__ __forceinline__ float half_swap_sum(float x) {
  float lo, hi;
  half_pair(x, lo, hi);
  return lo + hi;
}

// Byte offset of 16-byte chunk c of row `row` inside a K tile (row-major, D bf16 per row).
template <int D>
__device__ __forceinline__ int k_lds_off(int row, int c) {
  constexpr int RB = 2 * D;             // row bytes
  constexpr int R2 = 256 / RB;          // rows per 256-byte bank line
  constexpr int NC = RB / 16;           // chunks per row
  return row * RB + ((c ^ ((row / R2) % NC)) << 4);
}
// Byte offset of 16-byte chunk c of row `row` inside a V tile: 32-byte slots XOR-swizzled
// by the row so that the four rows a transposing read touches fall on distinct banks.
template <int D>
__device__ __forceinline__ int v_lds_off(int row, int c) {
  constexpr int RB = 2 * D;
  int slot = c >> 1;
  int swz = (D == 128) ? ((row & 3) << 1) : (row & 2);
  return row * RB + ((slot ^ swz) << 5) + ((c & 1) << 4);
}

// Which (batch*head, query tile) a workgroup computes.  The grid is two-dimensional - x: batch*head,
// y: query tile - so the indices come from the
// hardware instead of integer divisions (a division costs ~40 dependent instructions and the
// decoding sits in front of every workgroup's first load).  Workgroups are dealt round-robin to
// the 8 XCDs in the order of their linear id, which is x-fastest, and the x extent is a multiple
// of 8 whenever xcd_map is set: XCD = blockIdx.x mod 8.  XCD x gets the K/V heads x, x+8, ... and
// all query heads and query tiles that read them, so a head's K/V stays in one L2.
__device__ __forceinline__ void decode_block(const AttnParams& p, int& qt, int& b, int& hq, int& hk) {
  const int gq = p.gq, sh = p.gq_log2;   // query heads per K/V head; its log2, or -1 if not a power of two
  int bh = (int)blockIdx.x, qi = (int)blockIdx.y;
  if (p.xcd_map) {
    int x = bh & 7, hi = bh >> 3;
    if (p.xcd_map == 2) {   // x = XCD + 8 * query tile, y = head within the XCD
      qi = hi;
      hi = (int)blockIdx.y;
    }
    const int kvi = sh >= 0 ? hi >> sh : hi / gq;
    const int mem = sh >= 0 ? hi & (gq - 1) : hi % gq;
    bh = (kvi * 8 + x) * gq + mem;
  }
  b = p.B == 1 ? 0 : bh / p.Hq;
  hq = bh - b * p.Hq;
  hk = sh >= 0 ? hq >> sh : hq / gq;
  qt = p.n_qtiles - 1 - qi;  // late query tiles (most keys under a causal mask) first
}

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// A pointer the compiler must keep in an SGPR pair (it is wave-uniform by construction).
__device__ __forceinline__ const __bf16* uniform_ptr(const __bf16* ptr) {
  const unsigned long long v = (unsigned long long)ptr;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (const __bf16*)(((unsigned long long)hi << 32) | lo);
}

// Workgroup barrier without the memory fence of __syncthreads(): the tile hand-off is
// ordered by explicit s_waitcnt vmcnt() on the direct-to-LDS loads instead.
__device__ __forceinline__ void wg_barrier() { __builtin_amdgcn_s_barrier(); }

// The same for the partitioned form: a one-dimensional grid over units (K/V head of a batch entry, part
// of the keys) and, inside a unit, the row tiles that read its keys.  Every XCD takes one eighth of that
// list, a contiguous piece, so what shares keys mostly shares an L2 and no XCD is left without work: whole units
// dealt to XCDs in turn kept four XCDs idle with four units (3076 rows x 8 heads on 3898 keys 111 us against 77
// uncut).  Returns false for the ids that only fill the last eight up.
struct PartBlock { int tile, b, hk, hq0, part, group; };
__device__ __forceinline__ bool decode_part(const AttnParams& p, PartBlock& w) {
  const int per_xcd = (int)gridDim.x >> 3;
  const int at = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
  const int u = divide(p.by_members, at), m = at - u * p.members;
  if (u >= p.units) return false;
  const int kv = divide(p.by_parts, u);
  w.part = u - kv * p.n_parts;
  w.b = divide(p.by_hkv, kv);
  w.hk = kv - w.b * p.Hkv;
  w.group = kv * p.members + m;
  const int head = p.pack ? 0 : divide(p.by_qtiles, m);
  w.hq0 = w.hk * p.gq + head;
  w.tile = p.n_qtiles - 1 - (m - head * p.n_qtiles);
  return true;
}

template <int N>
using IC = std::integral_constant<int, N>;

// The rows of a partitioned launch: row r of the row space of heads hq0, hq0 + 1, ... is Query row r mod Sq
// of head hq0 + r / Sq.  pos_span: smallest and largest Query position among rows first .. first + n - 1.
__device__ __forceinline__ int part_rows_total(const AttnParams& p) { return p.pack ? p.gq * p.Sq : p.Sq; }
__device__ __forceinline__ void pos_span(const AttnParams& p, int first, int n, int& lo, int& hi) {
  const int last = min(first + n, part_rows_total(p)) - 1;
  const int ha = divide(p.by_sq, first), hb = divide(p.by_sq, last);
  lo = ha == hb ? first - ha * p.Sq : 0;
  hi = ha == hb ? last - hb * p.Sq : p.Sq - 1;
}
// Parts of the keys that any row of the tile sees, the first one always counted: parts 0 .. n - 1 are computed.
__device__ __forceinline__ int live_parts(const AttnParams& p, int pos_last) {
  const int seen = p.causal ? max(0, min(p.Sk, pos_last + p.causal_off + 1)) : p.Sk;
  return max(1, divide(p.by_part_keys, seen + p.part_keys - 1));
}

// LDS behind the K/V rings and, once these are dead, behind the waves' transposed 32 x D fp32 tiles (byte offsets
// from the start): Update weight and case of each row, the rows' output offsets (partitioned form), exponent reference
// and sum of each wave's rows and the references of later segments (more than one key group).
template <int D, int R, int G, int NS = ring_depth(D, R, G)>
struct Lds {
  static constexpr int rings = 2 * NS * tile_keys<D, R, G, NS>() * 2 * D, tiles = R * G * 32 * 4 * D, rows = R * 32;
  static constexpr int w = rings > tiles ? rings : tiles, mode = w + rows * 4, off = mode + rows * 4;
  static constexpr int sums = off + rows * 8, refs = sums + (G > 1 ? G * rows * 8 : 0);
  static constexpr int max_refs = G > 1 && NS == 3 ? kMaxRefsTrio : kMaxRefs;
  static constexpr int tables(int form) {
    return G > 1 ? (in_segments(form) ? refs + max_refs * rows * 4 : refs) : form == kPart || form == kPartSegments ? sums : off;
  }
  static constexpr int query = D == 128 && G == 1 ? R * 2048 : 0;   // a quarter of the Query rows, behind the tables (see the prologue)
  static constexpr int bytes(int form) { return tables(form) + query; }
};

// Sixteen bytes of row r of row group rg, from the waves' tiles in LDS (chunk-swizzled, one tile for each key group):
// the sum over the key groups.
template <int D, int R, int G>
__device__ __forceinline__ f32x4 row_piece(const char* lds, int rg, int r, int c) {
  const char* const at = lds + rg * (32 * 4 * D) + r * (4 * D) + ((c ^ (r & 15)) << 4);
  f32x4 x = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
  for (int g = 1; g < G; g++) {
    const f32x4 y = *reinterpret_cast<const f32x4*>(at + g * R * (32 * 4 * D));
#pragma unroll
    for (int e = 0; e < 4; e++) x[e] += y[e];
  }
  return x;
}

// Epilogue of the partitioned form.  The workgroup's normalised tiles lie in LDS, lse_blk is the log-sum-exp of the lane's
// row over the workgroup's part of the keys (-inf also
// for a row whose weights hold a NaN, which not_a_number says apart).  With one live part the tile is stored or
// merged as it is, otherwise tile and lse go to the scratch slot of (row tile, part) for the fold kernel.  Each key group
// stores its share of the row group's rows; the first one plans the Updates and writes the lse.
template <int D, int EPI, int R, int G>
__device__ __forceinline__ void part_epilogue(const AttnParams& p, char* lds, int lane, int rg, int kgrp, int q0, int b, int hq0, int group, int part,
                                              int n_live, float lse_blk, bool not_a_number) {
  constexpr int CPRF = D / 4, RPI_OUT = 64 / CPRF, NIT = 32 / G / RPI_OUT;
  const int ql = lane & 31, rr = kgrp * (32 / G) + lane / CPRF, cc = lane % CPRF;
  const int n_rows = part_rows_total(p), n_valid = n_rows - (q0 + rg * 32);   // rows of this row group (32 or more: all)
  const bool own_row = kgrp == 0 && lane < 32 && ql < n_valid;

  if (n_live > 1) {
    const int64_t slot_row = ((int64_t)group * p.n_parts + part) * p.part_rows + rg * 32;
    float* const dst = p.part_out + slot_row * D + 4 * cc;
    if (G > 1) __syncthreads();
    else __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes are visible to all its lanes
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int r = it * RPI_OUT + rr;
      const f32x4 o = row_piece<D, R, G>(lds, rg, r, cc);
      if (r < n_valid) *reinterpret_cast<f32x4*>(dst + (int64_t)r * D) = o;
    }
    if (own_row) p.part_lse[slot_row + ql] = not_a_number ? __builtin_nanf("") : lse_blk;
    return;
  }
  float* const tab_w = reinterpret_cast<float*>(lds + Lds<D, R, G>::w) + rg * 32;
  int* const tab_mode = reinterpret_cast<int*>(lds + Lds<D, R, G>::mode) + rg * 32;
  int64_t* const off = reinterpret_cast<int64_t*>(lds + Lds<D, R, G>::off) + rg * 32;
  if (kgrp == 0 && n_valid > 0) {
    const int row = min(q0 + rg * 32 + ql, n_rows - 1), head = divide(p.by_sq, row), pos = row - head * p.Sq;
    const int64_t l_at = (int64_t)b * p.l_sb + (int64_t)(hq0 + head) * p.l_sh + (int64_t)pos * p.l_ss;
    const UpdatePlan pl = plan_update(EPI == kEpiMerge ? p.lse[l_at] : -INFINITY, lse_blk);
    if (lane < 32) {
      off[ql] = (int64_t)b * p.o_sb + (int64_t)(hq0 + head) * p.o_sh + (int64_t)pos * p.o_ss;
      tab_w[ql] = pl.w;
      tab_mode[ql] = pl.mode;
    }
    if (own_row) p.lse[l_at] = pl.new_lse;
  }
  if (G > 1) __syncthreads();
  else __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), as above
#pragma unroll
  for (int it = 0; it < NIT; it++) {
    const int r = it * RPI_OUT + rr;
    if (r >= n_valid) continue;
    f32x4 o = row_piece<D, R, G>(lds, rg, r, cc);
    const int64_t at = off[r] + 4 * cc;
    if (EPI == kEpiBf16) {
      bf16x4 ob;
#pragma unroll
      for (int e = 0; e < 4; e++) ob[e] = (__bf16)o[e];
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + at) = ob;
    } else {
      f32x4* const dst = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.out) + at);
      if (EPI == kEpiMerge) {
        UpdatePlan pl;
        pl.w = tab_w[r];
        pl.mode = tab_mode[r];
        pl.new_lse = 0.f;
        o = apply_update(pl, *dst, o);
      }
      *dst = o;
    }
  }
}

// EPI selects the epilogue: kEpiBf16 / kEpiF32 store block_out and block_lse; kEpiMerge folds
// the block straight into fp32 accumulators with the Update of Sec. 3.1 (no block_out round trip).
//
// PART is the form for grids that would leave most of the chip idle (a decode step, a short prompt
// behind a long cache).  (1) The rows of a workgroup are (query head of one K/V head's group, Query
// row) pairs when that needs fewer workgroups: a decode step with grouped heads then reads every key
// once instead of once per query head.  (2) The keys are cut into p.n_parts parts of p.part_keys
// keys, each computed exactly as a launch over that part alone would; the block results go to a
// scratch buffer in fp32 and fold_parts_kernel adds them up in key order (a fixed
// order: bitwise reproducible).  Bound: HBM for a decode step, MFMA otherwise, plus the fold.  Four decode steps
// over 8192 keys each (4 sequences, 32 heads on 8 K/V heads) 355 -> 136 us, 500 Query rows x 32 heads
// behind 12000 keys 216 -> 94 us against the plain form.
//
// FORM kChunks replays Algorithm 1 block by block: with block results that are rounded to bf16 on their way to the
// Update, or (chunks shorter than a sub-tile, which no reference of the running softmax can be kept for) in fp32.
// A workgroup keeps its Query tile of chunk c and runs through the K/V chunks in the order the schedule
// brings them, c, c + 1, ... mod n (causal: only those not after c); each block ends in the merging
// epilogue, the first one unrounded onto an empty accumulator.  One launch instead of two per block: no
// block result in memory, no idle tail between the blocks (chunks of 1502 rows x 16 heads fill 96 of 256
// compute units), the longest chunks first.  Bound: as the plain form, plus an epilogue for each block.
// Causal 6008 rows in 4 chunks, 16 heads: 401 -> 167 us in 256-row workgroups, 157 in shape 4 x 1; the same bits as the steps where both have
// as many key groups.
//
// FORM kSegments and kPartSegments are the plain and the partitioned form for launches that take a row's exponent reference anew
// every p.renew keys (rings of several segments, and block steps that round as their parts would).  Kernels of their own: the tests for a renewal and the
// bodies of inner tiles that hold one are a quarter of the code, and a short call runs through most of the code once, from a cold instruction cache
// (8 heads of 512 rows on as many keys 9.42 -> 9.29 us without them, 16 at D 64 7.42 -> 7.31).
template <int D, int EPI, int FORM, int R, int G, int NS = ring_depth(D, R, G)>
__device__ __forceinline__ void attend(const AttnParams& p) {
  constexpr bool PART = FORM == kPart || FORM == kPartSegments, CHUNKS = FORM == kChunks;
  constexpr int W = R * G, BM = 32 * R;    // waves, Query rows of a workgroup
  static_assert(!CHUNKS || EPI == kEpiMerge, "blocks of the chunk form are merged");
  constexpr int RB = 2 * D;
  constexpr int KS = D / 16;               // MFMA k-steps over the head dim
  constexpr int DB = D / 32;               // 32-wide d blocks of the output
  constexpr int CPR = D / 8;               // 16-byte chunks per row
  typedef Lds<D, R, G, NS> L;
  constexpr int BN = tile_keys<D, R, G, NS>();   // keys per LDS tile
  constexpr int TILE_BYTES = BN * RB;
  constexpr int RPI = 1024 / RB;           // tile rows one wave-wide 16-byte load instruction covers
  constexpr int IPW = BN / RPI / W;        // load instructions per wave, tile and tensor
  constexpr int SUB = 32;                  // keys per sub-tile (one MFMA row block)
  constexpr int NSUB = BN / SUB;           // sub-tiles per tile
  constexpr int NSW = NSUB / G;            // sub-tiles of one key group (= steps of a wave) per tile
  constexpr int KA = NSW == 1 ? 4 : 3, VA = NS - 2;   // K and V tile issued in tile u: u + KA, u + VA
  constexpr bool TRIO = G > 1 && NS == 3;
  constexpr int NG = NSW * NS % 2 ? 2 * NS : NS;      // tiles after which ring slots and register sets come round
  static_assert(NSUB % G == 0 && (NSW * NG) % 2 == 0, "the S / P register sets alternate with the step parity");
  static_assert(IPW >= 1, "tile too small for the workgroup");
  static_assert(FORM != kPartSegments || G == 1, "packed rings: one key group (see choose_shape)");
  static_assert((!PART || L::tables(FORM) >= L::sums) && (!in_segments(FORM) || G == 1 || L::tables(FORM) > L::refs),
                "the row offsets and the references lie in the LDS that is asked for");

  extern __shared__ __attribute__((aligned(1024))) char lds[];  // K ring | V ring

  // which batch, head and query tile this workgroup computes (wave-uniform)
  int qt, b, hq, hk;
  PartBlock pb = {0, 0, 0, 0, 0, 0};
  if constexpr (PART) {
    if (!decode_part(p, pb)) return;
    qt = pb.tile; b = pb.b; hq = pb.hq0; hk = pb.hk;
  } else {
    decode_block(p, qt, b, hq, hk);
  }
  int chunk = 0;
  if constexpr (CHUNKS) {   // grid y runs over (chunk, query tile), both from the last on
    const int y = (int)blockIdx.y / p.n_qtiles;
    chunk = p.chunk_end - 1 - y;
    qt += y * p.n_qtiles;
  }
  const int64_t chunk_row = (int64_t)chunk * p.Sq;
  // Chunk form at D 64 with one key group: what every block can compute anew is not held from block to block, neither in vector registers (168 for
  // three workgroups a compute unit: 4 spilled, and a kernel with scratch starts later) nor in scalar ones, whose spills take vector registers.  Causal
  // blocks of 600 rows in 4 chunks, 64 heads 86.7 -> 85.4 us, 96 heads of 300 rows in 4 chunks 99.2 -> 95.7.  (At D 128 nothing but scalars spills, and counting anew costs
  // more: 6008 rows in 4 chunks, 16 heads 161 -> 168.)
  constexpr bool LEAN = CHUNKS && G == 1 && D == 64;
  const int wave_id = LEAN ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
  f32x16 o_acc[DB];         // O^T of the wave's rows, not yet divided by the sums
  float m_ref, l_run;       // exponent reference of the lane's row, in raw (unscaled) score units; the lane's share of its sum of exp

  // Chunk form, one key group: the Update of block `done`, whose result is in the registers.  Between two blocks a wave's accumulators lie
  // in its rows of `out` as they lie in its lanes, 16 bytes of every lane side by side, so blocks before the last need no transposition
  // through LDS: the rings are free at once and the next block's first loads go out in front of the Update, whose accumulator loads come in behind them (one after
  // the other the two took 4.8 us of a block's 20; causal 6008 rows in 4 chunks, 16 heads 164.4 -> 157.5 us; not to wait for its stores in front of the next block gives nothing).  A wave with fewer than 32 rows has no place for that and keeps every piece where it belongs.
  constexpr bool IN_LANES = CHUNKS && G == 1;
  auto chunk_update = [&](int done, bool last) __attribute__((always_inline)) {
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), ql = lane & 31, hf = lane >> 5;
    int bb = b, hh = hq, wave = LEAN ? wave_id : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if constexpr (LEAN) asm volatile("" : "+s"(bb), "+s"(hh), "+s"(wave));
    const int qw0 = qt * BM + wave * 32, n_valid = p.Sq - qw0;
    if (n_valid <= 0) return;
    constexpr int CPRF = D / 4, RPI_OUT = 64 / CPRF, NIT = 32 / RPI_OUT;
    static_assert(NIT == 4 * DB, "as many pieces a lane as rows a lane touches");
    const bool whole = n_valid >= 32;
    const int rr = lane / CPRF, cc = lane % CPRF;
    float* const rows = reinterpret_cast<float*>(p.out) + (int64_t)bb * p.o_sb + (int64_t)hh * p.o_sh + (chunk_row + qw0) * p.o_ss;
    float* const place = whole ? rows + (int64_t)rr * p.o_ss + 4 * cc : rows + (int64_t)min(ql, n_valid - 1) * p.o_ss + 4 * hf;
    const int64_t next = whole ? (int64_t)RPI_OUT * p.o_ss : 8;
    f32x4 x[NIT];
#pragma unroll
    for (int it = 0; it < NIT; it++)
      x[it] = done > 0 ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(place + it * next)) : f32x4{0.f, 0.f, 0.f, 0.f};
    float* const l_at = p.lse + (int64_t)bb * p.l_sb + (int64_t)hh * p.l_sh + (chunk_row + qw0 + min(ql, n_valid - 1)) * p.l_ss;
    const float l_tot = half_swap_sum(l_run), inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    UpdatePlan pl = plan_update(done > 0 ? *l_at : -INFINITY, l_tot > 0.f ? m_ref * p.scale + logf(l_tot) : -INFINITY);
    if (done == 0) pl.mode = 2;   // a first block is stored as it is, also where it is NaN (with lse -inf)
    if (hf == 0 && ql < n_valid) *l_at = pl.new_lse;
    char* const my = lds + wave * (32 * 4 * D);
    const bool round = done > 0 && p.chunk_bf16;
    float* dst = place;
    if constexpr (LEAN) asm volatile("" : "+v"(dst));   // the loads' addresses are not held for the stores
#pragma unroll
    for (int it = 0; it < NIT; it++, dst += next) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        o[e] = o_acc[it >> 2][4 * (it & 3) + e] * inv;
        if (round) o[e] = (float)(__bf16)o[e];
      }
      o = apply_update(pl, x[it], o);
      if (whole && last) *reinterpret_cast<f32x4*>(my + ql * (4 * D) + (((2 * it + hf) ^ (ql & 15)) << 4)) = o;
      else if (ql < n_valid) __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(dst));
    }
    if (whole && last) {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes are visible to all its lanes
#pragma unroll
      for (int it = 0; it < NIT; it++) x[it] = row_piece<D, R, 1>(my, 0, it * RPI_OUT + rr, cc);
#pragma unroll
      for (int it = 0; it < NIT; it++) __builtin_nontemporal_store(x[it], reinterpret_cast<f32x4*>(place + it * next));
    }
  };
  int done = -1;   // block whose Update is still to come
  for (int block = 0; block < (CHUNKS ? p.n_chunks : 1); block++) {
  const int kv_chunk = CHUNKS ? (chunk + block < p.n_chunks ? chunk + block : chunk + block - p.n_chunks) : 0;
  if (CHUNKS && p.causal && kv_chunk > chunk) continue;
  int tid = threadIdx.x, wave;
  if constexpr (LEAN) {
    unsigned zero = 0;
    wave = wave_id;
    asm volatile("" : "+v"(zero), "+s"(wave));
    tid = wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
  } else {
    if constexpr (CHUNKS) asm volatile("" : "+v"(tid));   // nothing derived from it is held in registers from block to block (179 spills otherwise)
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept in an SGPR
  }
  const int lane = tid & 63, ql = lane & 31, hf = lane >> 5;
  const int rg = G == 1 ? wave : wave % R, kgrp = G == 1 ? 0 : wave / R;   // row group, key group
  const bool causal = CHUNKS ? p.causal && block == 0 : p.causal != 0;
  int Sk = p.Sk, causal_off = p.causal_off;
  const int q0 = qt * BM, qw0 = q0 + rg * 32;
  const int qrow = qw0 + ql;
  // rows of this workgroup's row space: the Query rows of one head, or of a whole group of heads
  const int n_rows = PART ? part_rows_total(p) : p.Sq;
  const int qrow_ld = min(qrow, n_rows - 1);
  // Query position of this lane's row (its head is hq + lane_head), the smallest and largest position
  // of the wave's rows, the largest of the workgroup's: what the causal rule needs
  int lane_head = 0, lane_pos = qrow, pos_first = qw0, pos_last = min(qw0 + 31, p.Sq - 1), pos_last_wg = min(q0 + BM, p.Sq) - 1;
  int n_live = 1;   // parts of the keys that any row of this workgroup sees
  if constexpr (PART) {
    lane_head = divide(p.by_sq, qrow_ld);
    lane_pos = qrow_ld - lane_head * p.Sq;
    int unused;
    pos_span(p, min(qw0, n_rows - 1), 32, pos_first, pos_last);
    pos_span(p, q0, BM, unused, pos_last_wg);
    n_live = live_parts(p, pos_last_wg);
    if (pb.part >= n_live) return;
    const int k0 = pb.part * p.part_keys;
    Sk = min(Sk - k0, p.part_keys);
    causal_off -= k0;
  }

  // Key range of this workgroup in tiles (needed to start the loads; the wave's own range follows below)
  int kv_end = Sk;
  if (causal) kv_end = max(0, min(Sk, pos_last_wg + causal_off + 1));
  const int n_tiles = (kv_end + BN - 1) / BN;

  const __bf16* kg = p.k + (int64_t)b * p.k_sb + (int64_t)hk * p.k_sh;
  const __bf16* vg = p.v + (int64_t)b * p.v_sb + (int64_t)hk * p.v_sh;
  if constexpr (CHUNKS) {
    kg += (int64_t)kv_chunk * p.Sk * p.k_ss;
    vg += (int64_t)kv_chunk * p.Sk * p.v_ss;
  }
  if constexpr (PART) {
    kg += (int64_t)pb.part * p.part_keys * p.k_ss;
    vg += (int64_t)pb.part * p.part_keys * p.v_ss;
  }

  // Direct global -> LDS staging (no VGPRs, no ds_write): one wave-wide instruction deposits
  // lane l's 16 bytes at lds_base + 16*l, i.e. RPI consecutive tile rows.  The swizzle is
  // applied on the global side: the lane that fills LDS position (row, pc) fetches the chunk
  // the swizzle maps there.  Addresses are a wave-uniform 64-bit tile base (SGPR pair) plus a
  // per-lane 32-bit byte offset that never changes, so issuing a tile costs no vector
  // arithmetic.  Rows past the end of the keys re-read the last key (they are masked later):
  // the last, possibly partial, tile has its own clamped offsets.  Nothing is loaded beyond the last tile the workgroup
  // sees: what the ring holds there takes part in scores that are masked and in no product with V.  (A ring that ran ahead of its end
  // re-read the last tile five times, and the workgroup waited for that before it ended: 64 rows on 64 keys 6.47 -> 5.88 us.)
  const int last_tile = n_tiles - 1;
  unsigned k_off[IPW], v_off[IPW], k_off_last[IPW], v_off_last[IPW];
#pragma unroll
  for (int i = 0; i < IPW; i++) {
    const int row = (wave * IPW + i) * RPI + lane / CPR, pc = lane % CPR;
    const int kc = (pc ^ ((row / (256 / RB)) % CPR)) * 8;
    const int vswz = (D == 128) ? ((row & 3) << 1) : (row & 2);
    const int vc = ((((pc >> 1) ^ vswz) << 1) | (pc & 1)) * 8;
    const int row_last = max(0, min(row, Sk - 1 - last_tile * BN));
    k_off[i] = (unsigned)(((int64_t)row * p.k_ss + kc) * 2);
    v_off[i] = (unsigned)(((int64_t)row * p.v_ss + vc) * 2);
    k_off_last[i] = (unsigned)(((int64_t)row_last * p.k_ss + kc) * 2);
    v_off_last[i] = (unsigned)(((int64_t)row_last * p.v_ss + vc) * 2);
  }
  // Issued as inline asm: the compiler would otherwise treat every later LDS read as possibly
  // aliasing the in-flight load and drain vmcnt to 0 in front of it, serialising the pipeline;
  // here completion is waited for explicitly, one tile ahead of the first use.
  // The statement overwrites m0.  The compiler reserves m0 and sets it itself right before each of
  // its own uses (dynamic register indexing, LDS-direct forms), none of which this kernel
  // contains: every register-array index is a compile-time constant.  (m0 cannot be named in
  // the clobber list: it is a reserved register and the compiler rejects the promise.)
  const unsigned lds_base = (unsigned)(unsigned long)(lptr_t)lds;
  auto dma16 = [&](const __bf16* base, unsigned off, unsigned lds_off) __attribute__((always_inline)) {
    const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base + lds_off);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0v), "v"(off), "s"(base) : "memory");
  };
  // Tiles are issued strictly in order, so the tile base is a running wave-uniform pointer.
  const __bf16* k_next = uniform_ptr(kg);
  const __bf16* v_next = uniform_ptr(vg);
  const int64_t k_tile_stride = (int64_t)BN * p.k_ss, v_tile_stride = (int64_t)BN * p.v_ss;
  int k_left = last_tile, v_left = last_tile;  // tiles still ahead of the pointer
  auto issue_k = [&](int slot) __attribute__((always_inline)) {
    if (k_left < 0) return;
    const bool last = k_left == 0;
#pragma unroll
    for (int i = 0; i < IPW; i++)
      dma16(k_next, last ? k_off_last[i] : k_off[i], slot * TILE_BYTES + (wave * IPW + i) * 1024);
    k_next = uniform_ptr(k_next + k_tile_stride);
    k_left--;
  };
  auto issue_v = [&](int slot) __attribute__((always_inline)) {
    if (v_left < 0) return;
    const bool last = v_left == 0;
#pragma unroll
    for (int i = 0; i < IPW; i++)
      dma16(v_next, last ? v_off_last[i] : v_off[i], (NS + slot) * TILE_BYTES + (wave * IPW + i) * 1024);
    v_next = uniform_ptr(v_next + v_tile_stride);
    v_left--;
  };

  // ---- prologue: the wave's Query rows and K_0..K_2, V_0, V_1 into the rings.  The loads go out
  // before the rest of the set-up (this wave's key range, LDS read addresses, cleared accumulators)
  // so that their latency, the longest wait of a workgroup's life, runs under that arithmetic.
  //
  // The Query rows take the same way as K: whole rows, 1 KiB an instruction, into the wave's own share of ring slots that are filled
  // last (V from the top, at D = 128 with two instructions a tile K_3 as well), swizzled alike, and from there into the
  // B-operand layout.  With one key group at D = 128 a quarter of them lies behind the tables, so that K_3 (128-row workgroups) and V_1 (256-row ones) need not wait for them (64 heads of 1024,
  // causal, 0.9 % less, 128 heads of 827 rows on 184 keys 1.7 %).  (Straight into registers a quad of lanes touches four rows, and 64 such loads kept a compute unit's
  // vector-memory path busy for 1.5 us in front of the later waves' K/V loads: 256 keys in 4 segments x 2 heads 7.93 -> 7.71 us, 4 x 2
  // heads of 1503 20.9 -> 20.5, 500 rows x 32 heads on 12500 keys 95.4 -> 93.8; long launches, which the power limit bounds, the same.)  A wave touches its own share
  // only, so no barrier is needed; what the slots are for is loaded behind it.
  constexpr int QP = 32 * RB / 1024, Q_SLOTS = (QP + IPW - 1) / IPW;   // instructions, ring slots
  static_assert(Q_SLOTS <= 4 && (Q_SLOTS <= NS - VA || NS == 4), "Query rows fit into slots that are filled last");
  constexpr bool APART = L::query > 0;   // the last slot's pieces lie behind the tables; the third slot is K_3's of 256-row workgroups
  static_assert(!APART || (Q_SLOTS == 4 && IPW == 2 && L::tables(FORM) % 1024 == 0), "two pieces of every wave lie apart");
  constexpr bool V1_LATE = VA == 2 && (APART ? KA == 4 : Q_SLOTS >= 3), K3_LATE = KA == 4 && Q_SLOTS == 4 && !APART;
  constexpr int AHEAD = IPW * ((KA == 4 && !K3_LATE && !TRIO ? 3 : 2) + (VA == 2 && !V1_LATE ? 2 : 1)), LATE = IPW * ((V1_LATE ? 1 : 0) + (K3_LATE ? 1 : 0));
  auto q_slot = [&](int piece) __attribute__((always_inline)) -> int {   // LDS offset of a piece (RPI rows)
    const int s = piece / IPW;
    if (APART) {
      const int slot = s == 2 && KA == 3 ? NS - 1 : 2 * NS - 1 - s;
      return (s == 3 ? L::tables(FORM) : slot * TILE_BYTES) + (wave * IPW + piece % IPW) * 1024;
    }
    return (2 * NS - 1 - s - (s == 3 ? 1 : 0)) * TILE_BYTES + (wave * IPW + piece % IPW) * 1024;
  };
  auto issue_q = [&]() __attribute__((always_inline)) {
    const __bf16* const qb = p.q + (int64_t)b * p.q_sb + (int64_t)hq * p.q_sh + chunk_row * p.q_ss;
#pragma unroll
    for (int i = 0; i < QP; i++) {
      const int r = i * RPI + lane / CPR, at = min(qw0 + r, n_rows - 1);
      int head = 0, pos = at;
      if (PART && p.pack) {
        head = divide(p.by_sq, at);
        pos = at - head * p.Sq;
      }
      const __bf16* src = qb + (int64_t)pos * p.q_ss + ((lane % CPR) ^ ((r / (256 / RB)) % CPR)) * 8;
      if (PART) src += (int64_t)head * p.q_sh;
      const unsigned m0v = __builtin_amdgcn_readfirstlane(lds_base + q_slot(i));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0v), "v"(src) : "memory");
    }
  };
  // Behind K_0, which the first products need beside them (in front of it too a call of 2 x 6 heads of 340 rows on 652 keys at D 64 takes 8.43 us, behind it
  // 8.36), and in front of the other tiles, so that they are in their registers when K is there, where key groups make a launch's first steps count; behind all where
  // several workgroups share a compute unit or HBM bounds the launch.  us, in front / behind: 113 rows x 8 heads on 1314 keys at D 64 11.94 / 12.05,
  // bf16 blocks of 3488 rows in 8 chunks, 4 heads 52.96 / 53.74; 128 heads of 442 at D 64 11.67 / 11.31, four decode steps of 8192 keys 138.0 / 135.5.
  constexpr bool Q_FIRST = !PART && G > 1;
  if (n_tiles > 0) issue_k(0);
  // At most 16 rows, a decode step's, go straight into registers behind the tiles: of the pieces of 32 rows most would be loaded for nothing, and the way through LDS is
  // one wait longer.  One row x 8 heads on 2 K/V heads of 2048 keys 12.02 -> 11.55 us (11.85 before the rows went through LDS), 8 heads of 1500
  // 12.54 -> 12.13; from 24 rows on LDS is faster (24 x 8 heads on 512 keys, which is not cut, 9.23 straight and 9.06).  In the chunk form at D 64: 4 chunks of one row
  // 16.16 -> 15.78.  Not where the choice costs more than it gives: cut launches at D 64 (4 sequences on 8192 keys 18.23 -> 18.69), uncut ones (64 rows x 4 heads
  // on 512 keys at D 64 1 %), the chunk form at D 128 (scalar spills, 1 - 2 %).
  constexpr bool FEW = G > 1 && (D == 128 ? PART : CHUNKS);
  const bool straight = FEW && n_rows <= 16;
  if (Q_FIRST && !straight && (!CHUNKS || qw0 < n_rows)) issue_q();
  constexpr bool RENEW = in_segments(FORM);
  constexpr bool KNOWN = RENEW && G > 1;    // references of later segments are found in the prologue
  // Key range of this wave (in 32-key sub-tiles): behind the loads, but where rows of K are loaded by it.
  int wave_kv_end, jw;      // jw: sub-tiles this wave has visible keys in
  int kmask_from;           // a sub-tile starting at kstart needs masking iff kstart > kmask_from
  // Where the reference is renewed for a segment that starts at key r: at r, or at the next multiple of 2^renew_log2 keys while that
  // lies in the stretch (up to renew_end) that no row of the wave needs a mask for, four quarters and more before the keys end.  A
  // multiple is a group of inner tiles of 256-row workgroups; a function of the wave's rows and the keys alone, so every shape of the
  // workgroup renews at the same keys and rounds the same weights.
  const int renew_log2 = p.renew_log2;
  int renew_end;
  auto wave_range = [&]() __attribute__((always_inline)) {
    wave_kv_end = 0;
    if (qw0 < n_rows) {
      wave_kv_end = Sk;
      if (causal) wave_kv_end = max(0, min(Sk, pos_last + causal_off + 1));
    }
    jw = (wave_kv_end + SUB - 1) / SUB;
    int from = Sk - SUB;
    if (causal) from = min(from, pos_first + causal_off - SUB + 1);
    kmask_from = __builtin_amdgcn_readfirstlane(from);
    renew_end = 0;
    if (RENEW && p.renew >= 1 << renew_log2) {
      const int j = min(jw, kmask_from >= 0 ? kmask_from / SUB : -1) - (1 << (renew_log2 - 7)) + 1;   // a quarter's last sub-tile must pass both tests
      const int quarters = j < 0 ? 0 : min(j >> (renew_log2 - 7), ((Sk - 1) >> (renew_log2 - 2)) - 4) + 1;
      renew_end = __builtin_amdgcn_readfirstlane(max(0, quarters) >> 2 << renew_log2);
    }
  };
  auto renew_key = [&](int r) __attribute__((always_inline)) -> int {
    return max(r, min((r + (1 << renew_log2) - 1) >> renew_log2 << renew_log2, renew_end));
  };
  // The first sub-tiles of later segments, whose largest scores are the references there (see masked_max below): K as it lies in memory is the
  // A operand, so their rows go straight into registers, two references at a time.  Behind Q and in front of the other tiles, so that the
  // one wait for Q covers them too (fetched behind it they cost a second latency: 2 heads of 256 rows in 4 segments 10.76 -> 9.72 us at D 128, with the
  // renewals in front of the stream; at D 64 8.60 -> 7.50, 8 heads of 1024 17.6 -> 16.6 and 13.1 -> 12.3).
  int n_ref = 0;   // references of later segments that the wave needs, at most L::max_refs (see choose_shape)
  bf16x8 ref_a[KNOWN ? KS : 1], ref_b[KNOWN ? KS : 1];
  auto load_ref = [&](int s, auto& kf) __attribute__((always_inline)) {
    const __bf16* kp = kg + (int64_t)min(renew_key((s + 1) * p.renew) + ql, Sk - 1) * p.k_ss + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) kf[ks] = *reinterpret_cast<const bf16x8*>(kp + 16 * ks);
  };
  if constexpr (KNOWN) {   // (launched with p.renew > 0 only)
    wave_range();
    n_ref = __builtin_amdgcn_readfirstlane(divide(p.by_renew, max(0, wave_kv_end - 1)));
    if (kgrp < n_ref) {
      load_ref(kgrp, ref_a);
      if (kgrp + G < n_ref) load_ref(kgrp + G, ref_b);
    }
  }
  if (n_tiles > 0) {
    issue_v(0);
    issue_k(1);
    if (VA == 2 && !V1_LATE) issue_v(1);
    issue_k(2);
    if (KA == 4 && !K3_LATE && !TRIO) issue_k(3);
  }
  // (A wave without rows loads none, and what it then reads takes part in nothing: with clamped rows loaded all the same 32 rows x 16 heads on 32 keys take
  // 5.57 us, 5.16 without, 64 rows x 4 heads on 64 keys at D 64 4.58 and 4.34.  In front of the other tiles
  // of a plain launch the test costs as much as it gives, 0.5 - 1 % more; the chunk form, whose blocks load their rows again and again, takes it there too: 4 chunks of 8 rows
  // x 16 heads 22.25 -> 21.90, of 31 23.42 -> 22.96.)
  if (!Q_FIRST && !straight && qw0 < n_rows) issue_q();
  bf16x8 qf[KS];   // Q^T fragments: lane (q, hf) holds Q[q][16*ks + 8*hf .. +7] for every k-step
  if (FEW && straight) {
    if (n_tiles > 0) {   // (nothing lies in their slots)
      if (K3_LATE) issue_k(3);   // (first: it is read one tile earlier than V_1)
      if (V1_LATE) issue_v(1);
    }
    const __bf16* qp = p.q + (int64_t)b * p.q_sb + (int64_t)(PART ? hq + lane_head : hq) * p.q_sh + (PART ? lane_pos : chunk_row + qrow_ld) * p.q_ss;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks + 8 * hf);
  }
  if constexpr (IN_LANES) {
    if (done >= 0) chunk_update(done, false);
    done = block;
  }

  if constexpr (!KNOWN) wave_range();
  // wave-uniform loop bounds, forced into scalar registers so that every per-step test is one compare
  const int jw_own = G == 1 ? jw : max(0, jw - kgrp + G - 1) / G;                     // those of this key group: kgrp, kgrp + G, ...
  const int jw_first = __builtin_amdgcn_readfirstlane(jw_own);                        // last allowed step that opens a tile
  const int jw_in = __builtin_amdgcn_readfirstlane(min(jw_own, NSW * n_tiles - 1));   // last allowed step inside a tile

  // Per-lane LDS read offsets.
  // K operand: lane (key = ql, hf) reads chunk 2*ks + hf of row 32*kt + ql.
  // (All read addresses are LDS byte addresses with the ring base folded in, so that ring
  // slot and sub-tile offsets are instruction immediates.)
  unsigned k_rd[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ks++) k_rd[ks] = lds_base + kgrp * (SUB * RB) + k_lds_off<D>(ql, 2 * ks + hf);
  // V^T operand through the transposing read: within each group of 16 lanes, lane i supplies
  // the address of row (i/4) of the 4-key group, 8-byte segment (i%4) of the 16 d's the
  // group covers, and receives the 4 keys of d = i.  (The V ring base is folded in.)
  unsigned v_rd[DB];
  {
    const int i16 = lane & 15, gq = (lane >> 4) & 1;
    const int row = 4 * hf + (i16 >> 2);
#pragma unroll
    for (int db = 0; db < DB; db++)
      v_rd[db] = lds_base + NS * TILE_BYTES + kgrp * (SUB * RB) + v_lds_off<D>(row, 4 * db + 2 * gq) + (i16 & 3) * 8;
  }

#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int i = 0; i < 16; i++) o_acc[db][i] = 0.f;
  // Largest sub-tile sum (16 weights of one row) the fast path accepts: 2^80.  The weights, their
  // bf16 roundings and the fp32 accumulators all carry an 8-bit exponent, so precision does not
  // depend on the magnitude; the cap only has to keep sums over all keys (up to 2^30, i.e. 2^25
  // sub-tiles, |v| up to 2^7) below 2^127.  A score must therefore exceed the reference by 55 (in natural
  // units) before the reference is moved: on all but pathological inputs that happens once, at
  // the row's first keys.
  constexpr float kSumCap = 0x1p80f;
  m_ref = -INFINITY;
  float mc = 0.f;           // m_ref * c2 (0 while m_ref is -inf), kept alongside m_ref
  l_run = 0.f;
  float sum_cap = -1.f;     // largest sub-tile sum the fast path accepts; negative until m_ref is finite and where it is renewed
  // Shapes of fewer than 256 rows renew inside a group of inner tiles too: a group of 4 x 1's (192 keys at D 64) may hold a key at which
  // the reference is renewed, and block steps renew at any multiple of 128 keys.  Such a group has a body of its own, whose steps look at
  // renew_at without a branch (one key group): the cap is lowered and the slow path does the rest.  (In every inner step the look costs
  // the DiT shape 0.6 % and 1 head of 9984 rows in 2 segments 4 %; renewed by the general body alone 4 heads of 2048 in 8 at D 64 take 28.2
  // us for 24.8, 2 x 16 heads of 499 rows on 3201 keys 39.4 for 36.0.)
  constexpr bool RENEW_INNER = RENEW && R < 8;
  int segment_at = RENEW ? p.renew : 0;                                      // key at which the next segment starts
  int renew_at = RENEW && p.renew > 0 ? renew_key(segment_at) : 0x7fffffff;  // the first step that starts here or later renews m_ref
  int segment = -1;         // later segment the wave is in, -1: the first one
  constexpr bool REF_AHEAD = KNOWN && D == 64 && !TRIO;   // read a segment ahead (at D 128 the register for it is one too many)
  float next_ref = 0.f;
  auto next_segment = [&]() __attribute__((always_inline)) {
    if (!KNOWN) sum_cap = -1.f;
    segment_at += p.renew;
    renew_at = renew_key(segment_at);
    segment++;
  };
  const float c2 = p.scale * 1.4426950408889634f;  // scale * log2(e)

  // ---- one step ---------------------------------------------------------------------
  // Step j (sub-tile j starts at key kstart) runs, as ONE interleaved instruction stream,
  //   MFMA : S_{j+1} = K_{j+1} Q^T   (NQK MFMAs, operands read from LDS by the PREVIOUS step)
  //          O += V_{j-1}^T P_{j-1}^T (NPV MFMAs, operands read from LDS during the QK half)
  //   LDS  : while the PV half runs, the K operands of step j+1 are read (into `pre`), so the
  //          read stream never stops at a step boundary or at a barrier (the tile they come
  //          from became visible a whole tile earlier)
  //   VALU : P_j = exp2((S_j - m_ref) * c2) and its row sums
  // QK goes first so that S_{j+1} is complete long before the next step's softmax reads it.
  //
  // P = exp2((s - m_ref) * scale*log2e) with an exponent reference m_ref that is NOT the
  // running maximum: any reference gives the same out = O/l and lse = m_ref*scale + ln l, so
  // the common path takes no row maximum.  Since P >= 0, a sub-tile sum <= kSumCap bounds
  // every P.  Only if some lane's sum exceeds the cap (or is NaN), or the reference is still
  // -inf, the slow path runs after the stream: row maximum, raise the reference, rescale l
  // and the O accumulators (which by then include P_{j-1}, consistently), redo the exponentials.
  // With p.renew the slow path also runs once every p.renew keys and may lower the reference to its
  // sub-tile's maximum: the weight of that maximum is then 1 and bf16 holds it exactly.  One
  // reference for a whole sequence has one such weight a row where blocks attended one by one have one each,
  // and the rounding of the largest weights is most of the error: 256 keys 1.42e-3 in blocks of 64, 1.60e-3 with one
  // reference, 1.42e-3 renewed every 64 keys.
  // Row sums use the unrounded fp32 P: summing the bf16-rounded weights would cost up to
  // 2^-8 relative in l, more than the 1e-3 budget of lse for rows that see only a few keys.
  //
  // The stream is written out in the order it should issue - per MFMA: one operand's LDS
  // reads, the MFMA, and a slice of the softmax whose three dependent stages (fma, exp2,
  // add/convert) are staggered across consecutive slices - and pinned with sched_barrier.
  constexpr int NPV = 2 * DB, NQK = KS;
  static_assert(NPV == NQK, "the two halves of a step carry the same number of MFMAs");
  typedef const s16x4 __attribute__((address_space(3)))* lds_tr_ptr;
  typedef const bf16x8 __attribute__((address_space(3)))* lds_b128_ptr;
  auto load_k = [&](int ks, unsigned k_imm) __attribute__((always_inline)) -> bf16x8 {
    return *(lds_b128_ptr)(unsigned long)(k_rd[ks] + k_imm);
  };
  auto load_v = [&](int i, unsigned v_imm) __attribute__((always_inline)) -> bf16x8 {
    const int t = i / DB, db = i % DB;
    const unsigned a = v_rd[db] + v_imm + 16 * t * RB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(lds_tr_ptr)(unsigned long)a);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(lds_tr_ptr)(unsigned long)(a + 8 * RB));
    const bf16x4 lo_b = __builtin_bit_cast(bf16x4, lo), hi_b = __builtin_bit_cast(bf16x4, hi);
    return __builtin_shufflevector(lo_b, hi_b, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  bf16x8 pre[NQK];  // K operands of the next step's QK half, read one step ahead

  auto step = [&](int kstart, auto first_c, auto v_imm_c, auto k_imm_next_c, f32x16& s_in, f32x16& s_out,
                  bf16x8 (&p_in)[2], bf16x8 (&p_out)[2], auto inner_c) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_c)::value != 0;   // no previous sub-tile: QK half only
    constexpr bool INNER = decltype(inner_c)::value != 0;   // every key of the sub-tile is visible to every row: no mask test
    constexpr bool CHECKED = decltype(inner_c)::value == 2; // and the reference may be renewed here
    constexpr int n_mfma = FIRST ? NQK : NQK + NPV;
    constexpr int EPM = 16 / n_mfma;  // softmax elements handled per MFMA slice
    static_assert(16 % n_mfma == 0, "softmax elements must divide evenly over the MFMAs");
    constexpr unsigned v_imm = decltype(v_imm_c)::value, k_imm_next = decltype(k_imm_next_c)::value;

    // Key groups know a segment's reference beforehand: the weights of this sub-tile are taken in it at once (the slow path below would
    // take them twice, 0.2 us a renewal), and what is summed so far follows behind the stream, whose PV half still adds weights in the old one.
    float renewed = 1.f;
    bool renew = false;
    if constexpr (KNOWN && !FIRST && (!INNER || CHECKED)) {
      if (__builtin_expect(kstart >= renew_at, 0)) {
        next_segment();
        if (segment < n_ref) {   // (else no row of the wave sees the segment)
          renew = true;
          const float* const at = reinterpret_cast<const float*>(lds + L::refs) + segment * BM + rg * 32 + ql;
          const float seg_ref = REF_AHEAD ? next_ref : *at;
          if (REF_AHEAD) next_ref = at[segment + 1 < n_ref ? BM : 0];
          // down as well, while the sum stays below 2^40 in the new units, as below; not where the row sees none of the keys
          const float lowered = half_swap_max(l_run) * __builtin_amdgcn_exp2f((m_ref - seg_ref) * c2);
          const bool take = seg_ref > m_ref || (seg_ref > -INFINITY && lowered <= 0x1p40f);
          const float m_new = take ? seg_ref : m_ref;
          renewed = m_new == m_ref ? 1.f : __builtin_amdgcn_exp2f((m_ref - m_new) * c2);
          l_run *= renewed;
          m_ref = m_new;
          if (m_ref > -INFINITY) {
            mc = m_ref * c2;
            sum_cap = kSumCap;
          }
        }
      }
    }

    if (!INNER && kstart > kmask_from) {  // some key of the sub-tile is past Sk or above this wave's first diagonal
      int limit = Sk - 1;
      if (causal) limit = min(limit, lane_pos + causal_off);
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const int key = kstart + 8 * (i >> 2) + 4 * hf + (i & 3);
        if (key > limit) s_in[i] = -INFINITY;
      }
    }

    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = 0.f;
    bf16x8 pv_ops[NPV], nxt[NQK];
    float tq[16], ex[16];
    unsigned pw[8];
    float ps0 = 0.f, ps1 = 0.f;
    // Softmax element group g (EPM elements) passes stage A (fma) in slice g-2, stage B (exp2) in
    // slice g-1 and stage C (sum, convert) in slice g, so the stream ends with the last MFMA
    // and nothing but the sum check is left behind it.  The convert is opaque to the compiler,
    // which would otherwise sink all of them behind the slow-path branch.
    auto stage_a = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < EPM; k++) tq[g * EPM + k] = __builtin_fmaf(s_in[g * EPM + k], c2, -mc);
    };
    auto stage_b = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < EPM; k++) ex[g * EPM + k] = __builtin_amdgcn_exp2f(tq[g * EPM + k]);
    };
    auto stage_c = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < EPM; k++) {
        const int e = g * EPM + k;
        if (e & 1) {
          ps1 += ex[e];
          asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(pw[e >> 1]) : "v"(ex[e - 1]), "v"(ex[e]));
        } else {
          ps0 += ex[e];
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < n_mfma; i++) {
      if (i < NQK) {
        if (FIRST) nxt[i] = load_k(i, k_imm_next);
        else pv_ops[i] = load_v(i, v_imm);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pre[i], qf[i], acc, 0, 0, 0);
      } else {
        const int j = i - NQK;
        nxt[j] = load_k(j, k_imm_next);
        o_acc[j % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pv_ops[j], p_in[j / DB], o_acc[j % DB], 0, 0, 0);
      }
      if (i == 0) {
        __builtin_amdgcn_sched_barrier(0);  // the first MFMA issues before any softmax work
        stage_a(0);
        stage_b(0);
        stage_a(1);
      }
      if (i + 1 < n_mfma) stage_b(i + 1);
      if (i + 2 < n_mfma) stage_a(i + 2);
      stage_c(i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int h = 0; h < 2; h++) p_out[h] = __builtin_bit_cast(bf16x8, u32x4{pw[4 * h], pw[4 * h + 1], pw[4 * h + 2], pw[4 * h + 3]});
    float psum = ps0 + ps1;
    if (KNOWN && renew) {
#pragma unroll
      for (int db = 0; db < DB; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) o_acc[db][i] *= renewed;
    }
    float cap = sum_cap;
    if (CHECKED && !KNOWN) cap = kstart >= renew_at ? -1.f : sum_cap;

    if (__builtin_expect(__any(!(psum <= cap)), 0)) {   // sum_cap < 0 while m_ref is -inf, so that case is included
      while (CHECKED && !KNOWN && kstart >= renew_at) next_segment();   // (once, the keys lie as far apart as a wave's sub-tiles; as an if it spills 31 SGPRs in shape 2 x 2 at D 64)
      float tmax = s_in[0];
#pragma unroll
      for (int i = 1; i < 16; i++) tmax = fmaxf(tmax, s_in[i]);
      tmax = half_swap_max(tmax);
      float m_new = fmaxf(m_ref, tmax);
      // Renewed: down as well, while what the row has summed so far stays below 2^40 in the new units (else weights of
      // this sub-tile do not count beside it).  Both halves of a row decide alike.
      if (__any(sum_cap < 0.f && m_ref > tmax)) {
        const float lowered = half_swap_max(l_run) * __builtin_amdgcn_exp2f((m_ref - tmax) * c2);
        if (sum_cap < 0.f && tmax > -INFINITY && lowered <= 0x1p40f) m_new = tmax;
      }
      const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * c2);  // m_ref = -inf -> 0; equal -> 1
      const float a = (m_new == -INFINITY) ? 0.f : alpha;                 // (-inf) - (-inf) would be NaN
      l_run *= a;
#pragma unroll
      for (int db = 0; db < DB; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) o_acc[db][i] *= a;
      m_ref = m_new;
      mc = (m_ref == -INFINITY) ? 0.f : m_ref * c2;
      sum_cap = (m_ref == -INFINITY) ? -1.f : kSumCap;
      const float mc2 = mc;
      float q0s = 0.f, q1s = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_in[i], c2, -mc2));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_in[i + 1], c2, -mc2));
        p_out[i >> 3][i & 7] = (__bf16)p0;
        p_out[i >> 3][(i & 7) + 1] = (__bf16)p1;
        q0s += p0;
        q1s += p1;
      }
      psum = q0s + q1s;
    }
    l_run += psum;
    s_out = acc;
#pragma unroll
    for (int i = 0; i < NQK; i++) pre[i] = nxt[i];
  };

  // Tiles that are certain to lie before the last tile of the keys need neither the choice between
  // the two offset sets nor the end-of-stream test.
  auto issue_k_inner = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < IPW; i++) dma16(k_next, k_off[i], slot * TILE_BYTES + (wave * IPW + i) * 1024);
    k_next = uniform_ptr(k_next + k_tile_stride);
    k_left--;
  };
  auto issue_v_inner = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < IPW; i++) dma16(v_next, v_off[i], (NS + slot) * TILE_BYTES + (wave * IPW + i) * 1024);
    v_next = uniform_ptr(v_next + v_tile_stride);
    v_left--;
  };

  // One exponent reference for a row and segment, whatever the number of key groups, and renewed at the same keys (renew_key): the
  // weights are then rounded alike in every shape of the workgroup (but where a row's scores leave the fast path's range: each key
  // group raises its own).  Those of later segments are found here, each by one key group, from K rows
  // that go straight into registers (K is the A operand as it lies in memory).
  auto masked_max = [&](const f32x16& s, int kstart) __attribute__((always_inline)) -> float {
    // every row sees all of it (at D 128 no choice where it is one maximum a launch or block: bf16 blocks of 2000 rows in 4 chunks, 4 heads, causal, 37.8 us with
    // it, 37.4 without, 8 heads of 512 9.40 and 9.34)
    if ((KNOWN || D == 64) && kstart <= kmask_from) {
      float t = s[0];
#pragma unroll
      for (int i = 1; i < 16; i++) t = fmaxf(t, s[i]);
      return half_swap_max(t);
    }
    int limit = Sk - 1;
    if (causal) limit = min(limit, lane_pos + causal_off);
    float t = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; i++) t = kstart + 8 * (i >> 2) + 4 * hf + (i & 3) <= limit ? fmaxf(t, s[i]) : t;
    return half_swap_max(t);
  };
  if (!straight) {
    if (Q_FIRST && last_tile >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD) : "memory");   // (all of the tiles above are on their way)
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    {
      const unsigned at = lds_base + q_slot(ql / RPI) + (ql % RPI) * RB;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) qf[ks] = *(const bf16x8 __attribute__((address_space(3)))*)(unsigned long)(at + (((2 * ks + hf) ^ ((ql / (256 / RB)) % CPR)) << 4));
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) asm volatile("" ::"v"(qf[ks]));   // Q is in registers
    if (n_tiles > 0) {
      if (K3_LATE) issue_k(3);   // (first: it is read one tile earlier than V_1)
      if (V1_LATE) issue_v(1);
    }
  }

  if constexpr (KNOWN) {
    auto find = [&](int s, const bf16x8 (&kf)[KS]) __attribute__((always_inline)) {
      f32x16 sr;
#pragma unroll
      for (int i = 0; i < 16; i++) sr[i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) sr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sr, 0, 0, 0);
      const float t = masked_max(sr, renew_key((s + 1) * p.renew));
      if (hf == 0) *reinterpret_cast<float*>(lds + L::refs + (s * BM + rg * 32 + ql) * 4) = t;
    };
    for (int s = kgrp; s < n_ref; s += 2 * G) {   // (rows past the last reference are clamped, what they give is not kept)
      find(s, ref_a);
      if (s + 2 * G < n_ref) load_ref(s + 2 * G, ref_a);
      if (s + G < n_ref) find(s + G, ref_b);
      if (s + 3 * G < n_ref) load_ref(s + 3 * G, ref_b);
    }
  }

  // (Where K rows were loaded into registers this is a wait that the compiler knows: it does not see that the one for Q covers them, takes rows of a reference
  // to be on their way still, and waits for everything in each group of inner tiles, where it needs their registers again.  With that wait / without, us at D 128:
  // 1 head of 28948 rows in 2 segments 394 / 384, a block step of 4 x 16 heads of 373 rows on 9183 keys, renewed at its parts, 141 / 125.)
  if (LATE > 0 && !KNOWN && last_tile >= 3 && !straight) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LATE) : "memory");
  else __builtin_amdgcn_s_waitcnt(0);
  wg_barrier();  // B_0
  if (REF_AHEAD && n_ref > 0) next_ref = *reinterpret_cast<const float*>(lds + L::refs + (rg * 32 + ql) * 4);

  // Ring protocol.  Step j = NSW*u + kt is the wave's step kt in tile u; it reads the V operands of
  // its sub-tile j-1 and the K operands of its sub-tile j+2.  Barrier B_u sits in front of step NSW*u.
  // NSW > 1: K_u is read in steps NSW*u-2 .. NSW*(u+1)-3 and V_u in steps NSW*u+1 .. NSW*(u+1).
  // Right after B_w every wave issues the loads of K_{w+3} and V_{w+2} into the slots
  // K_{w-1} and V_{w-2} vacated (all waves are past step NSW*w-1); they are first read two
  // tiles later, so each wave waits for its share (all but the newest 2*IPW loads, in order)
  // right before B_{w+2} (towards the end, where nothing more is issued, all of it).  NSW = 1: K_u is read in step u-2, so K_{w+4} goes into the slot of K_w, which
  // all waves have left behind B_w from w = 2 on; K_0 and K_1 are read before step 0, so the
  // slot of K_0 is free at B_1, where K_4 is issued in front of K_5.  K_{w+2} and V_{w-1}, read first in step w, were issued
  // before the newest 2*IPW loads at B_w.  Rings of three tiles (NSW = 2): K_{w+3} goes into the slot of K_w and V_{w+1}, issued in
  // front of it, into the one of V_{w-2}; all but the newest IPW loads have landed at B_{w+1}, and K_3 is issued at B_1, like K_4 above.
  // Rings of three tiles and NSW = 1 (three workgroups a compute unit): K_{w+4} goes into the slot of K_{w+1} and V_{w+1}, issued in front of it, into the one of
  // V_{w-2}, both read last in step w-1; K_{w+2} and V_{w-1}, read first in step w, were issued before the newest 2*IPW loads at B_w. K_3, V_1 and K_4
  // go out behind a barrier of their own in front of step 0, where K_0 and K_1 have been read.  Six tiles until slots and register sets come round.
  // S and P alternate between two register sets: even steps read sA / pB and write sB / pA,
  // odd steps the other way round, so no step has to copy its results.
  f32x16 sA, sB;
  bf16x8 pA[2], pB[2];
  constexpr unsigned SUBB = SUB * RB;  // bytes of one sub-tile inside a tile
  // Step NSW*u + kt of the tile in ring slot su (previous tile in sp); at_c = u % NG.
  auto tile_step = [&](int u, auto at_c, auto kt_c, auto inner_c) __attribute__((always_inline)) {
    constexpr int at = decltype(at_c)::value, su = at % NS, kt = decltype(kt_c)::value;
    constexpr bool INNER = decltype(inner_c)::value != 0;   // the step certainly runs and needs no mask
    constexpr int sp = (su + NS - 1) % NS;
    constexpr unsigned v_imm = kt == 0 ? sp * TILE_BYTES + (NSW - 1) * G * SUBB : su * TILE_BYTES + (kt - 1) * G * SUBB;
    constexpr unsigned k_imm = (su + (kt + 2) / NSW) % NS * TILE_BYTES + (kt + 2) % NSW * G * SUBB;
    constexpr bool even = (NSW * at + kt) % 2 == 0;
    const int j = NSW * u + kt;
    const int kstart = G == 1 ? j * SUB : (j * G + kgrp) * SUB;
    if (INNER || j <= (kt == 0 ? jw_first : jw_in)) {
      if (RENEW && !KNOWN && !INNER && __builtin_expect(kstart >= renew_at, 0)) next_segment();
      if (even) step(kstart, IC<0>{}, IC<(int)v_imm>{}, IC<(int)k_imm>{}, sA, sB, pB, pA, inner_c);
      else step(kstart, IC<0>{}, IC<(int)v_imm>{}, IC<(int)k_imm>{}, sB, sA, pA, pB, inner_c);
    }
  };
  auto first_scores = [&]() __attribute__((always_inline)) {
    // S_0 = K_0[0:32] Q^T, plain (nothing to overlap with yet); operands of step 0 (the wave's sub-tile 1)
#pragma unroll
    for (int i = 0; i < 16; i++) sA[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_k(ks, 0), qf[ks], sA, 0, 0, 0);
    if constexpr (G > 1) {   // the reference comes from the first sub-tile of all, key group 0's
      f32x16 sr;
#pragma unroll
      for (int i = 0; i < 16; i++) sr[i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ks++)
        sr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(lds_b128_ptr)(unsigned long)(k_rd[ks] - kgrp * (SUB * RB)), qf[ks], sr, 0, 0, 0);
      m_ref = masked_max(sr, 0);
      if (m_ref > -INFINITY) {
        mc = m_ref * c2;
        sum_cap = kSumCap;
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) pre[ks] = load_k(ks, 1 % NSW * G * SUBB + 1 / NSW * TILE_BYTES);
  };
  auto first_steps = [&]() __attribute__((always_inline)) {
    // step 0: S_1 alongside the softmax of sub-tile 0 (no PV yet); prefetch the K operands of sub-tile 2
    constexpr unsigned k_imm0 = 2 % NSW * G * SUBB + 2 / NSW * TILE_BYTES;
    step(kgrp * SUB, IC<1>{}, IC<0>{}, IC<(int)k_imm0>{}, sA, sB, pB, pA, IC<0>{});
    // the other steps of tile 0 (tiles 0 and 1 sit in ring slots 0 and 1)
    if constexpr (NSW > 1) tile_step(0, IC<0>{}, IC<1>{}, IC<0>{});
    if constexpr (NSW > 2) {
      tile_step(0, IC<0>{}, IC<2>{}, IC<0>{});
      tile_step(0, IC<0>{}, IC<3>{}, IC<0>{});
    }
  };
  if (n_tiles > 0) {
    if (KA == 3 && NS == 4) issue_k(3 % NS);
    if (!TRIO) issue_v(VA % NS);
    if constexpr (TRIO) {
      if (jw > 0) {
        first_scores();
#pragma unroll
        for (int ks = 0; ks < KS; ks++) asm volatile("" ::"v"(pre[ks]));
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
      wg_barrier();                         // K_3 and K_4 go where K_0 and K_1 lay, once every wave has read them
      issue_k(0);
      issue_v(1);
      issue_k(1);
      if (jw > 0) first_steps();
    } else if (jw > 0) {   // (one branch over both: with two, 8 heads of 2048 in 4 chunks of bf16 blocks at D 128 take 38.2 us for 38.0)
      first_scores();
      first_steps();
    }
  }
  // tiles u = 1 .. n_tiles: steps NSW*u .. NSW*u + NSW-1 (the last tile index only has its first
  // step, which folds in the PV product of the final sub-tile; its softmax sees only masked keys)
  auto tile_body = [&](int u, auto slot_c, auto inner_c, auto second_c) __attribute__((always_inline)) {   // slot_c = u % NG; second_c: u = 1
    constexpr int su = decltype(slot_c)::value % NS;
    constexpr bool INNER = decltype(inner_c)::value != 0;
    // vmcnt; of a ring of three also lgkmcnt(0): the slot that is filled behind the barrier was read in the step before it
    constexpr int none = NS == 3 ? 0x0070 : 0x0F70;
    if (INNER || (u + KA - 1 <= last_tile && !(NS == 3 && !TRIO && decltype(second_c)::value))) __builtin_amdgcn_s_waitcnt(none | (NS == 3 && !TRIO ? IPW : 2 * IPW));
    else __builtin_amdgcn_s_waitcnt(none);           // the tile before issued no K: everything that is on its way
    wg_barrier();                                    // B_u
    if ((KA == 4 || NS == 3) && !TRIO && decltype(second_c)::value) issue_k(0);   // K_4 of a ring of four, K_3 of a ring of three
    if (INNER) {   // K_{u+KA}, V_{u+VA}; first what is needed first
      if (NS == 3) issue_v_inner((su + VA) % NS);
      issue_k_inner((su + KA) % NS);
      if (NS == 4) issue_v_inner((su + VA) % NS);
    } else {
      if (NS == 3) issue_v((su + VA) % NS);
      issue_k((su + KA) % NS);
      if (NS == 4) issue_v((su + VA) % NS);
    }
    tile_step(u, slot_c, IC<0>{}, inner_c);
    if constexpr (NSW > 1) tile_step(u, slot_c, IC<1>{}, inner_c);
    if constexpr (NSW > 2) {
      tile_step(u, slot_c, IC<2>{}, inner_c);
      tile_step(u, slot_c, IC<3>{}, inner_c);
    }
  };
  static_assert(NSW == 1 || NSW == 2 || NSW == 4, "tile_body spells out 1, 2 or 4 steps");
  // Inner tiles: every step of the tile runs in this wave without masking (all its keys are visible
  // to all of the wave's rows and lie inside the K/V segment) and the tiles it puts on their way
  // lie before the segment's last tile.  They take a tile body without the per-step tests; the
  // remaining tiles take the general one.  Both bodies hold the same barrier and the same number
  // of loads, so the waves of a workgroup may disagree about where the inner tiles end.
  const int j_inner = min(min(jw, NSUB * n_tiles - 1), kmask_from >= 0 ? kmask_from / SUB : -1) - (NSUB - 1);   // last sub-tile of the tile must pass both tests
  int u_inner = j_inner < 0 ? -1 : j_inner / NSUB;
  u_inner = __builtin_amdgcn_readfirstlane(min(u_inner, last_tile - KA - 1));   // loads issued in tile u reach tile u + KA
  if (RENEW && !RENEW_INNER && p.renew > 0) u_inner = min(u_inner, renew_end / BN - 1);   // up to there the reference is renewed where a group starts
  // tiles 1 .. NG - 1 (tile 0 was the prologue)
  if (1 <= n_tiles) tile_body(1, IC<1>{}, IC<0>{}, IC<1>{});
  if (2 <= n_tiles) tile_body(2, IC<2>{}, IC<0>{}, IC<0>{});
  if (NG > 3 && 3 <= n_tiles) tile_body(3, IC<3 % NG>{}, IC<0>{}, IC<0>{});
  if (NG > 4 && 4 <= n_tiles) tile_body(4, IC<4 % NG>{}, IC<0>{}, IC<0>{});
  if (NG > 5 && 5 <= n_tiles) tile_body(5, IC<5 % NG>{}, IC<0>{}, IC<0>{});
  // Groups of NG tiles: first the groups of inner tiles (up to where the reference is renewed, and on from there; see RENEW_INNER), then
  // general ones to the end.
  auto group = [&](int u, auto inner_c) __attribute__((always_inline)) {
    tile_body(u, IC<0>{}, inner_c, IC<0>{});
    tile_body(u + 1, IC<1>{}, inner_c, IC<0>{});
    tile_body(u + 2, IC<2>{}, inner_c, IC<0>{});
    if constexpr (NG > 3) tile_body(u + 3, IC<3 % NG>{}, inner_c, IC<0>{});
    if constexpr (NG > 4) {
      tile_body(u + 4, IC<4 % NG>{}, inner_c, IC<0>{});
      tile_body(u + 5, IC<5 % NG>{}, inner_c, IC<0>{});
    }
  };
  int u0 = NG;
  while (u0 + NG - 1 <= u_inner) {
    if (!RENEW_INNER && u0 * BN >= renew_at) next_segment();
    const int stop = RENEW_INNER ? min(u_inner, (int)((unsigned)renew_at / BN) - 1) : min(u_inner, (int)(((unsigned)renew_at - 1) / BN) + NG - 1);
    for (; u0 + NG - 1 <= stop; u0 += NG) group(u0, IC<1>{});
    if (RENEW_INNER && u0 + NG - 1 <= u_inner) {
      group(u0, IC<2>{});
      u0 += NG;
    }
  }
  for (; u0 <= n_tiles; u0 += NG) {
    tile_body(u0, IC<0>{}, IC<0>{}, IC<0>{});
    if (u0 + 1 <= n_tiles) tile_body(u0 + 1, IC<1>{}, IC<0>{}, IC<0>{});
    if (u0 + 2 <= n_tiles) tile_body(u0 + 2, IC<2>{}, IC<0>{}, IC<0>{});
    if (NG > 3 && u0 + 3 <= n_tiles) tile_body(u0 + 3, IC<3 % NG>{}, IC<0>{}, IC<0>{});
    if (NG > 4 && u0 + 4 <= n_tiles) tile_body(u0 + 4, IC<4 % NG>{}, IC<0>{}, IC<0>{});
    if (NG > 5 && u0 + 5 <= n_tiles) tile_body(u0 + 5, IC<5 % NG>{}, IC<0>{}, IC<0>{});
  }
  __builtin_amdgcn_s_waitcnt(0);  // no LDS write of this workgroup may still be in flight at exit

  // ---- epilogue: normalise, then store (or merge) with fully coalesced global accesses.
  // In the accumulator layout a lane holds 4-float pieces of ONE row, 32 bytes apart from its
  // neighbour's; each wave therefore transposes its 32 x D tile through a private, chunk-
  // swizzled LDS region (the rings are dead by now) and reads it back row-major, one 16-byte
  // chunk per lane, so that every global row is touched as one contiguous segment.
  __builtin_amdgcn_s_waitcnt(0);
  if constexpr (IN_LANES) {
    wg_barrier();   // every wave is done with the K/V rings and none of its loads is still landing
    continue;
  }
  if (G == 1) __syncthreads();  // every wave is done with the K/V rings and none of its loads is still landing (G > 1: below)
  {
  // The lane is counted anew: held over the loop, it and what follows from it spill at D = 128, and a kernel with
  // scratch starts about 1 us later.
  const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), ql = lane & 31, hf = lane >> 5;
  const int qrow = qw0 + ql;
  constexpr int ROWB = 4 * D;                 // bytes of one fp32 output row
  constexpr int CPRF = D / 4;                 // 16-byte chunks per fp32 row = lanes per row when reading back
  constexpr int RPI_OUT = 64 / CPRF;          // rows one wave-wide access covers
  char* const my = lds + wave * (32 * ROWB);
  float* const my_w = reinterpret_cast<float*>(lds + L::w) + rg * 32;     // Update weight of each of the row group's rows
  int* const my_mode = reinterpret_cast<int*>(lds + L::mode) + rg * 32;   // and its case
  float l_tot = half_swap_sum(l_run), m_tot = m_ref, f_own = 1.f;
  if constexpr (G > 1) {
    // The key groups' sums meet: every wave scales its share to the common reference (they differ only where a row's
    // scores left the fast path's range) and the tiles are added as they are read back.
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    f32x2* const sums = reinterpret_cast<f32x2*>(lds + L::sums);
    if (hf == 0) sums[wave * 32 + ql] = f32x2{m_ref, l_tot};
    __syncthreads();
    f32x2 each[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
      each[g] = sums[(g * R + rg) * 32 + ql];
      m_tot = fmaxf(m_tot, each[g][0]);
    }
    l_tot = 0.f;   // (no reference: nothing was seen and the sum is 0, or NaN)
#pragma unroll
    for (int g = 0; g < G; g++) l_tot += each[g][0] == -INFINITY ? each[g][1] : each[g][1] * __builtin_amdgcn_exp2f((each[g][0] - m_tot) * c2);
    f_own = m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_ref - m_tot) * c2);
  }
  const float inv = l_tot > 0.f ? f_own / l_tot : 0.f;
  const float lse_blk = l_tot > 0.f ? m_tot * p.scale + logf(l_tot) : -INFINITY;
#pragma unroll
  for (int db = 0; db < DB; db++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int c = 8 * db + 2 * g + hf;  // 16-byte chunk of d = 32*db + 8*g + 4*hf
      f32x4 o;
#pragma unroll
      for (int r = 0; r < 4; r++) o[r] = o_acc[db][4 * g + r] * inv;
      *reinterpret_cast<f32x4*>(my + ql * ROWB + ((c ^ (ql & 15)) << 4)) = o;
    }
  if constexpr (PART) {
    part_epilogue<D, EPI, R, G>(p, lds, lane, rg, kgrp, q0, b, hq, pb.group, pb.part, n_live, lse_blk, l_tot != l_tot);
    return;
  }
  // One key group: a wave reads back what it wrote itself.  More: each stores its share of the row group's rows once all
  // tiles (and the Update plans, by the first one) are written.
  auto tiles_written = [&]() __attribute__((always_inline)) {
    if (G > 1) __syncthreads();
    else __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes are visible to all its lanes
  };
  if (EPI != kEpiMerge) tiles_written();
  if (EPI != kEpiMerge && kgrp == 0 && hf == 0 && qrow < p.Sq)
    p.lse[(int64_t)b * p.l_sb + (int64_t)hq * p.l_sh + (int64_t)qrow * p.l_ss] = lse_blk;
  const int rr = kgrp * (32 / G) + lane / CPRF, cc = lane % CPRF;
  constexpr int NIT = 32 / G / RPI_OUT;
  const int64_t o_bh = (int64_t)b * p.o_sb + (int64_t)hq * p.o_sh + chunk_row * p.o_ss + 4 * cc;
  const int64_t l_bh = (int64_t)b * p.l_sb + (int64_t)hq * p.l_sh + chunk_row * p.l_ss;
  if (EPI == kEpiMerge) {
    // Out, Lse <- Update(block_out, block_lse) on the accumulators p.out / p.lse.  All of the
    // wave's accumulator rows are fetched first (the O registers are free by now), so their
    // latencies overlap instead of each load waiting behind the previous row's store.  Rows
    // past Sq fetch the last valid row and are never stored.  The accumulator is touched once
    // per launch, so it is read and written past the caches (non-temporal).
    float* const acc_out = reinterpret_cast<float*>(p.out);
    f32x4 x[NIT];
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int grow = min(qw0 + it * RPI_OUT + rr, p.Sq - 1);
      if (CHUNKS && block == 0) x[it] = f32x4{0.f, 0.f, 0.f, 0.f};
      else x[it] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(acc_out + o_bh + (int64_t)grow * p.o_ss));
    }
    // The Update of a row is planned once, by the lanes that own the row in the accumulator layout
    // (its two exponentials and its logarithm would otherwise be evaluated in every lane that
    // blends a chunk of the row, 16 times per wave at D = 128), while the accumulator pieces are
    // on their way.  The same lane reads the row's old lse and writes the new one.
    if (kgrp == 0) {
      const int64_t l_at = l_bh + (int64_t)min(qrow, p.Sq - 1) * p.l_ss;
      UpdatePlan plq = plan_update(CHUNKS && block == 0 ? -INFINITY : p.lse[l_at], lse_blk);
      if (CHUNKS && block == 0) plq.mode = 2;   // a first block is stored as it is, also where it is NaN (with lse -inf)
      if (hf == 0) {
        my_w[ql] = plq.w;
        my_mode[ql] = plq.mode;
        if (qrow < p.Sq) p.lse[l_at] = plq.new_lse;
      }
    }
    tiles_written();
    // All LDS reads of the wave's rows go out first (block piece, weight and case of its row), then
    // the pieces are blended and stored; the row address advances by a fixed step.
    f32x4 ov[NIT];
    UpdatePlan pl[NIT];
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int r = it * RPI_OUT + rr;
      ov[it] = row_piece<D, R, G>(lds, rg, r, cc);
      if (CHUNKS && block > 0 && p.chunk_bf16) {
#pragma unroll
        for (int e = 0; e < 4; e++) ov[it][e] = (float)(__bf16)ov[it][e];
      }
      pl[it].w = my_w[r];
      pl[it].mode = my_mode[r];
      pl[it].new_lse = 0.f;
    }
    float* dst = acc_out + o_bh + (int64_t)(qw0 + rr) * p.o_ss;
    const int64_t dst_step = (int64_t)RPI_OUT * p.o_ss;
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      if (qw0 + it * RPI_OUT + rr < p.Sq) __builtin_nontemporal_store(apply_update(pl[it], x[it], ov[it]), reinterpret_cast<f32x4*>(dst));
      dst += dst_step;
    }
  } else if (EPI == kEpiF32) {
    // Results are stored past the L2 (non-temporal), here and below: dirty lines would be written back when the kernel ends, with
    // nothing beside it.  256 heads of 256 rows 22.1 -> 20.6 us, 32 of 1024 24.6 -> 23.7, causal 8192 466 -> 463; bf16 results of causal
    // steps 1 - 5 % less, 4096 rows x 32 heads and the merge that reads them next 254.3 -> 256.3.  (Partials of a cut call and their fold: no change either way.)
    f32x4 ov[NIT];
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      const int r = it * RPI_OUT + rr;
      ov[it] = row_piece<D, R, G>(lds, rg, r, cc);
    }
    float* dst = reinterpret_cast<float*>(p.out) + o_bh + (int64_t)(qw0 + rr) * p.o_ss;
    const int64_t dst_step = (int64_t)RPI_OUT * p.o_ss;
#pragma unroll
    for (int it = 0; it < NIT; it++) {
      if (qw0 + it * RPI_OUT + rr < p.Sq) __builtin_nontemporal_store(ov[it], reinterpret_cast<f32x4*>(dst));
      dst += dst_step;
    }
  } else {
    // bf16 rows are half as long: a lane converts two neighbouring chunks and stores 16 bytes
    constexpr int LPR = D / 8;          // lanes per bf16 row
    constexpr int RPI_B = 64 / LPR;     // rows one wave-wide store covers
    constexpr int NIT_B = 32 / G / RPI_B;
    const int rb = kgrp * (32 / G) + lane / LPR, cb = lane % LPR;
    const int64_t ob_bh = (int64_t)b * p.o_sb + (int64_t)hq * p.o_sh + 8 * cb;
    f32x4 o0[NIT_B], o1[NIT_B];
#pragma unroll
    for (int it = 0; it < NIT_B; it++) {
      const int r = it * RPI_B + rb;
      o0[it] = row_piece<D, R, G>(lds, rg, r, 2 * cb);
      o1[it] = row_piece<D, R, G>(lds, rg, r, 2 * cb + 1);
    }
    __bf16* dst = reinterpret_cast<__bf16*>(p.out) + ob_bh + (int64_t)(qw0 + rb) * p.o_ss;
    const int64_t dst_step = (int64_t)RPI_B * p.o_ss;
#pragma unroll
    for (int it = 0; it < NIT_B; it++) {
      bf16x8 ob;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        ob[k] = (__bf16)o0[it][k];
        ob[4 + k] = (__bf16)o1[it][k];
      }
      if (qw0 + it * RPI_B + rb < p.Sq) __builtin_nontemporal_store(ob, reinterpret_cast<bf16x8*>(dst));
      dst += dst_step;
    }
  }
  }
  if constexpr (CHUNKS) __syncthreads();  // the next block's loads land where other waves may still read their rows
  }
  if constexpr (IN_LANES) chunk_update(done, true);
}

constexpr int waves_per_simd(int D, int NS) { return D == 64 && NS == 3 ? 3 : 2; }   // at least
template <int D, int EPI, int FORM, int R, int G>
__global__ void __launch_bounds__(64 * R * G, waves_per_simd(D, ring_depth(D, R, G))) block_attn_kernel(const AttnParams p) { attend<D, EPI, FORM, R, G>(p); }
template <int D, int EPI, int FORM, int R, int G>
__global__ void __launch_bounds__(64 * R * G, waves_per_simd(D, ring_depth(D, R, G))) segments_attn_kernel(const AttnParams p) { attend<D, EPI, FORM, R, G>(p); }
template <int EPI, int FORM>
__global__ void __launch_bounds__(64 * 2 * 2, 3) trio_attn_kernel(const AttnParams p) { attend<64, EPI, FORM, 2, 2, 3>(p); }

template <int D, int EPI, int FORM, int R, int G, int NS = ring_depth(D, R, G)>
hipError_t launch_one(const AttnParams& p, dim3 grid, hipStream_t stream) {
  constexpr int lds_bytes = Lds<D, R, G, NS>::bytes(FORM);
  static_assert(lds_bytes <= 160 * 1024 / (D == 64 && NS == 3 ? 3 : 1), "LDS budget exceeded");
  void (*kernel)(const AttnParams);
  if constexpr (NS != ring_depth(D, R, G)) kernel = trio_attn_kernel<EPI, FORM>;
  else if constexpr (in_segments(FORM)) kernel = segments_attn_kernel<D, EPI, FORM, R, G>;
  else kernel = block_attn_kernel<D, EPI, FORM, R, G>;
  // Raising the dynamic-LDS limit is a per-function, per-device setting: done once for each
  // device this process launches on (the flags are atomics, a repeated set is harmless).
  constexpr int kMaxDevices = 64;
  static std::atomic<bool> attr_set[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices || !attr_set[dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices) attr_set[dev].store(true, std::memory_order_release);
  }
  return launch_kernel(kernel, grid, dim3(64 * R * G), lds_bytes, stream, p);
}

template <int D, int FORM, int R, int G>
hipError_t launch_epilogue(const AttnParams& p, int epilogue, dim3 grid, hipStream_t stream) {
  if constexpr (FORM != kChunks) {
    if (epilogue == kEpiBf16) return launch_one<D, kEpiBf16, FORM, R, G>(p, grid, stream);
    if (epilogue == kEpiF32) return launch_one<D, kEpiF32, FORM, R, G>(p, grid, stream);
  }
  return launch_one<D, kEpiMerge, FORM, R, G>(p, grid, stream);
}

}  // namespace

template <int FORM>
hipError_t launch_trio(const AttnParams& p, int epilogue, dim3 grid, hipStream_t stream) {
  if (epilogue == kEpiBf16) return launch_one<64, kEpiBf16, FORM, 2, 2, 3>(p, grid, stream);
  if (epilogue == kEpiF32) return launch_one<64, kEpiF32, FORM, 2, 2, 3>(p, grid, stream);
  return launch_one<64, kEpiMerge, FORM, 2, 2, 3>(p, grid, stream);
}

template <int D, int R, int G>
hipError_t launch_attn_shape(const AttnParams& p, int epilogue, dim3 grid, hipStream_t stream) {
  if constexpr (D == 64 && R == 2 && G == 2) {
    if (p.shape == kShapeTrio) {
      if (p.n_chunks > 0 || p.n_parts > 0) return hipErrorInvalidValue;
      return p.renew > 0 ? launch_trio<kSegments>(p, epilogue, grid, stream) : launch_trio<kPlain>(p, epilogue, grid, stream);
    }
  }
  if (p.n_chunks > 0) return launch_epilogue<D, kChunks, R, G>(p, epilogue, grid, stream);
  if (p.n_parts > 0 && p.renew > 0) {   // rings only, whose heads are packed and whose workgroups have one key group
    if constexpr (G == 1) {
      if (epilogue == kEpiF32 && p.n_parts == 1) return launch_one<D, kEpiF32, kPartSegments, R, G>(p, grid, stream);
    }
    return hipErrorInvalidValue;
  }
  if (p.n_parts > 0) return launch_epilogue<D, kPart, R, G>(p, epilogue, grid, stream);
  if (p.renew > 0) return launch_epilogue<D, kSegments, R, G>(p, epilogue, grid, stream);
  return launch_epilogue<D, kPlain, R, G>(p, epilogue, grid, stream);
}

}  // namespace tr
