// C ABI of libtokenring: argument validation, descriptor -> kernel-parameter marshalling, the choice of a launch's
// form, and the step lists of TokenRing's schedules (for tr_schedule_steps: on one GPU a schedule is one launch).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "tr_internal.h"

namespace {

thread_local char g_err[512] = "";
thread_local tr::TimingEvents g_timing = {nullptr, nullptr};

tr_status fail(tr_status st, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return st;
}

int64_t elem_bytes(int32_t dtype) { return dtype == TR_BF16 ? 2 : 4; }

// Number of elements from ptr to one past the last addressed element of the view.
int64_t extent_elems(const tr_tensor* t) {
  if (t->B == 0 || t->H == 0 || t->S == 0 || t->D == 0) return 0;
  return (t->B - 1) * t->stride_b + (t->H - 1) * t->stride_h + (t->S - 1) * t->stride_s + t->D;
}

bool overlaps(const tr_tensor* a, const tr_tensor* b) {
  const int64_t ea = extent_elems(a) * elem_bytes(a->dtype), eb = extent_elems(b) * elem_bytes(b->dtype);
  if (ea == 0 || eb == 0) return false;
  const uintptr_t a0 = (uintptr_t)a->ptr, b0 = (uintptr_t)b->ptr;
  return a0 < b0 + (uintptr_t)eb && b0 < a0 + (uintptr_t)ea;
}

// Common checks of one descriptor. `row_align` = required multiple (in elements) of the strides
// and byte alignment of the pointer for vector access.
tr_status check_tensor(const char* name, const tr_tensor* t, bool allow_bf16, bool allow_f32, int row_align_bytes) {
  if (!t) return fail(TR_ERR_NULL, "%s: descriptor is NULL", name);
  if (t->dtype != TR_BF16 && t->dtype != TR_F32) return fail(TR_ERR_DTYPE, "%s: unknown dtype %d", name, (int)t->dtype);
  if ((t->dtype == TR_BF16 && !allow_bf16) || (t->dtype == TR_F32 && !allow_f32))
    return fail(TR_ERR_DTYPE, "%s: dtype %s not supported for this argument", name, t->dtype == TR_BF16 ? "bf16" : "fp32");
  if (t->B < 0 || t->H < 0 || t->S < 0 || t->D < 0) return fail(TR_ERR_SHAPE, "%s: negative dimension", name);
  if (t->B > INT32_MAX || t->H > INT32_MAX || t->S > (1 << 30) || t->D > INT32_MAX)
    return fail(TR_ERR_SHAPE, "%s: dimension too large", name);
  const bool empty = extent_elems(t) == 0;
  if (!empty && !t->ptr) return fail(TR_ERR_NULL, "%s: data pointer is NULL", name);
  if (t->stride_b < 0 || t->stride_h < 0 || t->stride_s < 0) return fail(TR_ERR_STRIDE, "%s: negative stride", name);
  if (!empty) {
    if (t->S > 1 && t->stride_s < t->D) return fail(TR_ERR_STRIDE, "%s: stride_s %lld smaller than D %lld", name, (long long)t->stride_s, (long long)t->D);
    const int64_t eb = elem_bytes(t->dtype);
    if (row_align_bytes > 1) {
      if (((uintptr_t)t->ptr) % row_align_bytes) return fail(TR_ERR_STRIDE, "%s: pointer not %d-byte aligned", name, row_align_bytes);
      if ((t->stride_b * eb) % row_align_bytes || (t->stride_h * eb) % row_align_bytes || (t->stride_s * eb) % row_align_bytes)
        return fail(TR_ERR_STRIDE, "%s: strides must be multiples of %d bytes", name, row_align_bytes);
    }
  }
  return TR_OK;
}

// A tensor the kernels write must not address one element through two index tuples (a zero or
// too small stride on a dimension larger than 1): rows are updated by different waves, so an
// overlapping view would race.  Sufficient test: ordered by stride, every dimension must step
// over the whole extent of the dimensions inside it.
tr_status check_written(const char* name, const tr_tensor* t) {
  if (extent_elems(t) == 0) return TR_OK;
  int64_t size[3] = {t->B, t->H, t->S}, stride[3] = {t->stride_b, t->stride_h, t->stride_s};
  for (int i = 0; i < 3; i++)
    for (int j = i + 1; j < 3; j++)
      if (stride[j] < stride[i]) {
        const int64_t a = size[i], b = stride[i];
        size[i] = size[j]; stride[i] = stride[j];
        size[j] = a; stride[j] = b;
      }
  int64_t inner = t->D;
  for (int i = 0; i < 3; i++) {
    if (size[i] <= 1) continue;
    if (stride[i] < inner) return fail(TR_ERR_STRIDE, "%s: a written tensor must not overlap itself (stride %lld < %lld elements inside it)", name, (long long)stride[i], (long long)inner);
    inner = stride[i] * (size[i] - 1) + inner;
  }
  return TR_OK;
}

// One block step of a schedule: Query segment qs attends K/V segment ks (equal segments of S),
// or, with ks2 >= 0, the pair of K/V segments ks and ks2 as one key range.
struct RingStep {
  int qs, ks;
  int ks2 = -1;
};

// View of `rows` rows of a tensor along S, from row r0 on.
tr_tensor rows_view(const tr_tensor* t, int64_t r0, int64_t rows) {
  tr_tensor r = *t;
  r.ptr = (char*)t->ptr + r0 * t->stride_s * elem_bytes(t->dtype);
  r.S = rows;
  return r;
}

// ---- partitioned attention launches: which calls, how many parts, and where the partial results go.

constexpr int kCUs = 256;
constexpr int kMaxRows = 256;   // Query rows of the largest workgroup
constexpr int kPartStreams = 4;
constexpr int64_t kPartBytes = (int64_t)33 << 20;   // 256 workgroups' partials of 256 rows at D = 128
constexpr int64_t kPartAlign = 128;   // parts begin on whole tiles of either head dim

struct PartPlan {
  int pack = 0, parts = 1, members = 0, row_tiles = 0, part_rows = 0;
  int64_t part_keys = 0, out_elems = 0;   // out_elems: floats of block_out in the scratch
  bool packs_uncut = false;               // heads are packed also where the keys are not cut
  int renew = 0;                          // of an uncut call: keys after which a row's exponent reference is taken anew
};

// Workgroups of a cut launch under the causal rule: those of the fullest XCD, for all eight.  A row tile has one for each part that some
// row of it sees, one at least; the kernel deals the tiles of all parts out in eight contiguous pieces (decode_part), and
// pieces of the first parts hold the most: 255 workgroups of 3 heads of 3929 rows in 5 parts are 58 on one XCD of 32 compute units.
int64_t causal_workgroups(const tr::AttnParams& p, int64_t heads, int64_t rows, int bm) {
  const int64_t tiles = (rows + bm - 1) / bm, gq = p.gq, per_xcd = (heads * p.n_parts * tiles + 7) / 8;
  int64_t live[tr::kMaxParts], least = tiles;   // row tiles of a head that have a part
  for (int i = 0; i < p.n_parts; i++) {
    // (tile t sees keys of part i from row i * part_keys - causal_off on)
    const int64_t first = std::max<int64_t>(0, (int64_t)i * p.part_keys - p.causal_off);
    live[i] = i == 0 ? tiles : std::max<int64_t>(0, tiles - first / bm) * (first < rows && (int64_t)i * p.part_keys < p.Sk);
    least = std::min(least, live[i]);
  }
  if (least == tiles) return heads * p.n_parts * tiles;
  int64_t on[8] = {};
  for (int64_t unit = 0, at = 0; unit < heads / gq * p.n_parts; unit++)
    for (int64_t h = 0; h < gq; h++, at += tiles)   // its live tiles lie in front
      for (int64_t a = at, end = at + live[unit % p.n_parts]; a < end;) {
        const int64_t x = a / per_xcd, stop = std::min(end, (x + 1) * per_xcd);
        on[x] += stop - a;
        a = stop;
      }
  return 8 * *std::max_element(on, on + 8);
}

// Shape of a launch's workgroups.  8 x 1 (256 rows) has the least traffic for its products and is the best use of a full chip
// over long key ranges.  4 x 1, several to a compute unit, hides set-up and epilogue and ends more evenly.  A launch that would leave
// compute units idle runs 4 x 2 or 2 x 2, whose waves also share the keys out among themselves.
// Chosen by an estimate of the launch's time (us) from measured costs: set-up and epilogue of a workgroup, and a tile of keys
// (64 at D 128, 128 at D 64) on an idle and on a full chip, on a compute unit with one, two, three workgroups, and with at most half of
// the waves at work.  Both sides of the lines, us for 8 x 1 / 4 x 1 / 4 x 2 / 2 x 2 at D 128: 8 heads of 256 rows 12.5 / - / 10.9 / 8.6; 16 of
// 1024 27.7 / 21.6 / 21.8 / 18.1; 32 of 1024 29.2 / 24.5 / 25.2 / 30.4; 64 of 1024 39.1 / 39.2 / 48.7 / 58.7, under the causal rule 30.8 / 28.0 / 34.7 / 43.9;
// 8 of 4096 84 / 71 / 69 / 85; 24 of 1777 51.2 / 51.5 / 59.7 / 64.9, under the causal rule 42.4 / 35.5 / 33.2 / 40.9; 16 of 8192 438 / 460.
// bf16 blocks: 50 calls of 2 to 48 heads in every shape, the one chosen 1.1 % above the fastest on average, six by 4 - 7 %.
// p holds the launch's parts and chunks; pack: the rows are those of a K/V head's whole group; out_bytes: of an output element; estimate: of the time, if asked for.
int choose_shape(const tr::AttnParams& p, int D, bool pack, int out_bytes, double* estimate = nullptr) {
  const int refs = p.renew > 0 ? (p.Sk - 1) / p.renew : 0;
  const int64_t rows = pack ? (int64_t)p.gq * p.Sq : p.Sq, heads = (int64_t)p.B * (pack ? p.Hkv : p.Hq);
  if (p.Sk == 0) return tr::kShape8x1;
  struct Cost { double fix, idle, busy, two, three, fix_few, few, block; };   // block: of a later block of the chunk form, in units of fix
  static const Cost costs[2][5] = {{{7.5, 1.52, 2.03, 0, 0, 5.2, 1.0, 1.7}, {6.5, 1.0, 1.12, 2.03, 2.96, 5.6, 0.95, 1.3},
                                    {7.1, 0.83, 1.09, 0, 0, 6.0, 0.65, 0.75}, {5.8, 0.61, 0.72, 0, 0, 5.4, 0.6, 0.75},
                                    {6.0, 0.62, 0.75, 1.15, 1.72, 5.6, 0.62, 0.75}},
                                   {{8.3, 1.1, 1.67, 0, 0, 6.2, 0.7, 1.7}, {8.5, 0.7, 0.95, 1.78, 0, 6.8, 0.65, 1.3},
                                    {9.0, 0.59, 0.93, 0, 0, 7.5, 0.5, 0.75}, {7.0, 0.47, 0.57, 0, 0, 6.5, 0.45, 0.75}}};
  const double tile_keys = D == 64 ? 128.0 : 64.0;
  const int64_t part = p.n_parts > 1 ? p.part_keys : p.Sk;
  const double later = p.n_chunks > 1 ? p.n_chunks - 1 : 0;   // blocks behind its first of the longest workgroup
  const double blocks = p.causal ? later / 2 : later, chunks = later + 1;   // later blocks of the average workgroup
  const double memory = (double)(heads * rows) * chunks * D * (2 + (p.n_parts > 1 ? 4 : out_bytes)) / 5.2e6;   // Query rows in, result out
  const bool trio = D == 64 && p.n_parts == 0 && p.n_chunks == 0;   // the forms that it has
  int best = tr::kShape8x1;
  double t_best = 0, seen_share = 0;   // seen_share: of the keys that the last row tile sees, by the average one (of the shape chosen)
  for (int shape = 0; shape < (trio ? 5 : 4); shape++) {
    const Cost& c = costs[D == 128][shape];
    const int bm = tr::shape_rows(shape), per_cu = tr::shape_per_unit(shape, D);
    const bool groups = shape >= tr::kShape4x2;
    const int64_t tiles = (rows + bm - 1) / bm;
    if (shape != tr::kShape8x1 && tiles > 65535) continue;   // a grid's second dimension
    if (groups && (refs > (shape == tr::kShapeTrio ? tr::kMaxRefsTrio : tr::kMaxRefs) || heads * tiles >= 8 * kCUs)) continue;
    // Trio: where all its workgroups run at once and a compute unit holds two or three, that is one to one and a half of 128 rows, which leave units
    // uneven.  us under the causal rule, the best of the other shapes / trio: 24 heads of 1777 rows 18.9 / 17.3, 32 of 1024 13.3 / 11.3, 8 of 4096 33.1 / 28.7, 4 of 9000 68.6 / 58.5,
    // 2 of 20000 152 / 136; rings of 16 of 2048 in 4 segments 22.4 / 18.3, 4 of 8192 in 2 52.4 / 49.1, 2 of 17644 in 4 119 / 108; beyond it 64 of 1024 15.7 / 17.4, 12 of 4096 36.3 / 36.7.
    // Not for a few keys, where set-up is the time, of two on a unit and more so of three: bf16 results of 256 heads of 88 rows 5.3 / 6.0, of 128 5.9 / 6.2, of 118 on 174 keys
    // 7.3 / 7.0; 128 heads of 280, whose units hold up to three, 7.3 / 7.9, of 336 8.2 / 8.7, fp32 results of 96 of 354 8.5 / 8.3.  (With more heads than units it stays: the other
    // shapes' estimates are furthest off there, 384 heads of 83 rows 9.4 in the one they choose, 7.4.)
    if (shape == tr::kShapeTrio) {
      const int64_t n = heads * tiles, seen = std::min<int64_t>(p.Sk, rows + p.causal_off);   // keys that the last row sees under the causal rule
      const bool few_keys = p.causal && p.causal_off >= 0 && heads <= kCUs && seen < (n > 2 * kCUs ? 352 : 160);
      if (n < 2 * kCUs || n > 3 * kCUs || few_keys) continue;
    }
    if (groups && p.renew > 0 && (p.renew < 64 || pack)) continue;   // renewals lie as far apart as a group's sub-tiles; packed rings fill the chip and never gain from key groups
    int64_t least = p.Sk, most = p.Sk, sum = p.Sk * tiles;   // keys that the first, the last, all row tiles of a head see
    if (p.causal && pack) {
      least = most = std::max<int64_t>(0, std::min<int64_t>(p.Sk, (int64_t)p.Sq + p.causal_off));
      sum = most * tiles;
    } else if (p.causal) {   // tile t sees the keys below (t + 1) * rows + causal_off
      most = std::max<int64_t>(0, std::min<int64_t>(p.Sk, rows + p.causal_off));
      least = std::max<int64_t>(0, std::min<int64_t>(most, bm + (int64_t)p.causal_off));
      const int64_t off = p.causal_off, all = std::min(tiles, std::max<int64_t>(0, (p.Sk - off + bm - 1) / bm - 1));
      const int64_t none = std::min(all, off < 0 ? -off / bm : 0);   // tiles [none, all) see some, [all, tiles) every key
      sum = (all * (all + 1) - none * (none + 1)) / 2 * bm + (all - none) * off + (tiles - all) * p.Sk;
    }
    double n = (double)(heads * tiles) * chunks, total = ((double)(heads * sum) + (double)(heads * tiles) * blocks * p.Sk) * chunks / tile_keys;
    if (p.n_parts > 1) n = p.causal && !pack ? (double)causal_workgroups(p, heads, rows, bm) : n * std::max(1.0, std::ceil((double)most / (double)part));
    const double longest = ((double)std::min(most, part) + later * p.Sk) / tile_keys;
    const double shortest = p.n_parts > 1 ? 0.0 : (double)least / tile_keys;
    const bool few = std::min<int64_t>(rows, bm) <= bm / 2;
    const double fill = std::min(1.0, n / kCUs * std::min(1.0, total / (n * longest + 1e-9)));   // less than n / kCUs where some workgroups end early
    const double alone = few ? c.few : c.idle + (c.busy - c.idle) * fill * fill;   // (a chip that is not full runs at a higher clock)
    // (What a later segment costs key groups more than one; us a segment, 4 x 1 and 2 x 2: 8 heads of 1024 in 8 at D 128 0.53 and 0.84, at D 64 0.50 and 0.62.)
    const double ref = shape == tr::kShape4x2 ? 0.7 + 0.6 * fill : (D == 64 ? 0.3 : 0.5) + 0.3 * fill;
    // (An odd number of sub-tiles is a step more for one of the key groups, which counts where there are few.  us, 4 x 1 and 2 x 2: rings without a mask of 288 keys in 4 at D 128 10.6
    // and 11.3, of 292 11.7 and 11.5, of 412 12.6 and 13.1, of 464 13.9 and 13.7, at D 64 of 156 in 2 6.3 and 6.9, of 280 in 4 8.4 and 8.8, of 324 9.4 and 9.4, of 408 10.0 and 9.6.)
    const bool odd = refs > 0 && !p.causal && p.Sk <= (D == 64 ? 288 : 416) && (p.Sk + 31) / 32 % 2 == 1;
    const double fix = (few ? c.fix_few : c.fix) + (groups ? ref * refs + (odd ? (D == 64 ? 0.6 : 0.8) : 0.0) : 0.0);
    const double rounds = std::ceil(n / kCUs);
    double time;
    if (per_cu > 1 && n > kCUs) {   // workgroups of one compute unit fill each other's gaps
      const double at_once = std::min<double>(per_cu, rounds), tile = at_once == 3 ? c.three : c.two;
      time = total * tile / (kCUs * at_once);
      if (!p.causal && rounds <= per_cu) time = longest * tile * (0.85 + 0.15 * n / (kCUs * rounds));   // all at once: as slow as the fullest compute unit
      // (Trio: half the rows, it ends more evenly: 313 causal calls in its window are 0.8 % above their fastest shape on average, with 0.15 2.9 %.)
      if (p.causal || later > 0) time += (shape == tr::kShapeTrio ? 0.05 : 0.15) * longest * tile;
      if (shape == tr::kShapeTrio) {
        // Where row tiles see about as many keys, a unit that holds three sets the time, however few others do.
        if (p.causal) time = std::max(time, 0.81 * (0.45 * longest + 0.55 * shortest) * tile);
        // Under the causal rule, whose order spreads a head's row tiles over the launch, they fetch K and V again and again once these are more than the L2s hold (32 MB),
        // at about 11 TB/s, the first time at 6.5; from the fifth tile on little is added, while the memory-side cache (256 MB) holds them.  us, the best of the other shapes / trio: chunks behind cached keys of 256
        // heads of 138 rows on 5315 keys (348 MB of K and V) 82 / 141, 192 of 256 on 2568 (126) 45 / 59, 128 of 110 on 1873 (122) 25 / 37, 256 of 99 on 2066 (68) 25 / 29, 48 of
        // 1005 on 6111 (75) 90 / 84, 128 of 251 on 743 (24) 12.0 / 11.2.  (737 such calls are 1.4 % above the fastest on average, without it 3 %, by up to three quarters.)
        const double once = (double)p.B * p.Hkv * most * D * 4, all = total * tile_keys * D * 4;
        if (p.causal && once > 60e6 && all > 1.2 * once) time = std::max(time, once / 6.5e6 + (once > 256e6 ? all - once : std::min(all - once, 3 * once)) / 11e6);
      }
      time = std::max(time, memory) + fix + 0.35 * blocks * fix * n / (kCUs * at_once);
      time = std::max(time, longest * alone + fix * (1 + c.block * later));
    } else {
      const double each = fix * (1 + c.block * later), average = fix * (1 + c.block * blocks);
      time = longest * alone + std::max(each, std::min(memory, 2 * each));
      if (n > kCUs && !p.causal) time = rounds * longest * alone + std::max(rounds * each, memory + 3 * rounds);
      if (n > kCUs && p.causal)   // every round has its shortest workgroup's time, what is left evens out
        time = std::max(time, (rounds * shortest + (total - n * shortest) / kCUs + 0.15 * (longest - shortest)) * alone + std::max(n * average / kCUs, memory));
    }
    // (The causal parts of a launch are not dealt out longest first, so that a second round costs more than its share:
    // 12 heads of 2306 rows on 2665 keys in 2 parts 43 us with 256 rows, 49 with 128.)
    if (shape != tr::kShape8x1 && p.n_parts > 1 && p.causal && n > kCUs * per_cu) continue;
    if (shape == tr::kShape8x1) {
      t_best = time * (n > kCUs ? 0.95 : 0.97);   // a last round that is nearly empty runs faster than a full one
    } else {   // over several rounds the estimates lie closer together than their errors, unless there are many
      // (Trio without a mask: 0.93 to 1.16 of the best other shape on 83 calls in its window, which the estimates don't tell apart: with 1.0 25 of them gain
      // 2 % and more and 10 lose as much, up to 10 %.  24 heads of 1777 rows 29.6 / 28.7, 128 of 300 on 300 keys 10.0 / 10.1, on 3000 45.9 / 43.1, where it is taken.)
      time *= shape == tr::kShapeTrio ? (p.causal ? 1.0 : 1.13) : n > 8 * kCUs ? 0.97 : n > kCUs * per_cu ? 1.03 : 1.0;
      if (time < t_best) {
        t_best = time;
        best = shape;
        seen_share = total / (n * longest + 1e-9);
      }
    }
  }
  // (Against a cut, whose workgroups are many and short, units that hold three of trio's count more: 16 heads of 2462 rows behind 25314 keys 323 / in three parts 287.)
  if (estimate) *estimate = t_best * (best == tr::kShapeTrio && p.causal ? 1.0 + 0.1 * std::max(0.0, seen_share - 0.6) : 1.0);
  return best;
}

// Chooses the form of a launch; false: the plain one.  may_cut false: the keys stay in one piece, which makes the
// result independent of the stream and of capture, whatever scratch is there.
//
// Heads are packed when that leaves at most four fifths of the row tiles: the rows that fill a tile up cost
// their share of the loads and of the time of its slowest wave all the same.  Without a cut they are packed only
// where that takes fewer rounds of workgroups (one row x 32 heads on 8 K/V heads of 4096 keys, 32 sequences: 184 us
// plain, 95 packed); as many rounds, or one, are better filled by the plain form (75 rows x 32 heads on 75 keys 17.6
// plain, 18.2 packed; 538 rows x 128 heads on 16 K/V heads of 1070 keys at D 64 43.4 and 45.0).
//
// The keys are cut where an estimate of the call's time (us) says so, over rounds of one workgroup per compute
// unit.  Measured: a tile of keys takes 0.7 (D 64, twice the keys: 1.0) while at most four waves of a workgroup
// have rows, else 1.1 (1.6) on an idle chip and 1.75 (2.15) on a full one, where the clock gives way; a workgroup's
// set-up and epilogue 8; the fold 5, 0.25 for each part of a row, and its partials at 3.5 TB/s; nothing is faster than
// K and V at 5 TB/s.
// Both sides of the line, us: 500 rows x 32 heads on 12500 keys 217 in one part, 100 in 4; 96 rows x 8
// heads on 2048 keys 27.7 and 17.4 in 4; 8 rows x 16 heads on 700 keys 13.8 and 15.2 in 2; 100 rows x 256 heads on
// 128 K/V heads of 2048 keys 40 uncut and 48 in 2; 1777 rows x 24 heads on as many 35 and 47 in 2; 4 sequences, 32 heads on 8 K/V heads of 8192 keys 85 and 30 in 4.
bool plan_parts(const tr::AttnParams& p, int D, bool may_cut, PartPlan& best) {
  const int bm = kMaxRows;
  const int64_t rows = (int64_t)p.gq * p.Sq, kv = (int64_t)p.B * p.Hkv;
  if (p.Sk == 0 || p.Sq == 0 || kv == 0 || rows > ((int64_t)1 << 24)) return false;
  const int64_t packed = (rows + bm - 1) / bm, plain = (int64_t)p.gq * p.n_qtiles;
  PartPlan c;
  c.pack = 5 * packed <= 4 * plain;
  c.row_tiles = c.pack ? (int)packed : p.n_qtiles;
  c.members = (int)(c.pack ? packed : plain);
  const int64_t space = c.pack ? rows : p.Sq, tiles = kv * c.members;
  c.part_rows = space > bm ? bm : (int)((space + 31) / 32 * 32);
  auto rounds = [](int64_t workgroups) { return (workgroups + kCUs - 1) / kCUs; };
  c.packs_uncut = c.pack && (tiles > 2 * kCUs || rounds(tiles) < rounds(kv * plain));
  best = c;
  if (tiles >= ((int64_t)1 << 23) - 8) return false;   // a one-dimensional grid holds less than 2^32 threads, 512 a tile
  if (tiles > 2 * kCUs || !may_cut) return c.packs_uncut;
  // keys that some row of row tile t sees
  auto seen = [&](int t) -> int64_t {
    if (!p.causal) return p.Sk;
    const int64_t last = c.pack ? p.Sq - 1 : std::min<int64_t>((int64_t)(t + 1) * bm, p.Sq) - 1;
    return std::max<int64_t>(0, std::min<int64_t>(p.Sk, last + p.causal_off + 1));
  };
  const double tile_keys = D == 64 ? 128.0 : 64.0, heads = (double)tiles / c.row_tiles;
  const int64_t all = seen(c.row_tiles - 1);
  const double stream = (double)kv * all * D * 4 / 5e6, fix = 8.0;
  const double few = D == 64 ? 1.0 : 0.7, idle = D == 64 ? 1.6 : 1.1, busy = D == 64 ? 0.55 : 0.65;
  auto estimate = [&](int64_t part_keys) {
    double n = 0, keys = 0;
    for (int t = 0; t < c.row_tiles; t++) {
      n += heads * (double)std::max<int64_t>(1, (seen(t) + part_keys - 1) / part_keys);
      keys += heads * (double)seen(t);
    }
    const double tile = c.part_rows <= 128 ? few : idle + busy * std::min(1.0, n / kCUs);
    const double longest = (double)std::min(all, part_keys) / tile_keys * tile + fix;
    double t = longest;
    if (n > kCUs) t = p.causal ? (keys / tile_keys * tile + n * fix) / kCUs + 0.5 * longest : (double)(((int64_t)n + kCUs - 1) / kCUs) * longest;
    return std::max(t, stream + fix);
  };
  double uncut = estimate(std::max<int64_t>(all, 1));
  if (c.pack && !c.packs_uncut) {   // a call that is not cut runs the plain form then
    const double tile = p.Sq <= 128 ? few : idle + busy * std::min(1.0, (double)(kv * plain) / kCUs);
    uncut = std::max((double)rounds(kv * plain) * ((double)all / tile_keys * tile + fix), stream + fix);
  }
  double t_best = 0.95 * uncut;
  for (int n = 2; n <= tr::kMaxParts; n++) {
    const int64_t part_keys = std::max<int64_t>(512, ((all + n - 1) / n + kPartAlign - 1) / kPartAlign * kPartAlign);
    const int64_t parts = (all + part_keys - 1) / part_keys, slot_rows = tiles * parts * c.part_rows;
    if (parts != n || slot_rows * (D + 1) * 4 > kPartBytes) continue;
    const double t = estimate(part_keys) + 5.0 + 0.25 * (double)parts + (double)slot_rows * D * 4 / 3.5e6;
    if (t >= t_best) continue;
    t_best = t;
    best.parts = (int)parts;
    best.part_keys = part_keys;
    best.out_elems = slot_rows * D;
  }
  // Workgroups of fewer rows take some of the calls back that 256-row ones would have to cut.  (Not
  // where heads are packed: uncut they would not be, and every key would be read once for each of them.)
  // The reference is renewed where the parts would have begun: the weights are those of the cut call.  (With one reference for all
  // keys, 66 such calls were 0.2 - 2 % further from 64 bits, and took 10 % less time.)  us cut and uncut, in shapes of fewer rows both:
  // 8 heads of 2041 under the causal rule 32.2 and 25.4; 16 of 446 rows on 1657 keys 23.1 and 22.0; 12 of 968 on 1316 33.1 and 18.6;
  // 8 of 860 on 2645 26.5 and 30.7; 32 of 290 on 6291 at D 64 33.3 and 39.8.
  if (best.parts > 1 && !c.pack) {
    double whole = 0, cut = 0;
    tr::AttnParams w = p;
    w.renew = (int)best.part_keys;
    choose_shape(w, D, false, 4, &whole);
    tr::AttnParams q = p;
    q.n_parts = best.parts;
    q.part_keys = (int)best.part_keys;
    choose_shape(q, D, false, 4, &cut);
    cut += 5.0 + 0.25 * best.parts + (double)best.out_elems * 4 / 3.5e6;
    // The line with the least regret of those tried, on 1970 calls near it: 0.6 % (D 64) and 0.4 % (D 128) above the faster side on average, 15 and 9 of them by more than a tenth;
    // the estimates as they are 1.9 % and one in fifteen.  (What it adds is the renewals of short calls: 3 heads of 1251 rows at D 64 12.4 cut and 14.3, 2 of 1053 at D 128 15.0 and 17.0;
    // with 3.0 0.9 % and 31.  With 0.85 and 4.0 at D 128 0.55 % and 15, long calls above all: 2 x 32 heads of 165 rows behind 8701 keys 73 and 90, 2 x 32 of 147 on 7438 62 and 81, 16 of 889 on
    // 8060 67 and 80.)
    whole = std::max(whole, stream + fix);
    if (std::max((D == 64 ? 0.85 * whole + 4.0 : 0.92 * whole + 2.5) + 0.6 * (best.parts - 1), 0.95 * whole) < cut) {
      best = c;
      best.renew = w.renew;
      return false;
    }
  }
  return best.parts > 1 || best.packs_uncut;
}

// Scratch of the partitioned launches: device arrays of the library itself (nothing is allocated on the device), a pool
// of kPartStreams regions per device.  Work on one stream runs in order, so a region is in use by one launch at a time if
// every launch that takes it over waits for the one before: an event behind each use says when that one is done.  The
// stream that used a region last waits for the event on the GPU (nothing to wait for while it lives, and in order
// also where its handle has come back as another stream's); any other stream takes the region that has been idle
// longest.  (The event rides on the fold's dispatch: recorded behind it, it costs 2.7 us a call.)  No region: while all
// are busy, for the per-thread default stream, whose handle stands for several, for a stream of another device than the
// current one, and under capture, because a graph may be replayed on any stream.
__device__ __align__(256) static unsigned char part_scratch[kPartStreams][kPartBytes];
struct PartRegion {
  char* bytes = nullptr;
  hipStream_t owner = nullptr;
  hipEvent_t done = nullptr;   // behind the last use
  uint64_t used = 0;
};
struct PartPool {
  std::mutex lock;             // held from the choice of a region until the launches that use it and its event are enqueued
  PartRegion regions[kPartStreams];
  int n = 0;                   // regions that have been used
  uint64_t uses = 0;
};

// The pool that serves launches on the stream, or NULL.
PartPool* part_pool_for(hipStream_t stream) {
  constexpr int kDevices = 64;
  static PartPool pools[kDevices];
  if (stream == hipStreamPerThread || stream == (hipStream_t)1) return nullptr;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (capture != hipStreamCaptureStatusNone) return nullptr;
  int dev = -1, stream_dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return nullptr;
  if (stream != nullptr && (hipStreamGetDevice(stream, &stream_dev) != hipSuccess || stream_dev != dev)) {
    (void)hipGetLastError();
    return nullptr;
  }
  return &pools[dev];
}

// A region for the stream, or NULL.  Called with the pool's lock held and its device current.
PartRegion* take_region(PartPool& pool, hipStream_t stream) {
  // A query may disturb another stream's capture in global mode; this one is harmless to it.
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  PartRegion* r = nullptr;
  for (int i = 0; i < pool.n; i++)
    if (pool.regions[i].owner == stream) r = &pool.regions[i];
  if (r) {
    if (hipStreamWaitEvent(stream, r->done, 0) != hipSuccess) r = nullptr;
  } else if (pool.n < kPartStreams) {
    PartRegion& fresh = pool.regions[pool.n];
    void* bytes = nullptr;
    if (hipGetSymbolAddress(&bytes, HIP_SYMBOL(part_scratch)) == hipSuccess &&
        hipEventCreateWithFlags(&fresh.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess) {
      fresh.bytes = (char*)bytes + (size_t)pool.n * kPartBytes;
      r = &fresh;
      pool.n++;
    }
  } else {
    for (PartRegion& c : pool.regions)
      if ((!r || c.used < r->used) && hipEventQuery(c.done) == hipSuccess) r = &c;
  }
  (void)hipGetLastError();   // "not ready" and the like are no errors of this call
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (r) {
    r->owner = stream;
    r->used = ++pool.uses;
  }
  return r;
}

// The shape of a launch over (head, query tile) pairs; how its workgroups are placed on the XCDs.
void use_shape(tr::AttnParams& p, int shape) {
  const int bm = tr::shape_rows(shape);
  p.shape = shape;
  p.bm = bm;
  p.n_qtiles = (p.Sq + bm - 1) / bm;
  p.xcd_map = (p.B * p.Hkv) % 8 == 0 && (int64_t)p.n_qtiles * p.B * p.Hq >= 8;
  // Without the causal rule all query tiles cost the same, and an XCD may finish the
  // query tiles of one head before it starts the next: half as many heads' K/V are then live in
  // its L2 at a time.  (Under a causal mask that order would bunch the heavy tiles.)
  if (p.xcd_map && !p.causal && p.n_chunks == 0 && (int64_t)p.B * p.Hq / 8 <= 65535) p.xcd_map = 2;
}

// The shape of a launch over the row tiles of K/V heads (of each query head, or with plan.pack of a K/V head's whole group).
void use_packed_shape(tr::AttnParams& p, const PartPlan& plan, int shape) {
  const int bm = tr::shape_rows(shape), space = plan.pack ? p.gq * p.Sq : p.Sq;
  p.shape = shape;
  p.bm = bm;
  p.pack = plan.pack;
  p.n_qtiles = (space + bm - 1) / bm;
  p.members = plan.pack ? p.n_qtiles : p.gq * p.n_qtiles;
  p.part_rows = space > bm ? bm : (space + 31) / 32 * 32;
}
int64_t scratch_rows(const tr::AttnParams& p) { return (int64_t)p.B * p.Hkv * p.members * p.n_parts * p.part_rows; }

// Settles form and shape of a call that plan_parts has looked at (planned: its answer); scratch: a region is there.
void settle_launch(tr::AttnParams& p, const PartPlan& plan, bool planned, int D, int epilogue, bool scratch) {
  const int out_bytes = epilogue == 0 ? 2 : epilogue == 1 ? 4 : 8;
  if (planned && plan.parts > 1 && scratch) {
    p.n_parts = plan.parts;
    p.part_keys = (int)plan.part_keys;
    use_packed_shape(p, plan, choose_shape(p, D, plan.pack, 4));
    if (scratch_rows(p) * (D + 1) * 4 > kPartBytes) use_packed_shape(p, plan, tr::kShape8x1);   // the form the plan has counted for
    p.units = p.B * p.Hkv * p.n_parts;
  } else if (planned && plan.packs_uncut) {
    // (Without scratch, all keys at once, here and below.  The parts one after the other, folded in the output, give the bits of the cut
    // form but pay a set-up and an epilogue for each: 1764 rows x 2 heads on 6491 keys 202 us replayed from a graph
    // against 91 in one pass, a decode step of 4 sequences on 8192 keys 121 against 90.)
    p.n_parts = 1;
    p.part_keys = (p.Sk + kPartAlign - 1) / kPartAlign * kPartAlign;
    use_packed_shape(p, plan, choose_shape(p, D, plan.pack, out_bytes));
    p.units = p.B * p.Hkv;
  } else {
    if (plan.renew > 0) {
      p.renew = plan.renew;
      p.renew_log2 = 29;   // at the parts' first keys, never later
    }
    use_shape(p, choose_shape(p, D, false, out_bytes));
  }
}

hipError_t launch_planned(tr::AttnParams& p, const PartPlan& plan, bool planned, int D, int epilogue, hipStream_t stream) {
  if (PartPool* pool = planned && plan.parts > 1 ? part_pool_for(stream) : nullptr) {
    std::lock_guard<std::mutex> hold(pool->lock);   // another thread on this stream must not enqueue between attention and fold
    if (PartRegion* r = take_region(*pool, stream)) {
      settle_launch(p, plan, planned, D, epilogue, true);
      p.part_out = (float*)r->bytes;
      p.part_lse = p.part_out + scratch_rows(p) * D;
      const hipError_t e = tr::launch_block_attn(p, D, epilogue, stream, r->done);
      if (e != hipSuccess) (void)hipEventRecord(r->done, stream);   // the fold did not go out, the attention may have
      return e;
    }
  }
  settle_launch(p, plan, planned, D, epilogue, false);
  return tr::launch_block_attn(p, D, epilogue, stream);
}

// The part of a launch's parameters that plan_parts looks at.
void set_shape(tr::AttnParams& p, const tr_tensor* q, const tr_tensor* k, int causal, int64_t off64) {
  p.B = (int)q->B; p.Hq = (int)q->H; p.Hkv = (int)k->H; p.Sq = (int)q->S; p.Sk = (int)k->S;
  p.causal = causal ? 1 : 0;
  const int64_t lim = (int64_t)1 << 30;
  p.causal_off = (int)(off64 > lim ? lim : (off64 < -lim ? -lim : off64));
  p.shape = tr::kShape8x1;
  p.bm = kMaxRows;
  p.n_qtiles = (p.Sq + p.bm - 1) / p.bm;
  p.gq = p.Hkv > 0 ? p.Hq / p.Hkv : 1;
}

// fuse_update: out/lse are fp32 accumulators and the block is merged into them by the kernel's epilogue.
// n_chunks > 0: all Query chunks against all K/V chunks block by block, rounded to bf16 if chunk_bf16; the tensors are
// views of chunk 0.  renew: keys after which a row's exponent reference is taken anew (0: never).  may_cut: the keys may
// be cut into parts.
tr_status attn_common(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int causal, int64_t off64, float scale,
                      const tr_tensor* out, const tr_tensor* lse, void* stream, bool fuse_update = false,
                      int n_chunks = 0, bool chunk_bf16 = false, int renew = 0, bool may_cut = true) {
  tr_status st;
  if ((st = check_tensor("q", q, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("k", k, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("v", v, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("out", out, !fuse_update, true, 16)) != TR_OK) return st;
  if ((st = check_tensor("lse", lse, false, true, 4)) != TR_OK) return st;
  if ((st = check_written("out", out)) != TR_OK || (st = check_written("lse", lse)) != TR_OK) return st;
  if (q->D != 64 && q->D != 128) return fail(TR_ERR_SHAPE, "head dim %lld not supported (64 or 128)", (long long)q->D);
  if (k->D != q->D || v->D != q->D || out->D != q->D) return fail(TR_ERR_SHAPE, "head dims of q, k, v, out differ");
  if (lse->D != 1) return fail(TR_ERR_SHAPE, "lse must have D = 1");
  if (k->B != q->B || v->B != q->B || out->B != q->B || lse->B != q->B) return fail(TR_ERR_SHAPE, "batch sizes differ");
  if (k->H != v->H || k->S != v->S) return fail(TR_ERR_SHAPE, "k and v shapes differ");
  if (out->H != q->H || lse->H != q->H || out->S != q->S || lse->S != q->S) return fail(TR_ERR_SHAPE, "out/lse shape does not match q");
  if (q->H > 0 && (k->H <= 0 || q->H % k->H)) return fail(TR_ERR_SHAPE, "query heads %lld not a multiple of K/V heads %lld", (long long)q->H, (long long)k->H);
  if (!(scale > 0.f) || !isfinite(scale)) return fail(TR_ERR_UNSUPPORTED, "scale must be finite and > 0");
  if (overlaps(out, q) || overlaps(out, k) || overlaps(out, v) || overlaps(lse, q) || overlaps(lse, k) || overlaps(lse, v) || overlaps(out, lse))
    return fail(TR_ERR_ALIAS, "outputs overlap inputs or each other");
  if ((int64_t)q->B * q->H > (1 << 24)) return fail(TR_ERR_SHAPE, "too many (batch, head) pairs");
  // the K/V staging addresses a 64-key tile with 32-bit byte offsets from the tile base
  if (k->stride_s > ((int64_t)1 << 24) || v->stride_s > ((int64_t)1 << 24))
    return fail(TR_ERR_STRIDE, "stride_s of k and v must not exceed 2^24 elements");

  tr::AttnParams p;
  memset(&p, 0, sizeof(p));
  p.q = (const __bf16*)q->ptr; p.k = (const __bf16*)k->ptr; p.v = (const __bf16*)v->ptr;
  p.out = out->ptr; p.lse = (float*)lse->ptr;
  p.q_sb = q->stride_b; p.q_sh = q->stride_h; p.q_ss = q->stride_s;
  p.k_sb = k->stride_b; p.k_sh = k->stride_h; p.k_ss = k->stride_s;
  p.v_sb = v->stride_b; p.v_sh = v->stride_h; p.v_ss = v->stride_s;
  p.o_sb = out->stride_b; p.o_sh = out->stride_h; p.o_ss = out->stride_s;
  p.l_sb = lse->stride_b; p.l_sh = lse->stride_h; p.l_ss = lse->stride_s;
  set_shape(p, q, k, causal, off64);
  p.scale = scale;
  p.renew = renew;
  p.renew_log2 = q->D == 64 ? 9 : 8;   // four tiles of a 256-row workgroup
  p.gq_log2 = -1;
  for (int sh = 0; sh < 31; sh++)
    if (p.gq == (1 << sh)) p.gq_log2 = sh;
  if (p.n_qtiles > 65535) return fail(TR_ERR_SHAPE, "Sq too long for one launch (at most 65535 query tiles of %d rows)", kMaxRows);
  if ((int64_t)p.n_qtiles * p.B * p.Hq >= ((int64_t)1 << 31)) return fail(TR_ERR_SHAPE, "too many workgroups for one launch");
  if (p.B == 0 || p.Hq == 0 || p.Sq == 0) return TR_OK;
  const int epilogue = fuse_update ? 2 : (out->dtype == TR_F32 ? 1 : 0);
  if (n_chunks > 0) {
    p.n_chunks = n_chunks;
    p.chunk_bf16 = chunk_bf16 ? 1 : 0;
    use_shape(p, choose_shape(p, (int)q->D, false, 8));
    const int step = std::max(1, 65535 / p.n_qtiles);   // chunks one grid holds; the later ones first, as inside a launch
    for (p.chunk_end = n_chunks; p.chunk_end > 0; p.chunk_end = p.chunk_begin) {
      p.chunk_begin = std::max(0, p.chunk_end - step);
      const hipError_t e = tr::launch_block_attn(p, (int)q->D, 2, (hipStream_t)stream);
      if (e != hipSuccess) return fail(TR_ERR_HIP, "chunk attention launch failed: %s", hipGetErrorString(e));
    }
    return TR_OK;
  }
  PartPlan plan;
  const bool planned = plan_parts(p, (int)q->D, may_cut, plan);
  const hipError_t e = launch_planned(p, plan, planned, (int)q->D, epilogue, (hipStream_t)stream);
  if (e != hipSuccess) return fail(TR_ERR_HIP, "block attention launch failed: %s", hipGetErrorString(e));
  return TR_OK;
}

// View of chunk `c` (of length C along S) of a tensor.
tr_tensor chunk_view(const tr_tensor* t, int64_t c, int64_t C) { return rows_view(t, c * C, C); }

inline int pmod(int a, int n) { return ((a % n) + n) % n; }

// Execution order of the block steps, all "devices" replayed in turn, and the number of equal
// segments the sequence is cut into.  Under the causal rule a step whose K/V segment lies
// after its Query segment is dropped (the caller masks ks == qs diagonally).
//   TokenRing (Algorithm 1): iteration i, device j (holds K_j, V_j) works on Query chunk (j-i) mod n.
//   Ring Attention (Sec. 2.1): device j keeps Q_j; at iteration i it holds K/V chunk (j-i) mod n.
//   Zigzag (Sec. 3.3.2): 2n segments, device g owns segments g and 2n-1-g of Q, K and V; the
//     Query pair circulates as in Algorithm 1.
//   Hybrid (Sec. 3.3.3): n = nodes * n_inner devices; K/V travel between nodes as in Ring
//     Attention (outer step t), Algorithm 1 runs among the n_inner devices of each node.
int build_schedule(int schedule, int n, int n_inner, bool causal, std::vector<RingStep>& steps) {
  steps.clear();
  auto add = [&](int qs, int ks) {
    if (!causal || ks <= qs) steps.push_back({qs, ks});
  };
  switch (schedule) {
    case TR_SCHED_TOKENRING:
      for (int i = 0; i < n; i++)
        for (int j = 0; j < n; j++) add(pmod(j - i, n), j);
      return n;
    case TR_SCHED_RING_ATTENTION:
      for (int i = 0; i < n; i++)
        for (int j = 0; j < n; j++) add(j, pmod(j - i, n));
      return n;
    case TR_SCHED_ZIGZAG:
      // Within an iteration the devices work concurrently, each on up to three segment pairs of
      // its own Query pair; they are emitted slot by slot (every device's first pair, then every
      // device's second, ...) so that pairs on distinct Query segments are adjacent and belong to one
      // group.  The order of the blocks each Query segment receives is unaffected.
      // When a Query segment meets both K/V segments of the device (always its later
      // segment), the two are one block step over the device's whole K/V; a device then has at
      // most two steps per iteration, on its two Query segments.
      for (int i = 0; i < n; i++) {
        for (int slot = 0; slot < 4; slot++) {
          for (int j = 0; j < n; j++) {
            const int c = pmod(j - i, n);
            const int qseg[2] = {c, 2 * n - 1 - c}, kseg[2] = {j, 2 * n - 1 - j};
            RingStep dev[4];
            int kept = 0;
            for (int a = 0; a < 2; a++)
              for (int b = 0; b < 2; b++) {
                if (kseg[b] > qseg[a]) continue;
                if (b == 1 && kept > 0 && dev[kept - 1].qs == qseg[a] && dev[kept - 1].ks2 < 0) dev[kept - 1].ks2 = kseg[b];
                else dev[kept++] = {qseg[a], kseg[b]};
              }
            if (slot < kept) steps.push_back(dev[slot]);
          }
        }
      }
      return 2 * n;
    case TR_SCHED_HYBRID: {
      const int nodes = n / n_inner;
      for (int t = 0; t < nodes; t++)
        for (int i = 0; i < n_inner; i++)
          for (int nd = 0; nd < nodes; nd++)
            for (int pp = 0; pp < n_inner; pp++) add(nd * n_inner + pmod(pp - i, n_inner), pmod(nd - t, nodes) * n_inner + pp);
      return n;
    }
    default:
      return 0;
  }
}

// One group of independent steps: steps [begin, end) of the list, all of them their Query segments' first blocks or
// none of them.
constexpr int kGroupMax = 32;
struct StepGroup { size_t begin, end; };

// Splits the step list into groups.  Consecutive steps that touch distinct Query segments and
// are of one kind (first block of their segment, which is written, or a later block, which is
// merged) are independent of each other - they are what different devices compute at the same
// time (at most kGroupMax steps).
std::vector<StepGroup> group_steps(const std::vector<RingStep>& steps, int n_seg) {
  std::vector<StepGroup> groups;
  std::vector<char> started((size_t)n_seg, 0);  // has this Query segment received its first block?
  std::vector<int> in_group((size_t)n_seg, -1); // index of the group that last used the segment
  size_t pos = 0;
  while (pos < steps.size()) {
    const int group_id = (int)groups.size();
    const bool merge = started[(size_t)steps[pos].qs] != 0;
    size_t end = pos;
    while (end < steps.size() && (int)(end - pos) < kGroupMax && (started[(size_t)steps[end].qs] != 0) == merge &&
           in_group[(size_t)steps[end].qs] != group_id) {
      in_group[(size_t)steps[end].qs] = group_id;
      end++;
    }
    for (size_t i = pos; i < end; i++) started[(size_t)steps[i].qs] = 1;
    groups.push_back({pos, end});
    pos = end;
  }
  return groups;
}

// Keys after which a ring of n_seg segments renews the exponent reference of a row: a segment in whole sub-tiles.
int ring_renewal(int64_t seg, int n_seg) { return n_seg > 1 ? (int)(seg / 32 * 32) : 0; }

// Every block step of a schedule on one GPU.  The K/V segments a Query segment meets lie side by side in one
// tensor, and the Update is associative and commutative: the running softmax over the whole visible key range
// folds the blocks in registers, so out and lse are written once and no accumulator is read back.  Against one
// launch per iteration with the Update in the epilogue (the form this replaces; same box, us before -> after):
// S 256 in 4 chunks 29.8 -> 7.9, causal 8192 in 8 segments 620 -> 460, causal 32768 in 8 chunks 7603 -> 6965,
// full 16384 at D 64 3555 -> 3201, GQA 131072 in 16 chunks 113.9 -> 109.2 ms: what goes are the set-up, the
// epilogue and the idle tail of every launch but one.  Query rows beyond what a grid holds go out as further launches.
// The keys are not cut (plan_parts): the result of a schedule is the same bits eagerly, in a graph and on any stream.
//
// A block attended alone has an exponent reference of its own, hence one weight that bf16 holds exactly.  So that the
// result is no further from the exact one than the blocks one by one, the reference is renewed once a segment; segments
// shorter than a sub-tile (32 keys) are attended block by block, a Query tile running through them in one launch
// (16 segments of 16 keys: 1.03e-3 by blocks, 1.17e-3 renewed at every sub-tile, 1.61e-3 with one reference).
tr_status attn_whole(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_seg, bool causal, float scale,
                     const tr_tensor* out, const tr_tensor* lse, void* stream) {
  const int64_t seg = q->S / n_seg, bm = kMaxRows;
  if (seg > 65535 * bm) return fail(TR_ERR_SHAPE, "segments of %lld rows are too long (at most 65535 query tiles of %d rows)", (long long)seg, (int)bm);
  if (n_seg > 1 && seg < 32) {
    const tr_tensor q0 = rows_view(q, 0, seg), k0 = rows_view(k, 0, seg), v0 = rows_view(v, 0, seg);
    const tr_tensor o0 = rows_view(out, 0, seg), l0 = rows_view(lse, 0, seg);
    return attn_common(&q0, &k0, &v0, causal, 0, scale, &o0, &l0, stream, true, n_seg);
  }
  const int renew = ring_renewal(seg, n_seg);
  const int64_t slab = 65535 * bm;
  int64_t r0 = 0;
  do {
    const int64_t rows = std::min(slab, q->S - r0);
    const tr_tensor qs = rows_view(q, r0, rows), os = rows_view(out, r0, rows), ls = rows_view(lse, r0, rows);
    const tr_status st = attn_common(&qs, k, v, causal, r0, scale, &os, &ls, stream, false, 0, false, renew, false);
    if (st != TR_OK) return st;
    r0 += rows;
  } while (r0 < q->S);
  return TR_OK;
}

constexpr size_t kWsAlign = 256;
size_t align_up(size_t x) { return (x + kWsAlign - 1) / kWsAlign * kWsAlign; }

}  // namespace

namespace tr {
TimingEvents take_timing_events() {
  const TimingEvents ev = g_timing;
  g_timing = {nullptr, nullptr};
  return ev;
}
}  // namespace tr

extern "C" {

const char* tr_last_error(void) { return g_err; }

tr_status tr_time_next_kernel(void* start_event, void* stop_event) {
  g_err[0] = 0;
  g_timing.start = static_cast<hipEvent_t>(start_event);
  g_timing.stop = static_cast<hipEvent_t>(stop_event);
  return TR_OK;
}
#ifndef TR_SOURCE_HASH_STR
#define TR_SOURCE_HASH_STR "0000000000000000"
#endif
// The tagged string is also what the build script looks for inside the binary to decide whether
// the library was compiled from the sources on disk.
__attribute__((used)) static const char tr_source_hash_tag[] = "TR_SOURCE_HASH=" TR_SOURCE_HASH_STR;
const char* tr_version(void) { return "tokenring-gfx950 0.2 (sources " TR_SOURCE_HASH_STR ")"; }

tr_status tr_block_attn(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int mask_kind, float scale,
                        const tr_tensor* out, const tr_tensor* lse, void* hip_stream) {
  g_err[0] = 0;
  if (mask_kind != TR_MASK_NONE && mask_kind != TR_MASK_CAUSAL_DIAG) return fail(TR_ERR_UNSUPPORTED, "unknown mask kind %d", mask_kind);
  if (mask_kind == TR_MASK_CAUSAL_DIAG && q && k && q->S != k->S)
    return fail(TR_ERR_SHAPE, "the diagonal causal mask needs Sq == Sk (got %lld, %lld)", (long long)q->S, (long long)k->S);
  return attn_common(q, k, v, mask_kind == TR_MASK_CAUSAL_DIAG, 0, scale, out, lse, hip_stream);
}

tr_status tr_block_attn_causal_at(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int64_t q_pos0, int64_t k_pos0,
                                  float scale, const tr_tensor* out, const tr_tensor* lse, void* hip_stream) {
  g_err[0] = 0;
  if (q_pos0 < 0 || k_pos0 < 0) return fail(TR_ERR_SHAPE, "chunk positions must be >= 0");
  return attn_common(q, k, v, 1, q_pos0 - k_pos0, scale, out, lse, hip_stream);
}

tr_status tr_block_attn_merge(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int mask_kind, float scale,
                              const tr_tensor* out_acc, const tr_tensor* lse_acc, void* hip_stream) {
  g_err[0] = 0;
  if (mask_kind != TR_MASK_NONE && mask_kind != TR_MASK_CAUSAL_DIAG) return fail(TR_ERR_UNSUPPORTED, "unknown mask kind %d", mask_kind);
  if (mask_kind == TR_MASK_CAUSAL_DIAG && q && k && q->S != k->S)
    return fail(TR_ERR_SHAPE, "the diagonal causal mask needs Sq == Sk (got %lld, %lld)", (long long)q->S, (long long)k->S);
  return attn_common(q, k, v, mask_kind == TR_MASK_CAUSAL_DIAG, 0, scale, out_acc, lse_acc, hip_stream, true);
}

// Checks of the host-only views; true: the sizes are in p.
static bool view_sizes(tr::AttnParams& p, const tr_tensor* q, const tr_tensor* k, int causal, int64_t q_pos0, int64_t k_pos0) {
  g_err[0] = 0;
  if (check_tensor("q", q, true, false, 16) != TR_OK || check_tensor("k", k, true, false, 16) != TR_OK) return false;
  if (q_pos0 < 0 || k_pos0 < 0) {
    fail(TR_ERR_SHAPE, "chunk positions must be >= 0");
    return false;
  }
  if ((q->D != 64 && q->D != 128) || k->D != q->D || k->B != q->B || (q->H > 0 && (k->H <= 0 || q->H % k->H))) {
    fail(TR_ERR_SHAPE, "q and k do not fit together");
    return false;
  }
  memset(&p, 0, sizeof(p));
  set_shape(p, q, k, causal, q_pos0 - k_pos0);
  return true;
}

int tr_block_attn_plan(const tr_tensor* q, const tr_tensor* k, int causal, int64_t q_pos0, int64_t k_pos0, int32_t* packed) {
  tr::AttnParams p;
  if (!view_sizes(p, q, k, causal, q_pos0, k_pos0)) return -1;
  PartPlan plan;
  const bool planned = plan_parts(p, (int)q->D, true, plan);
  if (packed) *packed = planned ? plan.pack : 0;
  return planned ? plan.parts : 1;
}

// The launch of a call on these shapes (tr_attn_workgroup); true: it is in p.
static bool view_launch(tr::AttnParams& p, const tr_tensor* q, const tr_tensor* k, int causal, int64_t q_pos0, int64_t k_pos0, int form, int n_chunks) {
  if (!view_sizes(p, q, k, causal, q_pos0, k_pos0)) return false;
  const int D = (int)q->D;
  if (form < TR_FORM_STEP_BF16 || form > TR_FORM_RING_BF16 || n_chunks < 1 || (form >= TR_FORM_RING && (q->S % n_chunks || k->S != q->S))) {
    fail(TR_ERR_SHAPE, "unknown form %d, or a sequence that is no multiple of %d chunks", form, n_chunks);
    return false;
  }
  const int64_t seg = q->S / n_chunks;
  if (form == TR_FORM_RING_BF16 || (form == TR_FORM_RING && n_chunks > 1 && seg < 32)) {
    p.Sq = p.Sk = (int)seg;
    p.n_chunks = n_chunks;
    use_shape(p, choose_shape(p, D, false, 8));
  } else {
    p.renew = form == TR_FORM_RING ? ring_renewal(seg, n_chunks) : 0;
    PartPlan plan;
    const bool planned = plan_parts(p, D, form != TR_FORM_RING, plan);
    settle_launch(p, plan, planned, D, form == TR_FORM_RING ? 1 : form, true);
  }
  return true;
}

int tr_attn_workgroup(const tr_tensor* q, const tr_tensor* k, int causal, int64_t q_pos0, int64_t k_pos0, int form, int n_chunks, int32_t* key_groups) {
  tr::AttnParams p;
  if (!view_launch(p, q, k, causal, q_pos0, k_pos0, form, n_chunks)) return -1;
  if (key_groups) *key_groups = tr::shape_key_groups(p.shape);
  return p.bm;
}

int tr_attn_workgroups_per_unit(const tr_tensor* q, const tr_tensor* k, int causal, int64_t q_pos0, int64_t k_pos0, int form, int n_chunks) {
  tr::AttnParams p;
  if (!view_launch(p, q, k, causal, q_pos0, k_pos0, form, n_chunks)) return -1;
  return tr::shape_per_unit(p.shape, (int)q->D);
}

tr_status tr_merge(const tr_tensor* out_acc, const tr_tensor* lse_acc, const tr_tensor* block_out, const tr_tensor* block_lse,
                   void* hip_stream) {
  g_err[0] = 0;
  tr_status st;
  if ((st = check_tensor("out_acc", out_acc, false, true, 16)) != TR_OK) return st;
  if ((st = check_tensor("lse_acc", lse_acc, false, true, 4)) != TR_OK) return st;
  if ((st = check_tensor("block_out", block_out, true, true, 8)) != TR_OK) return st;
  if ((st = check_tensor("block_lse", block_lse, false, true, 4)) != TR_OK) return st;
  if (block_out->dtype == TR_F32 && (st = check_tensor("block_out", block_out, true, true, 16)) != TR_OK) return st;
  if ((st = check_written("out_acc", out_acc)) != TR_OK || (st = check_written("lse_acc", lse_acc)) != TR_OK) return st;
  if (lse_acc->D != 1 || block_lse->D != 1) return fail(TR_ERR_SHAPE, "lse tensors must have D = 1");
  if (out_acc->D % 4) return fail(TR_ERR_SHAPE, "D = %lld must be a multiple of 4", (long long)out_acc->D);
  if (block_out->B != out_acc->B || block_out->H != out_acc->H || block_out->S != out_acc->S || block_out->D != out_acc->D)
    return fail(TR_ERR_SHAPE, "block_out shape does not match out_acc");
  if (lse_acc->B != out_acc->B || lse_acc->H != out_acc->H || lse_acc->S != out_acc->S) return fail(TR_ERR_SHAPE, "lse_acc shape does not match out_acc");
  if (block_lse->B != out_acc->B || block_lse->H != out_acc->H || block_lse->S != out_acc->S) return fail(TR_ERR_SHAPE, "block_lse shape does not match out_acc");
  if (overlaps(out_acc, block_out) || overlaps(out_acc, block_lse) || overlaps(lse_acc, block_out) || overlaps(lse_acc, block_lse) || overlaps(out_acc, lse_acc))
    return fail(TR_ERR_ALIAS, "accumulator and block tensors overlap");
  if ((int64_t)out_acc->B * out_acc->H * out_acc->S >= ((int64_t)1 << 32))
    return fail(TR_ERR_SHAPE, "too many elements for one launch");

  tr::MergeParams p;
  memset(&p, 0, sizeof(p));
  p.acc_out = (float*)out_acc->ptr; p.acc_lse = (float*)lse_acc->ptr;
  p.blk_out = block_out->ptr; p.blk_lse = (const float*)block_lse->ptr;
  p.ao_sb = out_acc->stride_b; p.ao_sh = out_acc->stride_h; p.ao_ss = out_acc->stride_s;
  p.al_sb = lse_acc->stride_b; p.al_sh = lse_acc->stride_h; p.al_ss = lse_acc->stride_s;
  p.bo_sb = block_out->stride_b; p.bo_sh = block_out->stride_h; p.bo_ss = block_out->stride_s;
  p.bl_sb = block_lse->stride_b; p.bl_sh = block_lse->stride_h; p.bl_ss = block_lse->stride_s;
  p.B = (int)out_acc->B; p.H = (int)out_acc->H; p.S = (int)out_acc->S; p.D = (int)out_acc->D;
  auto dense = [](const tr_tensor* t) {
    return t->stride_s == t->D && t->stride_h == t->S * t->D && t->stride_b == t->H * t->S * t->D;
  };
  p.contiguous = dense(out_acc) && dense(block_out) && dense(lse_acc) && dense(block_lse);
  if (p.B == 0 || p.H == 0 || p.S == 0 || p.D == 0) return TR_OK;
  const hipError_t e = tr::launch_merge(p, block_out->dtype == TR_BF16, (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail(TR_ERR_HIP, "merge launch failed: %s", hipGetErrorString(e));
  return TR_OK;
}

tr_status tr_merge_n(const tr_tensor* out, const tr_tensor* lse, const tr_tensor* const* block_outs,
                     const tr_tensor* const* block_lses, int n, int accumulate, void* hip_stream) {
  g_err[0] = 0;
  tr_status st;
  if (!block_outs || !block_lses) return fail(TR_ERR_NULL, "the arrays of partial results must not be NULL");
  if (n < 1 || n > tr::kMergeNMax) return fail(TR_ERR_SHAPE, "n = %d partials out of range [1, %d]", n, tr::kMergeNMax);
  if ((st = check_tensor("out", out, false, true, 16)) != TR_OK) return st;
  if ((st = check_tensor("lse", lse, false, true, 4)) != TR_OK) return st;
  if ((st = check_written("out", out)) != TR_OK || (st = check_written("lse", lse)) != TR_OK) return st;
  if (lse->D != 1) return fail(TR_ERR_SHAPE, "lse tensors must have D = 1");
  if (out->D % 4) return fail(TR_ERR_SHAPE, "D = %lld must be a multiple of 4", (long long)out->D);
  if (lse->B != out->B || lse->H != out->H || lse->S != out->S) return fail(TR_ERR_SHAPE, "lse shape does not match out");
  if (overlaps(out, lse)) return fail(TR_ERR_ALIAS, "out and lse overlap");
  if ((int64_t)out->B * out->H * out->S >= ((int64_t)1 << 32)) return fail(TR_ERR_SHAPE, "too many elements for one launch");
  const tr_tensor* bo0 = block_outs[0];
  const tr_tensor* bl0 = block_lses[0];
  for (int i = 0; i < n; i++) {
    const tr_tensor* bo = block_outs[i];
    const tr_tensor* bl = block_lses[i];
    if ((st = check_tensor("block_out", bo, true, true, 8)) != TR_OK) return st;
    if (bo->dtype == TR_F32 && (st = check_tensor("block_out", bo, true, true, 16)) != TR_OK) return st;
    if ((st = check_tensor("block_lse", bl, false, true, 4)) != TR_OK) return st;
    if (bo->B != out->B || bo->H != out->H || bo->S != out->S || bo->D != out->D) return fail(TR_ERR_SHAPE, "block_out %d: shape does not match out", i);
    if (bl->B != out->B || bl->H != out->H || bl->S != out->S || bl->D != 1) return fail(TR_ERR_SHAPE, "block_lse %d: shape does not match lse", i);
    if (bo->dtype != bo0->dtype) return fail(TR_ERR_DTYPE, "block_out %d: all partials must have one dtype", i);
    if (bo->stride_b != bo0->stride_b || bo->stride_h != bo0->stride_h || bo->stride_s != bo0->stride_s ||
        bl->stride_b != bl0->stride_b || bl->stride_h != bl0->stride_h || bl->stride_s != bl0->stride_s)
      return fail(TR_ERR_STRIDE, "partial %d: all partials must share their strides", i);
    if (overlaps(out, bo) || overlaps(out, bl) || overlaps(lse, bo) || overlaps(lse, bl))
      return fail(TR_ERR_ALIAS, "partial %d overlaps the result tensors", i);
  }

  tr::MergeNParams p;
  memset(&p, 0, sizeof(p));
  p.out = (float*)out->ptr; p.lse = (float*)lse->ptr;
  for (int i = 0; i < n; i++) { p.blk_out[i] = block_outs[i]->ptr; p.blk_lse[i] = (const float*)block_lses[i]->ptr; }
  p.o_sb = out->stride_b; p.o_sh = out->stride_h; p.o_ss = out->stride_s;
  p.l_sb = lse->stride_b; p.l_sh = lse->stride_h; p.l_ss = lse->stride_s;
  p.bo_sb = bo0->stride_b; p.bo_sh = bo0->stride_h; p.bo_ss = bo0->stride_s;
  p.bl_sb = bl0->stride_b; p.bl_sh = bl0->stride_h; p.bl_ss = bl0->stride_s;
  p.B = (int)out->B; p.H = (int)out->H; p.S = (int)out->S; p.D = (int)out->D;
  p.n = n; p.accumulate = accumulate ? 1 : 0;
  auto dense = [](const tr_tensor* t) {
    return t->stride_s == t->D && t->stride_h == t->S * t->D && t->stride_b == t->H * t->S * t->D;
  };
  p.contiguous = dense(out) && dense(bo0) && dense(lse) && dense(bl0);
  if (p.B == 0 || p.H == 0 || p.S == 0 || p.D == 0) return TR_OK;
  const hipError_t e = tr::launch_merge_n(p, bo0->dtype == TR_BF16, (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail(TR_ERR_HIP, "n-ary merge launch failed: %s", hipGetErrorString(e));
  return TR_OK;
}

size_t tr_ring_attn_blocks_workspace_bytes(const tr_tensor* q, int n_chunks, int block_dtype) {
  if (!q || n_chunks < 1 || q->B < 0 || q->H < 0 || q->S < 0 || q->D < 0 || q->S % n_chunks) return 0;
  if (block_dtype != TR_F32 && block_dtype != TR_BF16) return 0;
  const size_t C = (size_t)(q->S / n_chunks);
  const size_t rows = (size_t)q->B * (size_t)q->H * C;
  return align_up(rows * (size_t)q->D * (size_t)elem_bytes(block_dtype)) + align_up(rows * 4);
}

size_t tr_ring_attn_workspace_bytes(const tr_tensor* q, int n_chunks) {
  return tr_ring_attn_blocks_workspace_bytes(q, n_chunks, TR_F32);
}

}  // extern "C"

namespace {

// Algorithm 1 on one device.  block_dtype TR_F32: attn_whole.  TR_BF16: block by block, every block result after a
// Query chunk's first rounded to bf16 before its Update.  A workspace is only checked.
tr_status ring_attn_impl(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_chunks, int causal,
                         const tr_tensor* out, const tr_tensor* lse, float scale, int block_dtype, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
  if (!q || !k || !v || !out || !lse) return fail(TR_ERR_NULL, "a tensor descriptor is NULL");
  if (n_chunks < 1) return fail(TR_ERR_SHAPE, "n_chunks must be >= 1");
  if (q->S < 0 || q->S % n_chunks) return fail(TR_ERR_SHAPE, "sequence length %lld is not a multiple of n_chunks %d", (long long)q->S, n_chunks);
  if (k->S != q->S || v->S != q->S) return fail(TR_ERR_SHAPE, "q, k, v must have the same sequence length");
  if (out->dtype != TR_F32) return fail(TR_ERR_DTYPE, "out must be fp32 (it is the merge accumulator)");
  if (q->D > 0 && !(scale > 0.f)) scale = 1.0f / sqrtf((float)q->D);
  const int64_t C = q->S / n_chunks;

  // Validate every argument once through the single-step checks (chunk 0 views have the
  // same strides, dtypes and alignment class as all others).
  tr_status st;
  if ((st = check_tensor("q", q, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("k", k, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("v", v, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("out", out, false, true, 16)) != TR_OK) return st;
  if ((st = check_tensor("lse", lse, false, true, 4)) != TR_OK) return st;
  if ((st = check_written("out", out)) != TR_OK || (st = check_written("lse", lse)) != TR_OK) return st;
  if (out->B != q->B || out->H != q->H || out->S != q->S || out->D != q->D || lse->B != q->B || lse->H != q->H || lse->S != q->S || lse->D != 1)
    return fail(TR_ERR_SHAPE, "out/lse shape does not match q");

  const size_t need = tr_ring_attn_blocks_workspace_bytes(q, n_chunks, block_dtype);
  const size_t rows = (size_t)q->B * (size_t)q->H * (size_t)C;
  const bool given = workspace != nullptr;
  if (given && workspace_bytes == 0) return fail(TR_ERR_WORKSPACE, "workspace given with size 0 (need %zu bytes)", need);
  if (given && n_chunks > 1 && rows > 0) {
    if (((uintptr_t)workspace) % kWsAlign) return fail(TR_ERR_WORKSPACE, "workspace must be %zu-byte aligned", kWsAlign);
    if (workspace_bytes < need) return fail(TR_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", workspace_bytes, need);
    tr_tensor ws_all;  // alias check of the whole workspace against the user tensors
    memset(&ws_all, 0, sizeof(ws_all));
    ws_all.ptr = workspace; ws_all.dtype = TR_F32;
    ws_all.B = 1; ws_all.H = 1; ws_all.S = 1; ws_all.D = (int64_t)(need / 4);
    if (overlaps(&ws_all, q) || overlaps(&ws_all, k) || overlaps(&ws_all, v) || overlaps(&ws_all, out) || overlaps(&ws_all, lse))
      return fail(TR_ERR_ALIAS, "workspace overlaps a tensor argument");
  }

  if (overlaps(out, q) || overlaps(out, k) || overlaps(out, v) || overlaps(lse, q) || overlaps(lse, k) || overlaps(lse, v) || overlaps(out, lse))
    return fail(TR_ERR_ALIAS, "outputs overlap inputs or each other");
  if (n_chunks > 8192) return fail(TR_ERR_SHAPE, "n_chunks %d too large (at most 8192)", n_chunks);

  // fp32 blocks reach the Update unrounded, so folding them in registers is the same operation; bf16
  // blocks are rounded one by one on their way, as the caller asked.
  if (block_dtype == TR_F32) return attn_whole(q, k, v, n_chunks, causal != 0, scale, out, lse, hip_stream);
  const tr_tensor q0 = chunk_view(q, 0, C), k0 = chunk_view(k, 0, C), v0 = chunk_view(v, 0, C);
  const tr_tensor o0 = chunk_view(out, 0, C), l0 = chunk_view(lse, 0, C);
  return attn_common(&q0, &k0, &v0, causal != 0, 0, scale, &o0, &l0, hip_stream, true, n_chunks, true);
}

}  // namespace

extern "C" {

tr_status tr_ring_attn(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_chunks, int causal,
                       const tr_tensor* out, const tr_tensor* lse, float scale, void* workspace, size_t workspace_bytes,
                       void* hip_stream) {
  g_err[0] = 0;
  return ring_attn_impl(q, k, v, n_chunks, causal, out, lse, scale, TR_F32, workspace, workspace_bytes, hip_stream);
}

tr_status tr_ring_attn_blocks(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_chunks, int causal,
                              const tr_tensor* out, const tr_tensor* lse, float scale, int block_dtype, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  g_err[0] = 0;
  if (block_dtype != TR_F32 && block_dtype != TR_BF16) return fail(TR_ERR_DTYPE, "block_dtype %d is neither fp32 nor bf16", block_dtype);
  if (!workspace) return fail(TR_ERR_WORKSPACE, "tr_ring_attn_blocks needs a workspace");
  return ring_attn_impl(q, k, v, n_chunks, causal, out, lse, scale, block_dtype, workspace, workspace_bytes, hip_stream);
}

tr_status tr_ring_attn_noalloc(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_chunks, int causal,
                               const tr_tensor* out, const tr_tensor* lse, float scale, void* hip_stream) {
  g_err[0] = 0;
  // size check first (needs no device)
  const size_t need = tr_ring_attn_blocks_workspace_bytes(q, n_chunks, TR_F32);
  if (q && n_chunks >= 1 && q->S >= 0 && q->S % n_chunks == 0 && need > (size_t)TR_NOALLOC_SCRATCH_BYTES)
    return fail(TR_ERR_WORKSPACE, "tr_ring_attn_noalloc: one block result needs %zu bytes, the scratch limit is %zu "
                "(B * Hq * (S / n_chunks) * (D + 1) * 4 bytes must fit); use tr_ring_attn (it needs no workspace)", need,
                (size_t)TR_NOALLOC_SCRATCH_BYTES);
  if (!q || !k || !v || !out || !lse) return fail(TR_ERR_NULL, "a tensor descriptor is NULL");
  return ring_attn_impl(q, k, v, n_chunks, causal, out, lse, scale, TR_F32, nullptr, 0, hip_stream);
}

int64_t tr_schedule_steps(int schedule, int n_devices, int n_inner, int causal, int32_t* steps_out, int64_t capacity) {
  g_err[0] = 0;
  if (n_devices < 1 || n_devices > 4096) { fail(TR_ERR_SHAPE, "n_devices %d out of range [1, 4096]", n_devices); return -1; }
  if (schedule < TR_SCHED_TOKENRING || schedule > TR_SCHED_HYBRID) { fail(TR_ERR_UNSUPPORTED, "unknown schedule %d", schedule); return -1; }
  if (schedule == TR_SCHED_ZIGZAG && !causal) { fail(TR_ERR_UNSUPPORTED, "the zigzag partition only exists for the causal case"); return -1; }
  if (schedule == TR_SCHED_HYBRID && (n_inner < 1 || n_devices % n_inner)) {
    fail(TR_ERR_SHAPE, "hybrid schedule: n_inner %d must divide n_devices %d", n_inner, n_devices);
    return -1;
  }
  std::vector<RingStep> steps;
  const int n_seg = build_schedule(schedule, n_devices, n_inner, causal != 0, steps);
  const std::vector<StepGroup> groups = group_steps(steps, n_seg);
  int64_t n_out = 0;   // a step on a pair of K/V segments is reported as its two segment pairs
  for (size_t g = 0; g < groups.size(); g++)
    for (size_t i = groups[g].begin; i < groups[g].end; i++)
      for (int half = 0; half < (steps[i].ks2 >= 0 ? 2 : 1); half++, n_out++)
        if (steps_out && n_out < capacity) {
          steps_out[3 * n_out] = steps[i].qs;
          steps_out[3 * n_out + 1] = half ? steps[i].ks2 : steps[i].ks;
          steps_out[3 * n_out + 2] = (int32_t)g;
        }
  return n_out;
}

tr_status tr_ring_attn_sched(const tr_tensor* q, const tr_tensor* k, const tr_tensor* v, int n_devices, int causal,
                             int schedule, int n_inner, const tr_tensor* out, const tr_tensor* lse, float scale,
                             void* hip_stream) {
  g_err[0] = 0;
  if (!q || !k || !v || !out || !lse) return fail(TR_ERR_NULL, "a tensor descriptor is NULL");
  if (n_devices < 1 || n_devices > 4096) return fail(TR_ERR_SHAPE, "n_devices %d out of range [1, 4096]", n_devices);
  if (schedule < TR_SCHED_TOKENRING || schedule > TR_SCHED_HYBRID) return fail(TR_ERR_UNSUPPORTED, "unknown schedule %d", schedule);
  if (schedule == TR_SCHED_ZIGZAG && !causal)
    return fail(TR_ERR_UNSUPPORTED, "the zigzag partition only exists for the causal case");
  if (schedule == TR_SCHED_HYBRID && (n_inner < 1 || n_devices % n_inner))
    return fail(TR_ERR_SHAPE, "hybrid schedule: n_inner %d must divide n_devices %d", n_inner, n_devices);
  const int n_seg = schedule == TR_SCHED_ZIGZAG ? 2 * n_devices : n_devices;
  if (q->S < 0 || q->S % n_seg) return fail(TR_ERR_SHAPE, "sequence length %lld is not a multiple of %d segments", (long long)q->S, n_seg);
  if (k->S != q->S || v->S != q->S) return fail(TR_ERR_SHAPE, "q, k, v must have the same sequence length");
  if (out->dtype != TR_F32) return fail(TR_ERR_DTYPE, "out must be fp32 (it is the merge accumulator)");
  if (q->D > 0 && !(scale > 0.f)) scale = 1.0f / sqrtf((float)q->D);
  tr_status st;
  if ((st = check_tensor("q", q, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("k", k, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("v", v, true, false, 16)) != TR_OK) return st;
  if ((st = check_tensor("out", out, false, true, 16)) != TR_OK) return st;
  if ((st = check_tensor("lse", lse, false, true, 4)) != TR_OK) return st;
  if ((st = check_written("out", out)) != TR_OK || (st = check_written("lse", lse)) != TR_OK) return st;
  if (out->B != q->B || out->H != q->H || out->S != q->S || out->D != q->D || lse->B != q->B || lse->H != q->H || lse->S != q->S || lse->D != 1)
    return fail(TR_ERR_SHAPE, "out/lse shape does not match q");

  if (overlaps(out, q) || overlaps(out, k) || overlaps(out, v) || overlaps(lse, q) || overlaps(lse, k) || overlaps(lse, v) || overlaps(out, lse))
    return fail(TR_ERR_ALIAS, "outputs overlap inputs or each other");
  return attn_whole(q, k, v, n_seg, causal != 0, scale, out, lse, hip_stream);
}

}  // extern "C"
