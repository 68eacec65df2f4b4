// Host-side interface between the C ABI (api.hip) and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mea {

// Element strides of one [B, H, n, d] tensor (batch, head, row); features
// are contiguous.  Row 0 of (batch, head) bh starts at head_base(s, bh, H).
struct TensorStrides {
  int64_t b, h, r;
};
__host__ __device__ inline int64_t head_base(const TensorStrides& s, int bh, int heads) {
  return (int64_t)(bh / heads) * s.b + (int64_t)(bh % heads) * s.h;
}

// Keys visible to every query of (batch, head) bh: the batch's valid key
// length from kv_len (device array [B], clamped to [0, n_k]) or all n_k.
// Keys from there to n_k are masked like keys past the end; they stay
// readable memory, so loads are bounded by n_k.
__device__ inline int64_t valid_keys(const int* kv_len, int bh, int heads, int64_t n_k) {
  if (kv_len == nullptr) return n_k;
  const int64_t l = kv_len[bh / heads];
  return l < 0 ? 0 : (l > n_k ? n_k : l);
}

// Arguments of the forward kernels (passed by value).
struct FwdParams {
  const void* q;
  const void* k;
  const void* v;
  void* o;
  float* lse;     // [B*H, n_q] or null
  void* o_lo;     // 16-bit o only: rounding residual of o, contiguous [B*H, n_q, DV], or null
  float* part_o;  // split partials [S, B*H, n_q, D] (n_splits > 1)
  float* part_m;  // [S, B*H, n_q]
  float* part_l;  // [S, B*H, n_q]
  // Second partial buffer for the staged combine (n_splits > kCombineGroup):
  // ceil(S / kCombineGroup) splits in the same layout.
  float* part2_o;
  float* part2_m;
  float* part2_l;
  const int* kv_len;  // [B] valid keys per batch, or null (all n_k)
  int64_t n_q;
  int64_t n_k;
  int64_t keys_per_split;  // multiple of the key tile
  int bh;                  // B * H
  int n_qtiles;
  int n_splits;
  // Waves that share 32 queries in the 4-wave kernel (1, 2 or 4; it derives its
  // query tiles from this), or 0: the kernel that n_qtiles' tiles belong to.
  int stream_waves;
  int tile_order;    // causal problems: 0 head major, 1 tile major, 2 folded (tile_item)
  float scale;       // score scale
  float scale_log2;  // scale * log2(e)
  int heads;         // H (bh = b * H + h)
  TensorStrides sq, sk, sv, so;
};

// The summaries of more than kCombineGroup key ranges are combined in stages
// of kCombineGroup ranges each (Section 4's combine applied as a tree), so
// that the work stays parallel when there are few rows and many ranges.
constexpr int kCombineGroup = 16;

// Lazy reference maximum of the forward kernels (Section 3's running maximum,
// raised lazily): a tile raises the reference only when one of its scores
// exceeds it by more than this many powers of two, so weights stay <= 2^8 and
// the running numerator and denominator are rescaled only on such tiles.
constexpr float kRescaleSlack = 8.0f;
constexpr float kRescaleBound = 256.0f;  // 2^kRescaleSlack

// Floats of the second partial buffer (0 when the combine is one stage).
inline size_t combine_stage_floats(int64_t n_splits, int64_t rows, int64_t d) {
  if (n_splits <= kCombineGroup) return 0;
  const int64_t s1 = (n_splits + kCombineGroup - 1) / kCombineGroup;
  return (size_t)s1 * (size_t)rows * (size_t)(d + 2);
}

// Arguments of the backward kernels.
struct BwdParams {
  const void* q;
  const void* k;
  const void* v;
  const void* o;
  const void* o_lo;  // residual of a 16-bit o (contiguous [B*H, n_q, DV]) or null
  const void* d_o;
  const float* lse;
  void* dq;
  void* dk;
  void* dv;
  // Per-row initial values of the score and dP accumulators, written by the
  // preprocess kernel: s_init = -lse / scale (so that P = 2^(c * (S + s_init)),
  // c = scale * log2 e) and dp_init = -D with D_i = dO_i . O_i (so that
  // dS = P * (dP + dp_init)).  Rows n_q .. n_q_pad - 1 contribute nothing.
  // Problems that bwd_uses_row_records names (16-bit inputs and outputs,
  // d = 64) hold them as one 16-byte record per row, eight bf16 values {s_hi,
  // s_mid, s_lo, 0, d_hi, d_mid, d_lo, 0} whose three parts sum to s_init and
  // dp_init in float32 (padding rows: s = -2^100, d = 0), so that the two-group
  // kernels put them into the accumulators with one bf16 MFMA against a
  // constant operand; the others hold [B*H, n_q_pad] float32 arrays (padding
  // rows -inf and 0).
  float* s_init;
  float* dp_init;
  uint4* row_rec;
  // 16-bit inputs with float32 o and dO: dO rounded to the input dtype
  // (contiguous [B*H, n_q, DV]), written by the preprocess, so that the
  // dK/dV and dQ kernels of 16-bit outputs run on it; or null.
  void* do16;
  const int* kv_len;  // [B] valid keys per batch, or null (all n_k)
  int64_t n_q_pad;  // n_q rounded up to kBwdRowPad
  int64_t n_q;
  int64_t n_k;
  int bh;
  int n_qtiles;  // query tiles of the dQ kernel
  int n_ktiles;  // key tiles of the dK/dV kernel
  int tile_order;  // causal problems: see FwdParams
  int dq_first;    // one launch: dQ's workgroups before dK/dV's (bwd_dq_first)
  float scale;
  float scale_log2;
  int heads;  // H (bh = b * H + h)
  TensorStrides sq, sk, sv, so, sdo, sdq, sdk, sdv;
};

// Row padding of the backward's per-row arrays (a multiple of every query
// tile the backward kernels stage).
constexpr int kBwdRowPad = 64;

// Whether a backward's per-row values are 16-byte records, and with them
// whether it may run the two-group kernels (bwd_two_group_fills has the last
// word); every other backward takes two float32 arrays.  The host's workspace
// layout and the kernels' choice both come from this one predicate.  Causal problems of up to MEA_T64_BWD_CAUSAL_SMALL
// queries run the 4-wave kernels: measured on causal bf16 d = 64 problems,
// n = 1024-2048 (128-256 heads) took 5-13 % less time with them; at 3072 the
// two kinds tie, and from 4096 queries on the two-group kernels take 3-12 %
// less (6-7 % more before their plain tiles dropped the mask).  Unmasked
// problems of up to MEA_T64_BWD_SHORT queries run them too (the two-group dQ
// kernel's 256-query tiles are mostly padding there): bf16 d = 64, two-group /
// 4-wave, dK/dV + dQ: 2.796 / 2.293 ms at 8x16 heads, 65 queries, 65536
// keys; 3.123 / 2.886 at 256; 4.543 / 4.563 at 512; 0.226 / 0.180 at 4x32
// heads, 128 queries, 4096 keys; 0.343 / 0.324 at 512; 0.550 / 0.552 at
// 1024; 0.292 / 0.303 at 4x16x2048^2.  The two kinds give bitwise the same
// gradients.
#ifndef MEA_T64_BWD_CAUSAL_SMALL
#define MEA_T64_BWD_CAUSAL_SMALL 2048
#endif
#ifndef MEA_T64_BWD_SHORT
#define MEA_T64_BWD_SHORT 512
#endif
// Whether the two-group backward kernels exist for these types and head
// dimensions (whatever the problem's shape).
constexpr bool bwd_two_group_exists(bool is16, int d, int dv, bool same_out_dtype) {
  return is16 && d == 64 && dv == 64 && same_out_dtype;
}
constexpr bool bwd_two_group(bool is16, int d, int dv, bool same_out_dtype, bool causal, int64_t n_q) {
  return bwd_two_group_exists(is16, d, dv, same_out_dtype) && !(causal && n_q <= MEA_T64_BWD_CAUSAL_SMALL) &&
         !(!causal && n_q <= MEA_T64_BWD_SHORT);
}
// Whether a problem with records runs the two-group kernels (256 keys or
// queries per workgroup, one workgroup per CU) or the 4-wave kernels (128, two
// per CU, dK/dV and dQ in one launch), which read records too and give bitwise
// the same gradients while one wave takes all of a column's rows.  Below one
// two-group round (256 workgroups) the 4-wave kernels fill more of the chip;
// causal grids need two rounds before their uneven workgroups even out, and up
// to 1024 unmasked queries the last 256-query tile is padding to a large part, so
// that they need long keys and full rounds.
// Measured, dK/dV + dQ + preprocess in us, 4-wave / two-group, bf16 d = 64:
// unmasked 1x8x4096 (128 workgroups) 133 / 176, 1x10x4096 (160) 182 / 182,
// 1x12x4096 (192) 211 / 187, 1x4x8192 (128) 241 / 330, 16x8x600 75 / 96,
// 8x8x1024 (256) 78 / 77, 64 heads of 1024 on 16384 keys (256) 1029 / 954, 128 of 900
// (512) 1966 / 1825, 128 of 1000 on 2048 256 / 261, 64 of 768 on 16384 (192) 749 / 803,
// 100 of 1024 (400) 1523 / 1568; causal 1x8x8192 (256) 287 / 357, 2x16x4096 (512)
// 330 / 343, 1x16x8192 (512) 549 / 476, 1x8x16384 (512) 969 / 877.
inline bool bwd_two_group_fills(bool causal, int64_t n_q, int64_t n_k, int64_t bh) {
  const int64_t wq = bh * ((n_q + 255) / 256), wk = bh * ((n_k + 255) / 256);
  if (!causal && n_q <= 1024)
    return n_q > 768 && n_k >= 4096 && wq >= 224 && (wq + 255) / 256 * 256 - wq <= 32;
  return (wq < wk ? wq : wk) >= (causal ? 512 : 160);
}
// Workgroups of the 4-wave backward kernels when every wave has 32 rows of its
// own: 128 keys (dK/dV) or 128 queries (dQ) each.
inline int64_t bwd_tiles128(int64_t n_q, int64_t n_k, int64_t bh) {
  return bh * ((n_k + 127) / 128 + (n_q + 127) / 128);
}
// Waves of a 4-wave backward workgroup that share one 32-key column (dK/dV) or
// one set of 32 queries (dQ) and split the streamed rows between them: 4 or 2
// where 128-row workgroups would leave CUs idle.  Each such workgroup streams
// all rows for fewer columns, so it pays only until the chip is full; a causal
// problem is half as full as its tiles suggest once the tiles are many.  At
// d = 128 the wider stages leave LDS for two waves and one workgroup per CU.
// Measured, backward in us with 1 / 2 / 4 waves, bf16: d = 64 1x1x4096 (64
// tiles of 128) 99 / 80 / 55, 1x8x1024 (128) 30 / 25 / 20, 2x8x1024 (256) 32 /
// 28 / 37, 1x4x4096 (256) 96 / 83 / 103, 3x8x1024 (384) 38 / 43 / 52; causal
// 1x8x4096 (512) 109 / 90 / 118, 4x8x1024 (512) 37 / 42 / 53, 2x8x4096 (1024)
// 171 / 172 / 230; d = 128 2x8x512 (128) 32 / 25, causal 1x8x2000 (256) 101 /
// 68, unmasked 87 / 101, causal 1x12x2000 (384) 109 / 111.
// float32 fits one workgroup per CU whatever the shares, and its passes are
// longer: 64 rows a share pay up to the same counts, 32 rows (one stage of 128
// rows) only where a quarter of the CUs would be busy.  1 / 2 / 4 waves, d = 64
// 1x4x1000 (64 tiles) 168 / 66 / 47, 1x8x1000 (128) 168 / 69 / 81, 2x8x1000
// (256) 172 / 113 / 159, 3x8x1000 (384) 175 / 176; causal 1x8x1000 (128) 172 /
// 68 / 57, 4x8x1000 (512) 179 / 167, 1x8x4000 (512) 630 / 430 / 598; d = 128
// 1x8x1000 (128) 188 / 133, 2x8x1000 (256) 193 / 244, causal 191 / 204.
inline int bwd_stream_waves(bool is16, bool causal, int dmax, int64_t n_q, int64_t n_k, int64_t bh) {
  int64_t tiles = bwd_tiles128(n_q, n_k, bh);
  if (causal && (n_q > 1024 || (!is16 && dmax == 64))) tiles /= 2;
  if (dmax == 128) return tiles <= 128 ? 2 : 1;
  return tiles <= (is16 ? 128 : 64) ? 4 : (tiles <= 256 ? 2 : 1);
}
// Whether dK/dV and dQ run in one launch (4-wave kernels, one wave per
// column): faster wherever the two grids can fill each other's gaps, on large
// grids at d = 128 the mixed register allocation costs more.  Separate / one
// launch: d = 64 1x1x4096 162 / 99 us, 8x8x1024 causal 74 / 65, 32x32x1024
// causal 893 / 859; d = 128 8x16x2048 causal (4096 tiles) 647 / 622, 4x32x4096
// causal (8192) 2014 / 2042, 4x32x8192 causal 7280 / 7515.  Where a few dQ
// workgroups over many keys are the whole call nothing fills a gap, and that
// allocation's slower dQ (d = d_v = 128, unmasked) shows: 2x128 on 65536 keys (2 dQ
// workgroups) 1479 / 1649, 4x512 on 16384 (16) 408 / 428, 1x2048 on 65536 (16) 1551
// / 1668, but 16x256 on 16384 (32) 463 / 437, 5x128 on 4096 (5) 112 / 112; and not where
// dK/dV, alone, would take more than a tenth of the time (1x2048 on 16384 449 / 427).
inline bool bwd_one_launch(bool is16, bool causal, int d, int dv, int64_t n_q, int64_t n_k, int64_t bh) {
  if (is16 && !causal && d == 128 && dv == 128 && n_k > 6144 && bh * ((n_q + 127) / 128) <= 28 &&
      10 * n_q * ((bh * ((n_k + 127) / 128) + 255) / 256) <= n_k)
    return false;
  return (d == 64 && dv == 64) || bwd_tiles128(n_q, n_k, bh) <= 4096;
}
// Order of one launch's two kinds of workgroups, unmasked 16-bit (causal grids and
// float32 ones start with dK/dV): the longer ones first, so that the short ones fill what they leave.
// A dQ workgroup streams n_k keys and a dK/dV workgroup n_q queries, about twice
// as long each (half as much again at d = d_v = 128).  bf16, separate launches / dK/dV
// first / dQ first, us: d = 64 2x4096 on 62291 keys 1229 / 1454 / 939, 4x4096 on 14081
// 352 / 385 / 246, 32x1024 on 2185 119 / 95 / 88, but 16x2048 on 4096 153 / 141 / 149,
// 8x4096 on 4096 180 / 125 / 134; d = 128 32x1024 on 14632 856 / 955 / 782, 16x1498
// on 2931 168 / 179 / 153, but 5x4096 on 4096 243 / 165 / 189; d = 128, d_v = 64
// 2x8192 on 12765 752 / 481 / 521.
inline bool bwd_dq_first(int d, int dv, int64_t n_q, int64_t n_k) {
  return d == 128 && dv == 128 ? n_k > n_q + n_q / 2 : n_k > 2 * n_q;
}
// dtype: 0 float32, 1 fp16, 2 bf16; d and dv the head dimensions of q, k and
// of v, o.
inline bool bwd_uses_row_records(int dtype, int d, int dv, bool out_f32, bool causal, int64_t n_q) {
  return bwd_two_group(dtype != 0, d, dv, !out_f32, causal, n_q);
}

// Queries per workgroup of the 4-wave forward with one wave per 32 queries.
constexpr int kFwdBq = 128;
// 16-bit d = d_v = 64 causal forward: the two-group kernel (512-query
// workgroups, returns 512) for problems of more than MEA_T64_FWD_CAUSAL_SMALL
// queries with at least MEA_T64_FWD_CAUSAL_MIN_PAIRS (batch x heads x n_q^2)
// query-key pairs and at least MEA_T64_FWD_CAUSAL_MIN_WGS such workgroups,
// else the 4-wave kernel with 128-query workgroups (128).  A 512-query
// workgroup spends 8 key tiles on the diagonal, half of that work masked,
// which short sequences do not amortise, and a small grid of such workgroups
// (a few hundred, for 256 CUs) balances poorly.  Measured on causal bf16
// problems, the 4-wave kernel at three workgroups per CU against the
// two-group kernel: 2-3 % faster at 4x32x4608 and 8x16x6144, 5 % at
// 1x4x32768 (256 two-group workgroups), and faster at every n <= 4096; the
// two-group kernel 3.5, 8 and 18 % faster at 4x32x8192, 2x16x12288 and
// 1x16x16384.  Host plan and launch both use this.
#ifndef MEA_T64_FWD_CAUSAL_SMALL
#define MEA_T64_FWD_CAUSAL_SMALL 6144
#endif
#ifndef MEA_T64_FWD_CAUSAL_MIN_PAIRS
#define MEA_T64_FWD_CAUSAL_MIN_PAIRS 2.5e9
#endif
#ifndef MEA_T64_FWD_CAUSAL_MIN_WGS
#define MEA_T64_FWD_CAUSAL_MIN_WGS 384
#endif
inline int fwd_causal64_bq(int64_t n_q, int64_t bh) {
  const bool big = n_q > MEA_T64_FWD_CAUSAL_SMALL &&
                   (double)bh * (double)n_q * (double)n_q >= (double)MEA_T64_FWD_CAUSAL_MIN_PAIRS &&
                   bh * ((n_q + 511) / 512) >= MEA_T64_FWD_CAUSAL_MIN_WGS;
  return big ? 512 : kFwdBq;
}
// 16-bit d = d_v forward without the causal mask: the 4-wave kernel with
// 128-query workgroups when the two-group kernel's one query tile (BQ_pp =
// 512 queries at d = 64, 256 at d = 128) would be at least half padding,
// else the two-group kernel.  Measured (bf16, two-group / 4-wave): d = 64,
// 8x16 heads, 65536 keys: 0.907 / 0.497 ms at 65 queries, 1.009 / 0.797 at
// 256, 1.036 / 1.118 at 300, 1.184 / 1.532 at 512; d = 128: 1.003 / 0.781 at
// 65, 1.060 / 0.840 at 128, 1.041 / 1.361 at 160, 1.169 / 1.479 at 256.
// Above that the two kernels measured within about 10 % either way, with
// the two-group kernel ahead on the larger problems.
inline bool fwd_pp_unmasked(int64_t n_q, int bq_pp) { return 2 * n_q > bq_pp; }
// 16-bit d = d_v = 64 forward: queries per workgroup (512: the two-group
// kernel; 128: the 4-wave kernel).  These two name the kernels' tiles; fwd_grid
// has the last word and may take the 4-wave kernel where they name the two-group one.
inline int fwd64_bq(int64_t n_q, int64_t bh, bool causal) {
  if (causal) return fwd_causal64_bq(n_q, bh);
  return fwd_pp_unmasked(n_q, 512) ? 512 : kFwdBq;
}
// 16-bit d = d_v = 128 forward: 256 (the two-group kernel) or 128 (the 4-wave
// kernel) queries per workgroup.
inline int fwd128_bq(int64_t n_q, bool causal) { return causal || fwd_pp_unmasked(n_q, 256) ? 256 : kFwdBq; }

// How a forward that is not decode-shaped fills the chip: the two-group kernel
// (waves 0; where fwd64_bq or fwd128_bq name it) or the 4-wave kernel with 1, 2
// or 4 waves per 32 queries, and the key ranges that are combined afterwards.
struct FwdGrid {
  int waves;       // 0: two-group kernel
  int64_t ranges;  // key ranges wanted (the plan rounds them to whole tiles)
};
inline int64_t clamp64(int64_t x, int64_t lo, int64_t hi) { return x < lo ? lo : (x > hi ? hi : x); }
// Keys of a staged tile of the 4-wave forward with sw waves per 32 queries.
inline int fwd_stream_tile(bool is16, int sw) { return sw == 1 ? (is16 ? 64 : 32) : 32 * sw; }
// What a forward kernel takes: us to start and end, and us per 1000 keys of a
// workgroup with 1, 2 or 3 of its kind on the CU (0: that many do not fit).
// Fitted to 19 kinds of unmasked forward, 100 to 5000 measurements each over
// 1-200 heads, 1-16384 queries and 1-300000 keys (median errors 3-8 %).
struct FwdRate {
  double fixed, keys[3];
};
inline FwdRate fwd_rate(bool is16, int d, int dv, int waves) {
  if (!is16) {
    if (d == 64 && dv == 64) return waves == 1 ? FwdRate{5.3, {58.6, 92.9, 0}} : FwdRate{6.5, {43.6, 62.7, 0}};
    if (d == dv) return waves == 1 ? FwdRate{6.6, {113, 0, 0}} : FwdRate{4.6, {99.6, 0, 0}};
    if (d == 64) return waves == 1 ? FwdRate{6.8, {112, 151, 0}} : FwdRate{4.7, {71.3, 0, 0}};
    return waves == 1 ? FwdRate{6.6, {102, 148, 0}} : FwdRate{4.5, {76.1, 0, 0}};
  }
  if (d == 64 && dv == 64) {
    if (waves == 0) return {6.9, {27.2, 0, 0}};
    if (waves == 1) return {4.7, {14.4, 21.5, 28.9}};
    return waves == 2 ? FwdRate{4.8, {10.4, 14.2, 18.3}} : FwdRate{4.8, {7.05, 9.41, 0}};
  }
  if (d == dv) {
    if (waves == 0) return {5.7, {23.9, 0, 0}};
    return waves == 1 ? FwdRate{6.0, {25.2, 35.6, 0}} : FwdRate{6.4, {16.1, 23.9, 0}};
  }
  if (d == 64) return waves == 1 ? FwdRate{5.6, {20.7, 28.6, 0}} : FwdRate{5.7, {13.4, 19.2, 0}};
  return waves == 1 ? FwdRate{5.0, {18.2, 27.4, 0}} : FwdRate{5.4, {12.8, 18.2, 0}};
}
// Unmasked forwards: the kernel and the number of ranges whose rounds take least.
// n workgroups of L keys on 256 CUs take whole rounds of as many as fit, and a
// last one of fewer; ranges add a combine (3 us, 0.3 for each range up to 16 that it
// reads in a chain, 3 more where it is staged) and the writing and reading of the
// partial sums.  Only numbers of ranges that fill another CU's worth (n just below a
// multiple of 256) can be the best, or on a grid that never fills one a few.  Counting
// rounds finds what thresholds on the same numbers missed, us, thresholds /
// rounds: d = 64 1x17x8192 459 / 382, 65x1024 on 65536 keys 1988 / 1235, 136x1024
// on 65536 2567 / 2436; d = 128 40x2000 on 16383 776 / 626, 9x4000 on 262144 5119 /
// 3988; d = 64, d_v = 128 17x4096 on 16384 760 / 568, d = 128, d_v = 64 17x2048 on
// 16384 420 / 285; float32 d = 64 24x1500 on 8192 679 / 478, d = 128 17x2048 on
// 4096 884 / 610.  The chain of a combine shows on small grids, with it flat at 4 us /
// as here: d = 64 2x128 on 4096 18.0 / 13.1, 16x65 on 1024 12.3 / 10.4, d = 128 12x129
// on 3001 23.3 / 19.8.  With at most 3 rounds of ranges in place of 9: 136x1024 on 65536
// keys d = 64 2940.
inline FwdGrid fwd_grid_unmasked(bool is16, int d, int dv, int64_t n_q, int64_t n_k, int64_t bh) {
  const bool same = d == dv;
  const int64_t bq = d == 64 ? 512 : 256;
  FwdGrid best = {1, 1};
  double t_best = 0;
  for (int waves = 0; waves <= (is16 && same && d == 64 ? 4 : 2); waves += waves == 2 ? 2 : 1) {
    // Short streams of the two-group kernel's tiles do not pay for its prologue.
    if (waves == 0 &&
        !(is16 && same && n_k >= 512 && (d == 64 ? fwd64_bq(n_q, bh, false) : fwd128_bq(n_q, false)) == bq))
      continue;
    const int64_t rows = waves ? 128 / waves : bq, q_wgs = bh * ((n_q + rows - 1) / rows);
    const int64_t bk = waves ? fwd_stream_tile(is16, waves) : 64, k_tiles = (n_k + bk - 1) / bk;
    const int64_t r_max = clamp64(n_k / 128, 1, 64);
    const FwdRate k = fwd_rate(is16, d, dv, waves);
    const int per_cu = k.keys[2] > 0 ? 3 : (k.keys[1] > 0 ? 2 : 1);
    int64_t r_last = 0;
    for (int64_t m = -3; m <= 9; ++m) {
      const int64_t r = m <= 0 ? (m ? clamp64(2 << -m, 1, r_max) : 1) : clamp64(256 * m / q_wgs, 1, r_max);
      if (r == r_last || (m < 0 && r * q_wgs > 256)) continue;
      r_last = r;
      const int64_t tiles = (k_tiles + r - 1) / r, ranges = (k_tiles + tiles - 1) / tiles;
      const int64_t on_cu = (q_wgs * ranges + 255) / 256, last = on_cu % per_cu;
      double t = (double)(tiles * bk) * 1e-3 *
                 ((double)(on_cu / per_cu) * k.keys[per_cu - 1] + (last ? k.keys[last - 1] : 0));
      if (waves == 2 && n_q <= 32) t *= 1.15;  // half the waves have no queries
      t += k.fixed;
      if (ranges > 1) {
        t += 3 + 0.3 * (double)(ranges < kCombineGroup ? ranges : kCombineGroup) +
             (double)(bh * n_q * ranges * (dv + 2) * 8) * 0.22e-6 + (ranges > kCombineGroup ? 3 : 0);
        t *= 1.02;  // near ties to one range
      }
      if (t_best == 0 || t < t_best) {
        t_best = t;
        best = {waves, r};
      }
    }
  }
  return best;
}
// Causal forwards.  tiles = 128-query tiles of the 4-wave kernel, wgs = the
// two-group kernel's workgroups.  More waves per 32 queries and more key ranges
// both make more workgroups of the same work; waves re-read K and V through L2
// once more each, ranges cost partial sums and a combine, so waves fill the chip
// at short keys.  At long ones (from 3072 queries) the heaviest tile alone takes
// twice the mean of a grid that is resident at once, and ranges of about a round
// cut it.  us, without / with this rule's choice:
//   d = 64: 2x8x1024 (tiles 128) two-group 20 / 4 waves 13, 4x8x1024 (256) 20 / 2
//     waves 16; ranges 1x1x8192 (64) 66 / 33, 1x5x8192 (320) 122 / 92, 1x12x4096
//     (384) 63.9 / 61.9, but 1x14x4096 (448) 63.9 / 68.4, 1x8x4096 (256, 2 waves
//     without) 49.3 / 51.7
//   d = 128: 1x32x2047 (512) two-group 91 / 1 wave 62, 4x8x1024 (256) 33 / 2
//     waves 26, 16x16x600 (1280) 68 / 1 wave 63, but 4x32x2047 (2048) 179 / 1
//     wave 191; ranges 1x1x16384 (128) 266 / 112, 1x5x8192 (320) 206 / 110
//   d_v != d: ranges, d = 64 1x1x16384 (128) 225 / 116, 1x5x8192 (320) 175 / 132;
//     d = 128 1x2x8192 (128) 107 / 57
inline FwdGrid fwd_grid(bool is16, bool causal, int d, int dv, int64_t n_q, int64_t n_k, int64_t bh) {
  if (!causal) return fwd_grid_unmasked(is16, d, dv, n_q, n_k, bh);
  const int64_t tiles = bh * ((n_q + 127) / 128), wgs = bh * ((n_q + 255) / 256);
  const bool same = d == dv, wide = d == 128 || dv == 128;
  if (!is16) {
    const int w = tiles <= 32 ? 2 : 1;
    const int64_t slots = same && wide ? 256 : 512;
    return {w, n_k > n_q ? 1 : clamp64(slots / (tiles * w), 1, clamp64(n_k / (w == 2 ? 128 : 256), 1, 8))};
  }
  const bool long_keys = n_q >= 3072 && n_k >= 3072 && n_k <= n_q;
  if (same && d == 64) {
    if (fwd64_bq(n_q, bh, true) == 512) return {0, 1};
    if (long_keys && tiles > 32 && tiles <= 400) return {1, (767 + tiles) / tiles};
    return {tiles <= 128 ? 4 : (tiles <= 256 ? 2 : 1), tiles <= 32 ? clamp64(n_k / 256, 1, 4) : 1};
  }
  if (same) {
    if (tiles > 512 && n_q > 1024) return {0, 1};
    if (long_keys && wgs < 256) return {0, clamp64((255 + wgs) / wgs, 1, 16)};
  } else if (long_keys && tiles <= 320) {
    return {1, clamp64((575 + tiles) / tiles, 1, 16)};
  }
  return {tiles <= 256 ? 2 : 1, tiles <= 64 && n_k <= n_q && n_k >= 1024 ? 2 : 1};
}

// Order of a causal grid's tiles (tile_item in device.hpp).  Tile major starts
// the heaviest tiles of every head first, so the last workgroups are light
// ones: 5-30 % on grids of one to a few rounds (us, head / tile major: forward
// 8x16x2048 d = 64 133 / 112, 4x32x2047 d = 128 208 / 184; backward 8x8x1024 d =
// 64 70 / 52, 8x8x1024 d = 128 119 / 91, 4x32x4096 d = 64 1128 / 1071; forward +
// backward 3x5x9000 d = 64 1102 / 836, 2x32x8192 d = 64 2671 / 2493, 8x16x2000
// d = 128 float32 4531 / 3914).  It touches every head at once, which pays while
// K and V (and Q and dO, as much again) stay in the 256 MiB last-level cache.
// Past 128 MiB of K and V it gains little or loses, and the extra traffic costs
// clock in the kernels after it too: forward + backward 8x32x2047 d = 128 (256
// MiB) 1575 / 1593, 7x9x10364 d = 64, d_v = 128 (250 MB) 6805 / 7266, 4x32x8192 d =
// 128 (512 MiB) 9040 / 9510.  Folded evens out a grid that is resident at once
// (1x32x2047 d = 128 forward 65.5 / 61.9).
inline int causal_tile_order(int64_t kv_bytes, int64_t grid, bool may_fold) {
  if (kv_bytes > (int64_t)128 << 20) return 0;
  return may_fold && grid <= 512 ? 2 : 1;
}

// dtype codes follow mea_dtype: 0 = f32, 1 = f16, 2 = bf16.
// out_f32: o (and, in the backward, do) are float32 instead of the input dtype.
// Decode-shaped forward: 16-bit inputs and at most 64 queries per (batch,
// head) run the key-streaming decode kernel (key tile fwd_decode_tile(d)).
inline bool fwd_uses_decode(int dtype, int d, int dv, int64_t n_q) { return dtype != 0 && d == dv && n_q <= 64; }
inline int fwd_decode_tile(int d) { return d == 64 ? 64 : 32; }
hipError_t launch_decode(const FwdParams& p, int dtype, int d, bool causal, bool out_f32, hipStream_t stream);
// dv: head dimension of v and o (equal to d, or the other of 64 and 128).
hipError_t launch_fwd(const FwdParams& p, int dtype, int d, int dv, bool causal, bool out_f32,
                      hipStream_t stream);
hipError_t launch_bwd(const BwdParams& p, int dtype, int d, int dv, bool causal, bool out_f32,
                      hipStream_t stream);

}  // namespace mea
