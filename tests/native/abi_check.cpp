// Native driver of the C ABI's host code for the sanitizer build (test
// infrastructure).  The kernel launchers are recording stubs
// (launch_stubs.cpp), so nothing runs on a GPU: every call either fails
// validation or reaches a stub, whose recorded arguments are checked here --
// the key-split plan covers every key exactly once, the workspace regions the
// entry point carves lie inside the caller's buffer and do not overlap, and
// sizes near the int64 limits are rejected instead of overflowing.  Built
// with -fsanitize=address,undefined.  Exit status = number of failures.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <vector>

#include "../../include/mea.h"
#include "../../paper_2112_05682_amd/csrc/device.hpp"
#include "../../paper_2112_05682_amd/csrc/kernels.hpp"

namespace mea {
extern FwdParams g_last_fwd;
extern BwdParams g_last_bwd;
extern int g_fwd_calls, g_bwd_calls;
}  // namespace mea

static int failures = 0;
#define CHECK(cond, ...)                                   \
  do {                                                     \
    if (!(cond)) {                                         \
      fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
      fprintf(stderr, __VA_ARGS__);                        \
      fprintf(stderr, "\n");                               \
      ++failures;                                          \
    }                                                      \
  } while (0)

// Fake, 256-byte aligned device addresses: the stubs never dereference them.
static char* const WS = reinterpret_cast<char*>(uintptr_t(1) << 40);
static void* const P = reinterpret_cast<void*>(uintptr_t(1) << 36);

static mea_problem prob(int64_t B, int64_t H, int64_t nq, int64_t nk, int64_t d, int dtype, int causal,
                        int64_t dv = 0, int out_f32 = 0) {
  mea_problem p;
  memset(&p, 0, sizeof(p));
  p.batch = B;
  p.heads = H;
  p.n_q = nq;
  p.n_k = nk;
  p.d = d;
  p.dtype = dtype;
  p.causal = causal;
  p.scale = 0.125f;
  p.out_f32 = out_f32;
  p.d_v = dv;
  return p;
}

static bool inside(const void* a, size_t bytes, const char* base, size_t total) {
  const char* c = static_cast<const char*>(a);
  return c >= base && c + bytes <= base + total;
}
static bool disjoint(const void* a, size_t na, const void* b, size_t nb) {
  const char *x = static_cast<const char*>(a), *y = static_cast<const char*>(b);
  return x + na <= y || y + nb <= x;
}

static void check_fwd_plan(int64_t B, int64_t H, int64_t nq, int64_t nk, int64_t d, int dtype, int causal) {
  mea_problem p = prob(B, H, nq, nk, d, dtype, causal);
  size_t need = 0;
  CHECK(mea_attention_fwd_workspace_size(&p, &need) == MEA_OK, "fwd ws size");
  const int before = mea::g_fwd_calls;
  const mea_status st = mea_attention_fwd(&p, P, P, P, P, static_cast<float*>(P), nullptr,
                                          need ? WS : nullptr, need, nullptr);
  CHECK(st == MEA_OK && mea::g_fwd_calls == before + 1, "fwd call %d", (int)st);
  const mea::FwdParams& f = mea::g_last_fwd;
  if (dtype != MEA_F32 && nq > 64) {
    // The 16-bit plan's tiles are those of the kernel that the type and sizes name;
    // a 4-wave grid (stream_waves) makes its own at the launch (check_fwd_grid).
    const int64_t bq = d == 64 ? mea::fwd64_bq(nq, B * H, causal) : mea::fwd128_bq(nq, causal);
    CHECK(f.n_qtiles == (nq + bq - 1) / bq, "query tiles of %lld", (long long)bq);
  }
  // Keys the plan must cover: all of them, except that a decode-shaped causal
  // problem (16-bit, at most 64 queries) can see only its first n_q keys.
  const bool decode = dtype != MEA_F32 && nq <= 64;
  const int64_t n_keys = decode && causal && nk > nq ? nq : nk;
  CHECK(f.n_splits >= 1 && f.keys_per_split >= 1, "plan");
  CHECK((int64_t)f.n_splits * f.keys_per_split >= n_keys, "splits cover the keys (n_q %lld n_k %lld)",
        (long long)nq, (long long)nk);
  CHECK((int64_t)(f.n_splits - 1) * f.keys_per_split < n_keys, "no empty split");
  CHECK((need == 0) == (f.n_splits == 1), "workspace iff splits");
  if (f.n_splits > 1) {
    const size_t rows = (size_t)f.n_splits * (size_t)(B * H) * (size_t)nq;
    CHECK(inside(f.part_o, rows * d * 4, WS, need) && inside(f.part_m, rows * 4, WS, need) &&
              inside(f.part_l, rows * 4, WS, need),
          "partials inside the workspace (n_k %lld)", (long long)nk);
    CHECK(disjoint(f.part_o, rows * d * 4, f.part_m, rows * 4) && disjoint(f.part_m, rows * 4, f.part_l, rows * 4),
          "partials overlap");
    if (f.n_splits > mea::kCombineGroup) {
      const size_t r2 = (size_t)((f.n_splits + mea::kCombineGroup - 1) / mea::kCombineGroup) * (size_t)(B * H) * nq;
      CHECK(f.part2_o && inside(f.part2_o, r2 * d * 4, WS, need) && inside(f.part2_m, r2 * 4, WS, need) &&
                inside(f.part2_l, r2 * 4, WS, need),
            "stage buffer inside the workspace");
      CHECK(disjoint(f.part2_o, r2 * (d + 2) * 4, f.part_o, rows * (d + 2) * 4), "stage buffer overlaps");
    }
  }
}

// The grid that reaches the launcher is fwd_grid's: its kernel, ranges of whole
// staged tiles of that kernel that cover the keys without an empty one, and
// partials of all of them inside the workspace, for every head dimension pair.
static void check_fwd_grid(int64_t BH, int64_t nq, int64_t nk, int64_t d, int64_t dv, int dtype, int causal) {
  mea_problem p = prob(1, BH, nq, nk, d, dtype, causal, dv == d ? 0 : dv);
  size_t need = 0;
  CHECK(mea_attention_fwd_workspace_size(&p, &need) == MEA_OK, "fwd ws size");
  CHECK(mea_attention_fwd(&p, P, P, P, P, static_cast<float*>(P), nullptr, need ? WS : nullptr, need, nullptr) == MEA_OK,
        "fwd call %lld x %lld x %lld", (long long)BH, (long long)nq, (long long)nk);
  const mea::FwdParams& f = mea::g_last_fwd;
  const bool is16 = dtype != MEA_F32;
  const mea::FwdGrid g = mea::fwd_grid(is16, causal != 0, (int)d, (int)dv, nq, nk, BH);
  CHECK(f.stream_waves == g.waves && (g.waves == 0 || g.waves == 1 || g.waves == 2 || g.waves == 4), "kernel %d",
        f.stream_waves);
  CHECK(g.waves != 4 || (is16 && d == 64 && dv == 64), "four waves where no such kernel is built");
  const int64_t bq = d == 64 ? 512 : 256;
  CHECK(g.waves || (is16 && d == dv && f.n_qtiles == (nq + bq - 1) / bq), "two-group kernel on %lld-query tiles",
        (long long)bq);
  const int64_t tile = g.waves ? mea::fwd_stream_tile(is16, g.waves) : 64;
  CHECK(g.ranges >= 1 && g.ranges <= 64 && f.n_splits <= g.ranges, "ranges %d of %lld", f.n_splits, (long long)g.ranges);
  CHECK(f.keys_per_split % tile == 0 && f.keys_per_split * f.n_splits >= nk && f.keys_per_split * (f.n_splits - 1) < nk,
        "ranges of whole tiles (%lld x %lld x %lld, d %lld)", (long long)BH, (long long)nq, (long long)nk, (long long)d);
  CHECK((need == 0) == (f.n_splits == 1), "workspace iff ranges");
  if (f.n_splits == 1) return;
  const size_t rows = (size_t)f.n_splits * (size_t)BH * (size_t)nq;
  CHECK(inside(f.part_o, rows * dv * 4, WS, need) && inside(f.part_m, rows * 4, WS, need) &&
            inside(f.part_l, rows * 4, WS, need) && disjoint(f.part_o, rows * dv * 4, f.part_m, rows * 4) &&
            disjoint(f.part_m, rows * 4, f.part_l, rows * 4) && disjoint(f.part_o, rows * dv * 4, f.part_l, rows * 4),
        "partials apart and inside the workspace");
  if (f.n_splits <= mea::kCombineGroup) return;
  const size_t r2 = (size_t)((f.n_splits + mea::kCombineGroup - 1) / mea::kCombineGroup) * (size_t)BH * nq;
  CHECK(inside(f.part2_o, r2 * (dv + 2) * 4, WS, need) && f.part2_m == f.part2_o + r2 * dv && f.part2_l == f.part2_m + r2 &&
            disjoint(f.part2_o, r2 * (dv + 2) * 4, f.part_o, rows * (dv + 2) * 4),
        "second partials apart and inside the workspace");
}

// Every order of a causal grid's tiles takes its (tile, group) items once each.
static void check_tile_order(int n_tiles, int groups) {
  const int n = n_tiles * groups;
  for (int order = 0; order < 3; ++order) {
    std::vector<int> taken(n, 0);
    for (int w = 0; w < n; ++w) {
      const mea::TileItem it = mea::tile_item(w, n, n_tiles, order);
      const bool ok = it.tile >= 0 && it.tile < n_tiles && it.group >= 0 && it.group < groups;
      CHECK(ok, "order %d of %d x %d: item of workgroup %d", order, n_tiles, groups, w);
      if (ok) ++taken[it.group * n_tiles + it.tile];
    }
    int wrong = 0;
    for (int t : taken) wrong += t != 1;
    CHECK(wrong == 0, "order %d of %d x %d: %d items not taken once", order, n_tiles, groups, wrong);
  }
}

// The order the launcher gets is causal_tile_order's for the grid it launches:
// folded orders on the 4-wave kernel's resident grids alone, none unmasked.
static void check_tile_order_plan(int64_t BH, int64_t nq, int64_t d, int64_t dv, int dtype) {
  for (int causal = 0; causal < 2; ++causal) {
    mea_problem p = prob(1, BH, nq, nq, d, dtype, causal, dv == d ? 0 : dv);
    size_t need = 0;
    CHECK(mea_attention_fwd_workspace_size(&p, &need) == MEA_OK &&
              mea_attention_fwd(&p, P, P, P, P, static_cast<float*>(P), nullptr, need ? WS : nullptr, need, nullptr) == MEA_OK,
          "fwd call");
    const mea::FwdParams& f = mea::g_last_fwd;
    const int64_t rows = f.stream_waves ? 128 / f.stream_waves : (d == 64 ? 512 : 256);
    const int64_t grid = (nq + rows - 1) / rows * BH * f.n_splits, bytes = BH * nq * (d + dv) * (dtype == MEA_F32 ? 4 : 2);
    const int want = !causal || bytes > (int64_t)128 << 20 ? 0 : (f.stream_waves && grid <= 512 ? 2 : 1);
    CHECK(f.tile_order == want, "order %d of a %lld-workgroup grid, %lld x %lld, d %lld", f.tile_order, (long long)grid,
          (long long)BH, (long long)nq, (long long)d);
  }
}

// Unmasked grids just past a whole round of a kernel's workgroups do not run a
// second, nearly empty one: the plan's rounds, in keys, stay within a third of
// the work divided evenly over the chip's slots (2000 keys and more in each,
// where ranges cost little beside them).
static void check_fwd_rounds(int64_t BH, int64_t nq, int64_t nk, int64_t d, int64_t dv) {
  check_fwd_grid(BH, nq, nk, d, dv, MEA_BF16, 0);
  const mea::FwdParams& f = mea::g_last_fwd;
  const int64_t rows = f.stream_waves ? 128 / f.stream_waves : (d == 64 ? 512 : 256), q_tiles = (nq + rows - 1) / rows;
  const int64_t slots = 256 * (f.stream_waves == 0 ? 1 : (d == 64 && dv == 64 ? (f.stream_waves == 4 ? 2 : 3) : 2));
  const int64_t wgs = BH * q_tiles * f.n_splits, rounds = (wgs + slots - 1) / slots;
  const double even = (double)(BH * q_tiles) * nk / slots;
  if (even < 2000) return;
  CHECK((double)(rounds * f.keys_per_split) < 1.34 * even, "%lld x %lld x %lld d %lld: %lld rounds of %lld keys, even %.0f",
        (long long)BH, (long long)nq, (long long)nk, (long long)d, (long long)rounds, (long long)f.keys_per_split, even);
}

static void check_bwd_carving(int64_t B, int64_t H, int64_t nq, int64_t d, int dtype, int out_f32, int causal = 0) {
  mea_problem p = prob(B, H, nq, 300, d, dtype, causal, 0, out_f32);
  size_t need = 0;
  CHECK(mea_attention_bwd_workspace_size(&p, &need) == MEA_OK, "bwd ws size");
  CHECK(mea_attention_bwd(&p, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, WS, need, nullptr) == MEA_OK,
        "bwd call");
  const mea::BwdParams& b = mea::g_last_bwd;
  const size_t rows = (size_t)(B * H) * (size_t)b.n_q_pad;
  CHECK(b.n_q_pad >= nq && b.n_q_pad % mea::kBwdRowPad == 0 && b.n_q_pad - nq < mea::kBwdRowPad, "row padding");
  // 16-bit inputs with float32 outputs keep a 16-bit copy of dO, and the
  // kernels of 16-bit outputs (and their per-row layout) then run.
  const bool do16 = dtype != MEA_F32 && out_f32;
  CHECK((b.do16 != nullptr) == do16, "dO copy carved exactly for 16-bit inputs with float32 outputs");
  // The layout the host carved is the one the kernels of this problem read.
  const bool rec = mea::bwd_two_group(dtype != MEA_F32, (int)d, (int)d, !out_f32 || do16, causal != 0, nq);
  CHECK((b.row_rec != nullptr) == rec && (b.s_init == nullptr) == rec && (b.dp_init == nullptr) == rec,
        "per-row layout matches the kernels");
  if (b.row_rec) {
    CHECK(inside(b.row_rec, rows * 16, WS, need), "records inside the workspace");
  } else {
    CHECK(inside(b.s_init, rows * 4, WS, need) && inside(b.dp_init, rows * 4, WS, need), "arrays inside");
    CHECK(disjoint(b.s_init, rows * 4, b.dp_init, rows * 4), "per-row arrays overlap");
  }
  if (b.do16) {
    const size_t cbytes = (size_t)(B * H) * (size_t)nq * (size_t)d * 2;
    CHECK(inside(b.do16, cbytes, WS, need), "dO copy inside the workspace");
    CHECK(b.row_rec ? disjoint(b.do16, cbytes, b.row_rec, rows * 16)
                    : disjoint(b.do16, cbytes, b.s_init, rows * 4) && disjoint(b.do16, cbytes, b.dp_init, rows * 4),
          "dO copy overlaps the per-row values");
  }
  CHECK(mea_attention_bwd(&p, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, WS, need - 1, nullptr) ==
            MEA_ERR_WORKSPACE,
        "short workspace accepted");
}

int main() {
  // Validation: every rejection happens before a launch.
  const int calls0 = mea::g_fwd_calls + mea::g_bwd_calls;
  struct Bad {
    mea_problem p;
    mea_status want;
  } bad[] = {
      {prob(1, 1, 0, 10, 64, MEA_BF16, 0), MEA_ERR_INVALID_ARG},
      {prob(1, 1, 10, 10, 96, MEA_BF16, 0), MEA_ERR_UNSUPPORTED},
      {prob(1, 1, 10, 10, 64, 9, 0), MEA_ERR_UNSUPPORTED},
      {prob(1, 1, 10, 10, 64, MEA_BF16, 3), MEA_ERR_INVALID_ARG},
      {prob(1, 1, (int64_t)1 << 31, 10, 64, MEA_BF16, 0), MEA_ERR_INVALID_ARG},
      {prob((int64_t)1 << 40, (int64_t)1 << 40, 10, 10, 64, MEA_BF16, 0), MEA_ERR_INVALID_ARG},
      {prob((int64_t)1 << 30, 4, ((int64_t)1 << 31) - 1, ((int64_t)1 << 31) - 1, 128, MEA_BF16, 0),
       MEA_ERR_INVALID_ARG},
      {prob(INT64_MAX, 1, 1, 1, 64, MEA_BF16, 0), MEA_ERR_INVALID_ARG},
      {prob(1, 1, 10, 10, 64, MEA_BF16, 0, -64), MEA_ERR_INVALID_ARG},
  };
  for (const Bad& c : bad) {
    size_t ws = 0;
    CHECK(mea_attention_fwd_workspace_size(&c.p, &ws) == c.want, "validation");
    CHECK(mea_attention_fwd(&c.p, P, P, P, P, nullptr, nullptr, WS, 1 << 30, nullptr) == c.want, "fwd validation");
    CHECK(mea_attention_bwd(&c.p, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, WS, 1 << 30, nullptr) ==
              c.want,
          "bwd validation");
    CHECK(mea_attention_bwd_noalloc(&c.p, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, nullptr) ==
              c.want,
          "noalloc validation");
  }
  // Strides near the int64 limit are rejected, not overflowed.
  mea_problem ps = prob(4, 4, 100, 100, 64, MEA_BF16, 0);
  mea_strides st;
  memset(&st, 0, sizeof(st));
  const mea_tensor_strides cont = {4 * 100 * 64, 100 * 64, 64};
  st.q = st.k = st.v = st.o = st.d_o = st.dq = st.dk = st.dv = cont;
  st.k.batch = INT64_MAX - 7;
  ps.strides = &st;
  CHECK(mea_attention_fwd(&ps, P, P, P, P, nullptr, nullptr, nullptr, 0, nullptr) == MEA_ERR_INVALID_ARG,
        "overflowing stride accepted");
  st.k = cont;
  st.dq.head = 0;
  CHECK(mea_attention_bwd(&ps, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, WS, 1 << 30, nullptr) ==
            MEA_ERR_INVALID_ARG,
        "output head stride 0 accepted");
  // The allocation-free backward rejects problems beyond its static scratch.
  mea_problem big = prob(1, 64, 16384 + 1, 128, 64, MEA_BF16, 0);
  CHECK(mea_attention_bwd_noalloc(&big, P, P, P, P, nullptr, P, static_cast<float*>(P), P, P, P, nullptr) ==
            MEA_ERR_SCRATCH,
        "oversized problem accepted by the allocation-free backward");
  CHECK(mea::g_fwd_calls + mea::g_bwd_calls == calls0, "a rejected call reached a launcher");
  CHECK(strlen(mea_status_string(MEA_ERR_SCRATCH)) > 10 && strcmp(mea_status_string((mea_status)77), "unknown status") == 0,
        "status strings");

  // Planning and workspace carving over a sweep of shapes.
  const int64_t nks[] = {1, 63, 64, 65, 1000, 4095, 40000, 200001, (int64_t)1 << 20, ((int64_t)1 << 22) + 3};
  for (int64_t nk : nks)
    for (int dt : {MEA_F32, MEA_BF16})
      for (int causal : {0, 1})
        for (int64_t nq : {(int64_t)1, (int64_t)100, (int64_t)300, (int64_t)4096, (int64_t)4097})
          check_fwd_plan(1, 1, nq, nk, 64, dt, causal);
  check_fwd_plan(2, 3, 256, 1 << 20, 128, MEA_F16, 0);
  const struct { int64_t d, dv; } dims[] = {{64, 64}, {128, 128}, {64, 128}, {128, 64}};
  for (auto w : dims)
    for (int dt : {MEA_F32, MEA_BF16})
      for (int causal : {0, 1})
        for (int64_t bh : {1, 2, 3, 7, 17, 33, 64, 129, 257, 600})
          for (int64_t nq : {65, 127, 128, 129, 255, 257, 511, 513, 1024, 3071, 3072, 4097, 16384})
            for (int64_t nk : {1, 31, 33, 64, 127, 129, 255, 511, 513, 1023, 2048, 3071, 3073, 4097, 16383, 16384, 65537, 300001})
              check_fwd_grid(bh, nq, nk, w.d, w.dv, dt, causal);
  for (auto w : dims)
    for (int64_t bh : {1, 3, 9, 17, 33, 65, 100, 129, 200, 255, 257, 300, 400, 513, 600})
      for (int64_t nq : {512, 1024, 4096, 8192})
        for (int64_t nk : {16383, 16384, 65536})
          check_fwd_rounds(bh, nq, nk, w.d, w.dv);
  for (int n_tiles : {1, 2, 3, 5, 8, 9, 16, 31, 64, 511})
    for (int groups : {1, 2, 7, 8, 32, 57, 64, 101}) check_tile_order(n_tiles, groups);
  for (auto w : dims)
    for (int dt : {MEA_F32, MEA_BF16})
      for (int64_t bh : {1, 32, 64, 65, 257})
        for (int64_t nq : {65, 1024, 2047, 4096, 8192}) check_tile_order_plan(bh, nq, w.d, w.dv, dt);
  // A long causal head alone: ranges, where the heaviest tile would be the call.
  for (auto w : dims) {
    check_fwd_grid(1, 16384, 16384, w.d, w.dv, MEA_BF16, 1);
    CHECK(mea::g_last_fwd.n_splits >= 3, "one long causal head, d %lld: %d ranges", (long long)w.d, mea::g_last_fwd.n_splits);
  }
  CHECK(mea::fwd_grid(true, true, 64, 64, 3200, 3200, 16).ranges == 2 &&  // 400 and 425 tiles of 128 queries
            mea::fwd_grid(true, true, 64, 64, 3200, 3200, 17).ranges == 1 &&
            mea::fwd_grid(true, true, 64, 64, 3071, 3071, 8).ranges == 1,
        "causal ranges end with a resident grid, and start at 3072 keys");
  // The longer of dQ's and dK/dV's workgroups start first, and a few long dQ ones
  // at d = d_v = 128 have a launch of their own.
  CHECK(mea::bwd_dq_first(64, 64, 100, 201) && !mea::bwd_dq_first(64, 64, 100, 200) &&
            mea::bwd_dq_first(128, 64, 1, 3) && !mea::bwd_dq_first(64, 128, 4096, 4096) &&
            mea::bwd_dq_first(128, 128, 100, 151) && !mea::bwd_dq_first(128, 128, 100, 150),
        "order of one launch");
  CHECK(!mea::bwd_one_launch(true, false, 128, 128, 614, 6145, 1) &&
            mea::bwd_one_launch(true, false, 128, 128, 615, 6145, 1) &&
            !mea::bwd_one_launch(true, false, 128, 128, 10, 8192, 28) &&
            mea::bwd_one_launch(true, false, 128, 128, 10, 8192, 29) &&
            mea::bwd_one_launch(true, false, 128, 128, 128, 6144, 1) &&
            mea::bwd_one_launch(true, true, 128, 128, 128, 6145, 1) &&
            mea::bwd_one_launch(false, false, 128, 128, 128, 6145, 1) &&
            mea::bwd_one_launch(true, false, 64, 128, 128, 6145, 1) &&
            mea::bwd_one_launch(true, false, 64, 64, 128, 1 << 20, 64) &&
            !mea::bwd_one_launch(true, false, 64, 128, 128, 1 << 20, 1),
        "launches of the 4-wave backward");
  CHECK(mea::bwd_two_group_fills(false, 769, 4096, 56) && !mea::bwd_two_group_fills(false, 768, 4096, 64) &&
            !mea::bwd_two_group_fills(false, 1024, 4095, 64) && !mea::bwd_two_group_fills(false, 1024, 4096, 55) &&
            !mea::bwd_two_group_fills(false, 1024, 4096, 65) && mea::bwd_two_group_fills(false, 1024, 4096, 120) &&
            mea::bwd_two_group_fills(false, 1025, 4096, 65),
        "two-group backward of up to 1024 queries");
  // Both sides of each bound of the causal d = 64 kernel choice.
  for (int64_t nq : {(int64_t)6144, (int64_t)6145})
    check_fwd_plan(2, 64, nq, nq, 64, MEA_BF16, 1);
  for (int64_t h : {(int64_t)4, (int64_t)6}) check_fwd_plan(1, h, 32768, 32768, 64, MEA_F16, 1);
  for (int64_t nq : {(int64_t)12288, (int64_t)12800}) check_fwd_plan(1, 16, nq, nq, 64, MEA_BF16, 1);
  // Unmasked: the 4-wave kernel up to half of the two-group kernel's tile.
  for (int64_t nq : {(int64_t)256, (int64_t)257}) check_fwd_plan(2, 3, nq, 1000, 64, MEA_BF16, 0);
  for (int64_t nq : {(int64_t)128, (int64_t)129}) check_fwd_plan(2, 3, nq, 1000, 128, MEA_F16, 0);
  CHECK(mea::fwd64_bq(256, 6, false) == 128 && mea::fwd64_bq(257, 6, false) == 512 &&
            mea::fwd128_bq(128, false) == 128 && mea::fwd128_bq(129, false) == 256 && mea::fwd128_bq(100, true) == 256,
        "unmasked kernel choice");
  CHECK(mea::fwd_causal64_bq(6144, 128) == 128 && mea::fwd_causal64_bq(6145, 128) == 512 &&
            mea::fwd_causal64_bq(32768, 4) == 128 && mea::fwd_causal64_bq(32768, 6) == 512 &&
            mea::fwd_causal64_bq(12288, 16) == 128 && mea::fwd_causal64_bq(12800, 16) == 512,
        "causal d = 64 kernel choice");
  for (int64_t nq : {(int64_t)1, (int64_t)63, (int64_t)64, (int64_t)65, (int64_t)512, (int64_t)513, (int64_t)2048,
                     (int64_t)2049, (int64_t)16384})
    for (int dt : {MEA_F32, MEA_BF16})
      for (int64_t d : {(int64_t)64, (int64_t)128}) {
        for (int causal = 0; causal < 2; ++causal) {
          check_bwd_carving(2, 3, nq, d, dt, 0, causal);
          if (dt != MEA_F32) check_bwd_carving(2, 3, nq, d, dt, 1, causal);
        }
      }
  if (failures == 0) printf("abi_check ok\n");
  return failures;
}
