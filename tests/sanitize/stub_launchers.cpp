// Stand-ins for the kernel launchers, linked with the host planner
// (layout.cpp, api.cpp) into a CPU-only library built with AddressSanitizer
// and UndefinedBehaviorSanitizer.  Test infrastructure only: no GPU code runs.
//
// Every launcher checks the schedule it is handed against the invariants the
// kernels rely on (segments and key ranges inside their tables, tile and unit
// counts that add up, halved tiles on idle CUs, the merge's row blocks, the FP8
// store's amax accumulators cleared and taken once, rows inside the buffers,
// the pointers a launch reads)
// and aborts with a message on the first violation; a clean call returns
// hipSuccess (0) and counts the launch.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <cmath>

#include "rc_internal.h"

namespace {

long g_launches = 0;
long g_runs = 0;  // runs of the last copy table
long g_wgs = 0;   // work-groups of the last attention launch
const float* g_amax = nullptr;  // accumulators that the last attention launch clears or takes maxima into
long g_taken = 0;  // (batch, head)s whose amax it takes
long g_linear = -1;  // tile of the last projection, or 5 + the part of a cut one
long g_heads = -1;  // (batch, head)s whose amax the last FP8 prefill's attention launch takes

[[noreturn]] void fail(const char* what, long a, long b) {
  fprintf(stderr, "stub launcher: broken schedule: %s (%ld, %ld)\n", what, a, b);
  fflush(stderr);
  abort();
}

#define REQUIRE(cond, a, b) \
  do {                      \
    if (!(cond)) fail(#cond, long(a), long(b)); \
  } while (0)

void check_params(const rc::Params& p, int D, bool balanced) {
  using namespace rc;
  REQUIRE(D == 64 || D == 128, D, 0);
  REQUIRE(p.B >= 1 && p.H >= 1, p.B, p.H);
  REQUIRE(p.bm == rows_per_wg(1) || p.bm == rows_per_wg(2), p.bm, 0);
  REQUIRE(p.n_qseg >= 1 && p.n_qseg <= RC_MAX_SEGMENTS, p.n_qseg, 0);
  REQUIRE(p.q && p.o, 0, 0);
  REQUIRE(std::isfinite(p.scale_log2) && p.scale_log2 > 0.f, 0, 0);
  REQUIRE(p.fp8 == 0 || p.fp8 == 1, p.fp8, 0);
  REQUIRE(!p.fp8 || p.kv_scale, p.fp8, 0);
  int64_t tiles = 0, units = 0, prev_end = 0;
  bool reads[2] = {false, false};
  for (int i = 0; i < p.n_qseg; ++i) {
    const QSeg& s = p.qseg[i];
    REQUIRE(s.len >= 1 && s.row0 >= prev_end, i, s.row0);
    REQUIRE(int64_t(s.row0) + s.len <= p.n_rows, i, p.n_rows);
    prev_end = s.row0 + s.len;
    REQUIRE(s.tile0 == tiles, i, s.tile0);
    REQUIRE(s.unit0 == units, i, s.unit0);
    REQUIRE(s.r0 >= 0 && s.nr >= 0 && s.r0 + s.nr <= kMaxRanges, s.r0, s.nr);
    int64_t kt = 0;
    for (int r = s.r0; r < s.r0 + s.nr; ++r) {
      const KeyRange& k = p.range[r];
      REQUIRE(k.len >= 1 && k.start >= 0, r, k.len);
      REQUIRE(k.src == 0 || k.src == 1, r, k.src);
      REQUIRE(k.ntiles == (k.len + kBN - 1) / kBN, r, k.ntiles);
      reads[k.src] = true;
      kt += k.ntiles;
    }
    REQUIRE(kt == s.ktiles, i, kt);
    const int64_t nt = (s.len + p.bm - 1) / p.bm;
    tiles += nt;
    units += nt * s.ktiles;
  }
  REQUIRE(tiles == p.n_qtiles, tiles, p.n_qtiles);
  REQUIRE(units == p.units_bh, units, p.units_bh);
  for (int s = 0; s < 2; ++s)
    if (reads[s]) REQUIRE(p.src[s].k && p.src[s].v && p.src[s].k_st > 0 && p.src[s].v_st > 0, s, 0);
  // a tile's byte record count (64 tokens x token stride) stays below 2^32
  for (int s = 0; s < 2; ++s)
    if (reads[s]) REQUIRE(int64_t(kBN) * p.src[s].k_st <= (int64_t(1) << 32), s, p.src[s].k_st);
  if (balanced) {
    REQUIRE(p.splits == kSplitsBalanced && p.bal_wgs == kBalancedWGs, p.splits, p.bal_wgs);
    REQUIRE(p.units == int64_t(p.B) * p.H * p.units_bh, p.units, 0);
    REQUIRE(p.ws_o && p.ws_ml, 0, 0);
  } else {
    REQUIRE(p.splits >= 1 && p.splits <= kMaxSplits, p.splits, 0);
    REQUIRE(p.splits == 1 || (p.ws_o && p.ws_ml), p.splits, 0);
    REQUIRE(p.tail_num == 0 || (p.splits == 2 && p.tail_num > 0 && p.tail_num < 1024), p.tail_num, p.splits);
    REQUIRE(int64_t(p.B) * p.H <= 65535 * int64_t(65535), p.B, p.H);
  }
}

// Tiles run as two halves: the last ones of one unsplit launch, all of an even
// split or all of a last-round split, some of them with more than 256 rows,
// every half on a CU of its own.
void check_halves(const rc::Params& p) {
  using namespace rc;
  const int64_t tiles = int64_t(p.B) * p.H * p.n_qtiles;
  REQUIRE(p.half_tiles >= 0 && p.half_tiles <= tiles, p.half_tiles, tiles);
  if (p.half_tiles == 0) return;
  bool gain = false;
  for (int i = 0; i < p.n_qseg; ++i) gain = gain || p.qseg[i].len > p.bm / 2;
  REQUIRE(gain && p.bm == rows_per_wg(2), p.bm, gain);
  if (p.lr_tiles > 0) {
    REQUIRE(p.half_tiles == p.lr_tiles && 4 * p.lr_tiles <= kCUs, p.half_tiles, p.lr_tiles);
    return;
  }
  REQUIRE(p.tail_num == 0, p.tail_num, p.half_tiles);
  REQUIRE(p.splits == 1 ? !per_batch_launches(p) : p.half_tiles == tiles, p.splits, p.half_tiles);
  REQUIRE(attention_work_groups(p) + p.cp.blocks <= kCUs, attention_work_groups(p), p.cp.blocks);
}

bool aligned(const void* p, uintptr_t n) { return (reinterpret_cast<uintptr_t>(p) & (n - 1)) == 0; }

void check_copy(const rc::CopySeg* seg, int n_copy, int32_t n_cached) {
  REQUIRE(n_copy >= 1 && n_copy <= RC_MAX_SEGMENTS, n_copy, 0);
  int64_t dst = 0;
  for (int i = 0; i < n_copy; ++i) {
    REQUIRE(seg[i].len >= 1 && seg[i].src_row0 >= 0, i, seg[i].len);
    REQUIRE(seg[i].dst_row0 == dst, i, seg[i].dst_row0);
    // runs that follow each other in the source as in the cache are one
    REQUIRE(i == 0 || seg[i].src_row0 > seg[i - 1].src_row0 + seg[i - 1].len, i, seg[i].src_row0);
    dst += seg[i].len;
  }
  g_runs = n_copy;
  REQUIRE(dst == n_cached, dst, n_cached);
}

}  // namespace

namespace rc {

int launch_attention(const Params& p, int D, void*) {
  check_params(p, D, false);
  REQUIRE(p.lr_tiles >= 0 && p.lr_tiles < kCUs, p.lr_tiles, 0);
  if (p.lr_tiles > 0) {
    REQUIRE(p.splits == 2 && p.tail_num > 0 && p.cp.blocks == 0, p.splits, p.tail_num);
    REQUIRE(p.lr_tiles <= int64_t(p.B) * p.H * p.n_qtiles, p.lr_tiles, p.n_qtiles);
  }
  check_halves(p);
  REQUIRE(aligned(p.ws_o, 16) && aligned(p.ws_ml, 8), 0, 0);
  g_wgs = attention_work_groups(p);
  const CopyTail& c = p.cp;
  g_amax = c.blocks > 0 ? c.amax : nullptr;
  g_taken = g_amax ? c.rows / c.n_cached : 0;
  if (p.amax_clear) {
    REQUIRE(p.splits == 1 && !p.fp8 && !g_amax && c.blocks == 0, p.splits, c.blocks);
    REQUIRE(c.B == p.B && c.H == p.H, c.B, c.H);
    g_amax = p.amax_clear;
  }
  REQUIRE(c.blocks >= 0 && c.blocks <= kCUs, c.blocks, 0);
  if (c.blocks > 0) {
    REQUIRE(p.splits == 1 && !p.fp8, p.splits, p.fp8);
    REQUIRE(c.k_src && c.v_src, 0, 0);
    // bf16 buffers to copy into, or an amax to take and nothing to write
    REQUIRE(c.amax ? !c.k_dst && !c.v_dst : c.k_dst && c.v_dst, c.amax != nullptr, c.k_dst != nullptr);
    REQUIRE(c.B == p.B && c.H == p.H, c.B, c.H);
    REQUIRE(int64_t(c.B) * c.H * c.n_cached < (int64_t(1) << 31), c.n_cached, 0);
    REQUIRE(!c.amax || c.rows % c.n_cached == 0, c.rows, c.n_cached);
    REQUIRE(c.rows >= c.blocks && c.rows <= int64_t(c.B) * c.H * c.n_cached, c.rows, c.blocks);
    check_copy(c.seg, c.n_copy, c.n_cached);
  }
  ++g_launches;
  return 0;
}

int launch_attention_balanced(const Params& p, int D, void*) {
  check_params(p, D, true);
  g_wgs = attention_work_groups(p);
  ++g_launches;
  return 0;
}

int launch_combine_balanced(const Params& p, int D, void*) {
  check_params(p, D, true);
  ++g_launches;
  return 0;
}

int launch_combine_last_round(const Params& p, int D, void*) {
  check_params(p, D, false);
  REQUIRE(p.lr_tiles > 0 && p.splits == 2 && p.ws_o && p.ws_ml, p.lr_tiles, p.splits);
  REQUIRE(p.bm == rows_per_wg(2) && aligned(p.ws_o, 16) && aligned(p.ws_ml, 8), p.bm, 0);
  ++g_launches;
  return 0;
}

int launch_combine(const CombineParams& c, void*) {
  REQUIRE(c.ws_o && c.ws_ml && c.o, 0, 0);
  REQUIRE(c.splits >= 2 && c.splits <= kMaxSplits, c.splits, 0);
  REQUIRE(c.n_rows >= 1 && (c.D == 64 || c.D == 128), c.n_rows, c.D);
  REQUIRE(aligned(c.ws_o, 16) && aligned(c.ws_ml, 8) && aligned(c.o, 16), 0, 0);
  // every row in one block of up to 32 rows of its segment
  REQUIRE(c.n_seg >= 1 && c.n_seg <= RC_MAX_SEGMENTS, c.n_seg, 0);
  int64_t row = 0, block = 0;
  for (int i = 0; i < c.n_seg; ++i) {
    REQUIRE(c.seg[i].len >= 1 && c.seg[i].row0 == row, i, c.seg[i].row0);
    REQUIRE(c.seg[i].block0 == block, i, c.seg[i].block0);
    row += c.seg[i].len;
    block += (c.seg[i].len + 31) / 32;
  }
  REQUIRE(row == c.n_rows && block == c.n_blocks, c.n_rows, c.n_blocks);
  ++g_launches;
  return 0;
}

int launch_cache_store(const CacheStoreParams& c, void*) {
  REQUIRE(c.k_src && c.v_src && c.k_dst && c.v_dst, 0, 0);
  REQUIRE(c.total_rows == c.n_cached, c.total_rows, c.n_cached);
  REQUIRE(c.row0 >= 0 && c.row0 < int64_t(c.B) * c.H * c.n_cached, c.row0, c.n_cached);
  check_copy(c.seg, c.n_copy, c.n_cached);
  ++g_launches;
  return 0;
}

int launch_cache_store_fp8(const CacheStore8Params& c, void*) {
  REQUIRE(c.k_src && c.v_src && c.k_dst && c.v_dst && c.kv_scale, 0, 0);
  REQUIRE(c.n_cached <= kFp8MaxKeys, c.n_cached, 0);
  check_copy(c.seg, c.n_copy, c.n_cached);
  REQUIRE(c.bh0 >= 0 && c.bh0 <= c.B * c.H, c.bh0, c.B * c.H);
  // the attention launch before has cleared the accumulators and taken the first heads
  REQUIRE(g_amax == c.kv_scale && g_taken == c.bh0, g_taken, c.bh0);
  g_heads = c.bh0;
  ++g_launches;
  return 0;
}

int launch_linear(const LinearParams& q, void*) {
  REQUIRE(q.a && q.w && q.out, 0, 0);
  REQUIRE(q.M >= 1 && q.N >= 1 && q.K >= 1, q.M, q.N);
  REQUIRE(q.lda >= q.K && q.ldo >= q.N && (!q.r || q.ldr >= q.N), q.lda, q.ldo);
  // 16-byte loads and stores of whole tiles, 32-bit offsets inside 256 rows
  REQUIRE(q.N % 128 == 0 && q.K % 64 == 0, q.N, q.K);
  REQUIRE(aligned(q.a, 16) && aligned(q.w, 16) && aligned(q.r, 16) && aligned(q.out, 16), 0, 0);
  REQUIRE((q.lda | q.ldo | q.ldr) % 8 == 0 && 256 * 2 * std::max<int64_t>(q.lda, q.K) <= (int64_t(1) << 31), q.lda, q.K);
  const LinearPlan p = plan_linear(q);
  REQUIRE((p.tile >= 0) != (p.part >= 0) && p.tile < 5 && p.part < 3, p.tile, p.part);
  const int bn[] = {256, 128, 128, 128, 64};
  REQUIRE(q.N % (p.part >= 0 ? 256 : bn[p.tile]) == 0, q.N, p.tile);
  if (p.part >= 0) {
    REQUIRE(p.tiles == (q.M + 255) / 256 * (q.N / 256), p.tiles, q.M);
    REQUIRE(p.whole > 0 && p.whole % kCUs == 0 && p.whole < p.tiles, p.whole, p.tiles);
    REQUIRE((p.tiles - p.whole) * lin_parts(p.part) <= kCUs, p.tiles - p.whole, p.part);
  }
  g_linear = p.part >= 0 ? 5 + p.part : p.tile;
  ++g_launches;
  return 0;
}

// a fake, never dereferenced device address of the scratch array
int scratch_address(void** ptr) {
  *ptr = reinterpret_cast<void*>(uintptr_t(0x7f0000100000));
  ++g_launches;
  return 0;
}

}  // namespace rc

extern "C" long rc_stub_launches(void) { return g_launches; }
extern "C" long rc_stub_copy_runs() { return g_runs; }
extern "C" long rc_stub_amax_heads() { return g_heads; }
extern "C" long rc_stub_work_groups() { return g_wgs; }
extern "C" long rc_stub_linear_tile() { return g_linear; }
