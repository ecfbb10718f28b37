// Host-only test program (no GPU, no HIP): built from the library's HIP-free sources and the C oracle with
// -fsanitize=address,undefined by tests/test_host_model.py.
//
//  1. A host model of the attention kernels' key-range walk.  The kernels' tile arithmetic lives in
//     kvfold_consts.h (workgroup_rows, tile_map, key_range, dma_row) and the launch geometry in the planner;
//     both are used here exactly as the kernels use them.  For many shapes -- chunk length, cache length, group
//     size, prefix splits, units per wavefront (fp32: wavefronts per workgroup), fused append or not, plain and
//     sink + sliding-window steps, pieces that meet in the attention kernel and pieces that do not, few rows that need work on their way (rotary embedding, storage round trip), several units that rotate
//     the chunk's rows themselves -- every workgroup's pieces are walked as its kernel walks them -- the general bf16
//     kernel's ring with its run-ahead and the last tile fetched again past the end, the few-rows kernel's blocks of
//     32 keys in cyclic order, the decoding kernel's last block and its plain ones, the fp32 kernel's half tiles with their two sources -- and checked:
//       * every DMA source row lies inside what exists (cache rows below len_prev when the chunk's rows are not
//         in the cache yet, else below len_prev + C; chunk rows below C), with 32-bit offsets that do not wrap;
//       * a row that a query of the workgroup can see is fetched unclamped, from the right place;
//       * the pieces of all splits together cover every visible key of every row of the workgroup exactly once;
//       * the chunk's rows are appended exactly once: the workgroups' shares of the copy, or the rows that a few-rows
//         workgroup works on, which are all that it reads of the chunk, and none of which it fetches ahead of its work;
//       * what pieces leave for one another, and the counters they meet by, lie inside what there is;
//       * the blocks of the grid are the workgroups, each once, and the units of a piece lie on one XCD where each streams its keys for itself.
//  2. The planner and validate_config over a sweep of configurations (sanitizers watch the arithmetic).
//  3. The oracle on tiny inputs, plain and windowed (sanitizers watch its indexing).
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <thread>
#include <utility>
#include <vector>

#include "../paper_2605_12471_amd/csrc/kvfold_plan.h"

extern "C" {
int kvfold_oracle_attend_rows(const double*, const double*, int64_t, int64_t, int64_t, const double*, int64_t, int64_t,
                              int64_t, double, const int64_t*, int64_t, double*, double*, double*);
int kvfold_oracle_attend_rows_window(const double*, const double*, int64_t, int64_t, int64_t, const double*, int64_t,
                                     int64_t, int64_t, double, int64_t, int64_t, const int64_t*, int64_t, double*,
                                     double*, double*);
int kvfold_oracle_append_bytes(unsigned char*, int64_t, int64_t, int64_t, int64_t, const unsigned char*, int64_t, int64_t);
}

using namespace kvfold;

static long g_checks = 0, g_rotated = 0;  // g_rotated: steps whose readers rotate the chunk's rows
static long g_met = 0, g_two_met = 0;     // steps whose pieces meet, by the last workgroup and two by two
#define REQUIRE(cond, ...)                                   \
  do {                                                       \
    ++g_checks;                                              \
    if (!(cond)) {                                           \
      std::fprintf(stderr, "FAILED %s:%d: %s\n  ", __FILE__, __LINE__, #cond); \
      std::fprintf(stderr, __VA_ARGS__);                     \
      std::fprintf(stderr, "\n");                            \
      std::exit(1);                                          \
    }                                                        \
  } while (0)

// One row that a kernel reads for `key` (of the piece: the workgroup may need it; else it only has to exist).
struct Reader {
  const kvfold_config_t& cfg;
  int n_tokens;
  int64_t len_prev, readable_cache, last_key;
  int row_bytes;
  bool fused;
  std::vector<int>& seen;
  int64_t work_row0 = 0, work_row1 = 0;  // chunk rows in the cache that this workgroup has appended itself (readable_cache: all others)
  void read(const DmaRow& d, int64_t key, bool of_piece) {
    if (d.from_chunk) {
      REQUIRE(fused && (int64_t)d.row < n_tokens, "chunk row %u out of %d", d.row, n_tokens);
      REQUIRE((uint64_t)d.row * cfg.n_kv_heads * row_bytes + row_bytes <= (1ull << 32), "32-bit chunk offset wraps");
    } else {
      REQUIRE((int64_t)d.row < readable_cache || ((int64_t)d.row >= work_row0 && (int64_t)d.row < work_row1), "cache row %u not readable (%lld rows are)", d.row, (long long)readable_cache);
      REQUIRE((uint64_t)d.row * row_bytes + row_bytes <= (1ull << 32), "32-bit cache offset wraps");
    }
    if (of_piece && key <= last_key) {
      // inside the piece and not beyond the workgroup's last row: must be the key itself
      const int64_t got = d.from_chunk ? len_prev + d.row : d.row;
      REQUIRE(got == key, "key %lld is read from the row of key %lld", (long long)key, (long long)got);
      REQUIRE(d.from_chunk == (fused && key >= len_prev), "wrong source for key %lld", (long long)key);
      seen[(size_t)key]++;
    }
  }
};

// The general bf16 kernel: every tile of the piece row by row where it is issued as a whole (issue_tile), and the main loop's
// refills (issue_slab), which run NV + 1 tiles (K) and NV tiles (V) ahead, take every row to be a cache row, and fetch
// the last tile again past the end.
static void walk_ring(Reader& rd, const TileMap& tm, const KeyRange& kr, int nv) {
  auto tphys = [&](int t) { return t + (t >= tm.ns_t ? tm.skip : 0); };
  auto tlogical = [&](int tp) { return tp < tm.ns_t ? tp : tp - tm.skip > tm.ns_t ? tp - tm.skip : tm.ns_t; };
  for (int t = kr.t_begin; t < kr.t_end; ++t)
    for (int row = 0; row < kTileKeys; ++row) rd.read(dma_row(kr, tphys(t), row), (int64_t)tphys(t) * kTileKeys + row, true);
  const int len_after = (int)rd.len_prev + rd.n_tokens, t_new = kr.t_straddle >= 0 ? kr.t_straddle : kr.t_new;
  int t_plain = tlogical(len_after / kTileKeys < t_new ? len_after / kTileKeys : t_new);
  t_plain = t_plain >= kr.t_end ? kr.t_end : t_plain - nv - 1;
  for (int t = kr.t_begin; t < t_plain; ++t)
    for (int ahead : {nv, nv + 1}) {
      const int t_log = t + ahead < kr.t_end - 1 ? t + ahead : kr.t_end - 1, tp = tphys(t_log);
      for (int row : {0, kTileKeys - 1}) {
        const DmaRow plain{false, (unsigned)(tp * kTileKeys + row)}, is = dma_row(kr, tp, row);
        rd.read(plain, -1, false);
        REQUIRE(is.from_chunk == plain.from_chunk && is.row == plain.row, "refill of tile %d (tile %d) is not plain", t_log, t);
      }
    }
}

// The few-rows kernel: each of its 4 or 8 wavefronts takes every 4th or 8th block of 32 keys, in cyclic order from a place of its own.
// work: the workgroup appends the rows of the chunk that its piece holds, after the first block's fetch where that needs none of them.
static void walk_few(Reader& rd, const TileMap& tm, const KeyRange& kr, int nw, int64_t nkeys, int split, int g, bool work, std::vector<int>& appended) {
  int work_r0 = 0, work_r1 = 0;
  if (work && kr.t_begin < kr.t_end) {
    work_r0 = kr.t_begin * kTileKeys - (int)rd.len_prev;
    if (work_r0 < 0) work_r0 = 0;
    work_r1 = (int)kr.row_lim + 1 - (int)rd.len_prev;
  }
  REQUIRE(work_r1 <= rd.n_tokens, "work on row %d of %d", work_r1 - 1, rd.n_tokens);
  for (int r = work_r0; r < work_r1; ++r) appended[(size_t)r]++;
  auto first_key = [&](int b) { return b * 32 + ((b >> 1) >= tm.ns_t ? tm.skip * kTileKeys : 0); };
  const int b_all = 2 * tm.ntiles - (first_key(2 * tm.ntiles - 1) >= nkeys ? 1 : 0), b_end = 2 * kr.t_end < b_all ? 2 * kr.t_end : b_all;
  for (int w = 0; w < nw; ++w) {
    const int b_first = 2 * kr.t_begin + w, n_blocks = b_first < b_end ? (b_end - b_first + nw - 1) / nw : 0;
    int b = b_first + nw * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_blocks) >> 16);
    for (int i = 0; i < n_blocks; ++i) {
      REQUIRE(b >= b_first && b < b_end && (b - b_first) % nw == 0, "block %d of [%d, %d), wavefront %d", b, b_first, b_end, w);
      const bool ahead = i == 0 && (work_r1 <= work_r0 || b * 32 + 32 <= (int)rd.len_prev);  // fetched before the work
      rd.work_row0 = ahead ? 0 : rd.len_prev + work_r0;
      rd.work_row1 = ahead ? 0 : rd.len_prev + work_r1;
      const unsigned first = (unsigned)first_key(b), last = first + 31;
      const bool plain = last <= kr.row_lim && (last < kr.chunk_row0 || first >= kr.chunk_row0), nw_rows = first >= kr.chunk_row0;
      for (unsigned row = 0; row < 32; ++row)
        rd.read(plain ? DmaRow{nw_rows, first + row - (nw_rows ? kr.chunk_row0 : 0u)} : dma_row(kr, (int)first / kTileKeys, (int)first % kTileKeys + (int)row),
                (int64_t)first + row, true);
      b = b + nw < b_end ? b + nw : b_first;
    }
  }
}

// The kernel whose keys come straight into registers: each of four wavefronts takes every 4th block of 32 keys.  Its last block, if it has rows past the piece's last
// or of the chunk, comes first, each row from its own place; all others are asked for as they lie in the cache, in cyclic order from a place of its
// own.  work: the workgroup appends the chunk's rows of its piece ahead of every fetch.
static void walk_decode(Reader& rd, const TileMap& tm, const KeyRange& kr, int split, int g, bool work, std::vector<int>& appended) {
  constexpr int nw = 4;
  const int vis_last = (int)rd.len_prev + rd.n_tokens;
  REQUIRE(tm.ns_t == 0 && tm.skip == 0 && tm.ntiles == (vis_last + kTileKeys - 1) / kTileKeys && (int64_t)vis_last == rd.last_key + 1, "keys of the unit");
  int work_r0 = 0, work_r1 = 0;
  if (work && kr.t_begin < kr.t_end) {
    work_r0 = kr.t_begin * kTileKeys - (int)rd.len_prev;
    if (work_r0 < 0) work_r0 = 0;
    work_r1 = (int)kr.row_lim + 1 - (int)rd.len_prev;
  }
  REQUIRE(work_r1 <= rd.n_tokens, "work on row %d of %d", work_r1 - 1, rd.n_tokens);
  for (int r = work_r0; r < work_r1; ++r) appended[(size_t)r]++;
  rd.work_row0 = rd.len_prev + work_r0;
  rd.work_row1 = rd.len_prev + work_r1;
  const int b_all = (vis_last + 31) / 32, b_end = 2 * kr.t_end < b_all ? 2 * kr.t_end : b_all;
  for (int w = 0; w < nw; ++w) {
    const int b_first = 2 * kr.t_begin + w, n_blocks = b_first < b_end ? (b_end - b_first + nw - 1) / nw : 0;
    if (n_blocks == 0) continue;
    const int b_last = b_first + nw * (n_blocks - 1);
    const bool special = (unsigned)b_last * 32u + 31u > kr.row_lim || (unsigned)b_last * 32u + 31u >= kr.chunk_row0;
    const int n_plain = n_blocks - (special ? 1 : 0), b_plain = b_first + nw * n_plain;
    int b = b_first + nw * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_plain) >> 16);
    if (special)
      for (int row = 0; row < 32; ++row) rd.read(dma_row(kr, 0, b_last * 32 + row), (int64_t)b_last * 32 + row, true);
    for (int i = 0; i < n_plain; ++i) {
      REQUIRE(b >= b_first && b < b_plain && (b - b_first) % nw == 0, "block %d of [%d, %d), wavefront %d", b, b_first, b_plain, w);
      REQUIRE((unsigned)b * 32u + 31u <= kr.row_lim && (unsigned)b * 32u + 31u < kr.chunk_row0, "block %d is not plain", b);
      for (unsigned row = 0; row < 32; ++row) rd.read(DmaRow{false, (unsigned)b * 32u + row}, (int64_t)b * 32 + row, true);
      b = b + nw < b_plain ? b + nw : b_first;
    }
  }
}

// The fp32 kernel: half tiles, rows past the last one read as the last one; a last half beyond every row is left out.  Fused: the
// first half and those of the second loop take each row from its own side, those of the first loop, which ends before the
// first half that is not all cache, are cache rows.
static void walk_halves(Reader& rd, const TileMap& tm, const KeyRange& kr, int64_t nkeys_wg) {
  const int64_t len_after = rd.len_prev + rd.n_tokens, chunk0 = rd.fused ? rd.len_prev : (int64_t)1 << 40;
  auto first_key = [&](int h) { const int t = h >> 1; return (2 * (int64_t)(t + (t >= tm.ns_t ? tm.skip : 0)) + (h & 1)) * 32; };
  auto is_old = [&](int h) { return first_key(h) + 32 <= chunk0; };
  const int h_begin = 2 * kr.t_begin;
  int h_end = 2 * kr.t_end;
  if (h_end > h_begin && first_key(h_end - 1) >= nkeys_wg) --h_end;
  auto fetch = [&](int h, bool old) {
    for (int i = 0; i < 32; ++i) {
      const int64_t key = first_key(h) + i, row = key < len_after ? key : len_after - 1;
      const bool from_chunk = !old && row >= chunk0;
      rd.read(DmaRow{from_chunk, (unsigned)(from_chunk ? row - chunk0 : row)}, key, true);
    }
  };
  if (h_begin < h_end) fetch(h_begin, false);
  int h = h_begin;
  for (; h < h_end && is_old(h + 1 < h_end ? h + 1 : h); ++h)
    if (h + 1 < h_end) fetch(h + 1, true);
  for (; h < h_end; ++h)
    if (h + 1 < h_end) fetch(h + 1, false);
}

// The fp32 kernel of that kind: blocks in the same order, rows past the last one read as the last one; a block whose rows all exist and lie
// on one side of the old cache's end is read from one base.  (After its last block a wavefront fetches that one once more.)
static void walk_few_f32(Reader& rd, const TileMap& tm, const KeyRange& kr, int nw, int64_t nkeys, int split, int g) {
  const int64_t len_after = rd.len_prev + rd.n_tokens, chunk0 = rd.fused ? rd.len_prev : (int64_t)1 << 40;
  auto first_key = [&](int b) { return (int64_t)b * 32 + ((b >> 1) >= tm.ns_t ? tm.skip * kTileKeys : 0); };
  const int b_all = 2 * tm.ntiles - (first_key(2 * tm.ntiles - 1) >= nkeys ? 1 : 0), b_end = 2 * kr.t_end < b_all ? 2 * kr.t_end : b_all;
  for (int w = 0; w < nw; ++w) {
    const int b_first = 2 * kr.t_begin + w, n_blocks = b_first < b_end ? (b_end - b_first + nw - 1) / nw : 0;
    int b = b_first + nw * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_blocks) >> 16);
    for (int i = 0; i < n_blocks; ++i) {
      REQUIRE(b >= b_first && b < b_end && (b - b_first) % nw == 0, "block %d of [%d, %d), wavefront %d", b, b_first, b_end, w);
      const int64_t first = first_key(b), last = first + 31;
      const bool plain = last < len_after && (last < chunk0 || first >= chunk0), nw_rows = first >= chunk0;
      for (int j = 0; j < 32; ++j) {
        const int64_t key = first + j, row = key < len_after ? key : len_after - 1;
        const bool from_chunk = plain ? nw_rows : row >= chunk0;
        rd.read(DmaRow{from_chunk, (unsigned)((plain ? key : row) - (from_chunk ? chunk0 : 0))}, key, true);
      }
      b = b + nw < b_end ? b + nw : b_first;
    }
  }
}

// Where the pieces of a step leave their results and how they meet: all of it inside what a cache (or the static array) has.
static void check_pieces(const PlanCtx& pc, const Plan& pl, int n_tokens) {
  const kvfold_config_t& cfg = pc.cfg;
  const bool two = two_pieces_meet(pc, pl, pl.n_splits), meet = pieces_meet(pc, pl, n_tokens, pl.n_splits);
  if (pl.n_splits == 1) REQUIRE(!two && !meet, "one piece meets nobody");
  REQUIRE(!(two && meet), "merged twice");
  if (!pc.two_meet) REQUIRE(!two && !meet, "no counters");
  const int64_t d4 = cfg.head_dim * 4;
  if (meet) {  // [piece][token][query head] rows of O, and (m, l); a counter per KV head and number of pieces
    ++g_met;
    const int64_t rows = (int64_t)n_tokens * cfg.n_q_heads;
    REQUIRE(pl.direct && pl.n_splits <= kMaxSplits, "which kernel");
    REQUIRE(pl.n_splits * rows <= pc.ws_rows && pl.n_splits * rows * d4 < ((int64_t)1 << 32), "partial results");
    REQUIRE(pl.n_splits < kMeetStride && (int64_t)(cfg.n_kv_heads - 1) * kMeetStride + pl.n_splits < (int64_t)kMeetUnits * kMeetStride, "counter");
    // a wavefront's lanes hold a row, or two, and every piece of it
    const int per_wave = (int)((n_tokens * (cfg.n_q_heads / cfg.n_kv_heads) + 3) / 4);
    REQUIRE(per_wave <= 2 && pl.n_splits <= (per_wave == 2 && cfg.head_dim == 128 ? kMeetSplitsFew : kMeetSplits), "rows and pieces of the last workgroup");
  }
  if (two) {  // a wavefront's registers as they lie: 32 rows of O a unit, and 64 lanes' (m, l)
    ++g_two_met;
    const int64_t waves = (int64_t)cfg.n_kv_heads * pl.wgs_per_head * kUnitsPerWg, units = 2 * waves * pl.units_per_wave;
    REQUIRE(!pl.key_waves && waves <= kMergeCounters, "counter");
    REQUIRE(units * (cfg.head_dim / 32) * 4096 <= pc.ws_rows * d4 && units * 512 <= pc.ws_rows * 8, "partial results");
    REQUIRE(units * (cfg.head_dim / 32) * 4096 < ((int64_t)1 << 32), "32-bit offset of a partial result");
  }
}

static void walk_plan(const PlanCtx& pc, const Plan& pl, int n_tokens, int64_t len_prev, int n_sink, int64_t window, bool rope);

// As the cache would plan it, and where that makes a difference without counters and from the static array.
static void walk_step(const kvfold_config_t& cfg, int n_cu, int n_tokens, int64_t len_prev, int n_sink, int64_t window,
                      int force_splits, int force_upw, bool rope = false, int storage_bits = 0) {
  PlanCtx pc{};
  pc.cfg = cfg;
  pc.ws_rows = workspace_rows(&cfg);
  pc.n_cu = n_cu;
  pc.tune_splits = force_splits;
  pc.tune_units_per_wave = force_upw;
  pc.storage_bits = storage_bits;
  pc.two_meet = cfg.dtype == KVFOLD_BF16 && pc.ws_rows > 0;
  const Plan pl = make_plan(pc, n_tokens, len_prev + n_tokens, n_sink, window);
  walk_plan(pc, pl, n_tokens, len_prev, n_sink, window, rope);
  auto same = [&](const Plan& o) {
    return o.direct == pl.direct && o.key_waves == pl.key_waves && o.units_per_wave == pl.units_per_wave && o.waves_per_wg == pl.waves_per_wg &&
           o.n_splits == pl.n_splits && o.tiles_per_split == pl.tiles_per_split && o.pair_units == pl.pair_units && o.pair_order == pl.pair_order;
  };
  for (int other = 0; other < 2; ++other) {
    PlanCtx po = pc;
    if (other == 0)
      po.two_meet = false;
    else
      po.ws_rows = kStaticScratchRows;
    if (po.ws_rows < (int64_t)2 * n_tokens * cfg.n_q_heads || (other == 1 && (window > 0 || rope || storage_bits))) continue;
    const Plan o = make_plan(po, n_tokens, len_prev + n_tokens, n_sink, window);
    check_pieces(po, o, n_tokens);
    if (!same(o)) walk_plan(po, o, n_tokens, len_prev, n_sink, window, rope);
  }
}

static void walk_plan(const PlanCtx& pc, const Plan& pl, int n_tokens, int64_t len_prev, int n_sink, int64_t window, bool rope) {
  const kvfold_config_t& cfg = pc.cfg;
  const int64_t len_after = len_prev + n_tokens;
  const int storage_bits = pc.storage_bits, n_cu = pc.n_cu;
  check_pieces(pc, pl, n_tokens);
  const bool fused = attention_appends(pc, pl, n_tokens, rope), work = attention_works_on_rows(pc, pl, n_tokens, rope);
  REQUIRE(!(fused && work), "appended twice");
  const bool rotates = rope && fused;  // several units read the chunk's rows as handed in, and rotate what they read and append
  REQUIRE(cfg.dtype != KVFOLD_BF16 || rotates || fused == fused_append_applies(pc, n_tokens, len_prev, rope), "what kvfold_plan_t reports");
  REQUIRE(!rotates || (cfg.dtype == KVFOLD_BF16 && pl.key_waves && pl.units_per_head > 1 && window <= 0 && storage_bits == 0), "rows rotated by their readers");
  if (rotates) ++g_rotated;
  const int G = cfg.n_q_heads / cfg.n_kv_heads;
  const int upw_wg = pl.key_waves ? 1 : pl.waves_per_wg * pl.units_per_wave;
  const int row_bytes = cfg.head_dim * elem_size(cfg.dtype);
  REQUIRE(pl.n_splits >= 1 && pl.n_splits <= kMaxSplits && pl.tiles_per_split >= 1, "plan");
  REQUIRE(pl.n_splits == 1 || (int64_t)pl.n_splits * n_tokens * cfg.n_q_heads <= pc.ws_rows, "workspace");
  REQUIRE(pl.n_wgs == cfg.n_kv_heads * pl.wgs_per_head * pl.n_splits, "grid");
  if (window > 0) REQUIRE(!pl.pair_units && !pl.pair_order, "pairing under a window");
  REQUIRE(pl.waves_per_wg == kUnitsPerWg || (pl.waves_per_wg == 8 && cfg.dtype == KVFOLD_F32 && pl.units_per_wave == 1), "wavefronts");
  REQUIRE(!pl.few_rows || (cfg.dtype == KVFOLD_BF16 && window <= 0 && pl.units_per_head == 1 && pl.wgs_per_head == 1), "few rows");
  REQUIRE(!pl.direct || (pl.few_rows && n_tokens * G <= (cfg.head_dim == 64 ? 32 : 16)), "keys straight into registers");
  REQUIRE(pl.key_waves == 0 || pl.key_waves == 8 || (pl.key_waves == 4 && (window <= 0 || cfg.dtype == KVFOLD_F32)), "wavefronts that share a unit's keys");
  REQUIRE(pl.key_waves == 0 || cfg.dtype == KVFOLD_BF16 || pl.key_waves == (cfg.head_dim == 64 ? 8 : 4), "fp32 wavefronts");
  REQUIRE(pl.key_waves == 0 || (pl.wgs_per_head == pl.units_per_head && !pl.pair_units && !pl.pair_order), "one unit a workgroup");
  REQUIRE(!work || (pl.key_waves == 4 && pl.units_per_head == 1), "rows are worked on by the one workgroup of a piece");
  REQUIRE((int64_t)pl.wgs_per_head * upw_wg >= pl.units_per_head && (int64_t)pl.units_per_head * kRowsPerUnit >= (int64_t)n_tokens * G,
          "%d workgroups of %d units for %d tokens x %d heads", pl.wgs_per_head, upw_wg, n_tokens, G);

  // the grid: every workgroup is one block's, and where the keys of one unit are dealt to wavefronts the units of a piece share an XCD (but for
  // a piece that the end of an XCD's run cuts)
  {
    const int per_kvh = pl.wgs_per_head * pl.n_splits, grid = padded_grid(pl.n_wgs);
    const int lk = xcd_share_log2(cfg.n_kv_heads, pl.wgs_per_head, pl.n_splits, pl.key_waves > 0);
    std::vector<int> blocks((size_t)pl.n_wgs);
    std::set<std::pair<int, int>> piece_on_xcd;
    for (int b = 0; b < grid; ++b) {
      const int lid = logical_id((unsigned)b, (unsigned)grid, (unsigned)per_kvh, lk);
      REQUIRE(lid >= 0, "workgroup of block %d", b);
      if (lid >= pl.n_wgs) continue;
      blocks[(size_t)lid]++;
      piece_on_xcd.insert({lid / pl.wgs_per_head, b % kNumXcd});
    }
    for (int i = 0; i < pl.n_wgs; ++i) REQUIRE(blocks[(size_t)i] == 1, "workgroup %d has %d blocks", i, blocks[(size_t)i]);
    if (pl.key_waves && pl.n_splits > 1)
      REQUIRE((int)piece_on_xcd.size() <= cfg.n_kv_heads * pl.n_splits + kNumXcd - 1, "%d pieces on %d XCDs together", cfg.n_kv_heads * pl.n_splits, (int)piece_on_xcd.size());
  }

  // the chunk's rows, one KV head: its workgroups' shares of the copy
  std::vector<int> appended((size_t)n_tokens);
  if (fused) {
    const int per_kvh = pl.wgs_per_head * pl.n_splits, copy_rows = (n_tokens + per_kvh - 1) / per_kvh;
    for (int rem = 0; rem < per_kvh; ++rem)
      for (int r = rem * copy_rows; r < (rem + 1) * copy_rows && r < n_tokens; ++r) {
        REQUIRE((uint64_t)r * cfg.n_kv_heads * row_bytes + row_bytes <= (1ull << 32), "32-bit chunk offset wraps");
        REQUIRE((uint64_t)(len_prev + r) * row_bytes + row_bytes <= (1ull << 32), "32-bit cache offset wraps");
        appended[(size_t)r]++;
      }
  }
  std::vector<int> seen((size_t)len_after);
  for (int ug = 0; ug < pl.wgs_per_head; ++ug) {
    RowRange rr;
    if (pl.pair_units) {  // an early and a late unit per wavefront: the workgroup's keys run up to the late unit's rows
      rr.row_lo = 0;
      int ulast = pl.units_per_head - 1 - ug * kUnitsPerWg;
      if (ulast < 0) ulast = 0;
      rr.row_hi = unit_last_token(ulast, G, n_tokens);
    } else {
      rr = workgroup_rows(ug, upw_wg, pl.units_per_head, G, n_tokens);
    }
    const TileMap tm = tile_map(len_prev, rr.row_lo, rr.row_hi, n_sink, window);
    REQUIRE(tm.ntiles >= 1 && tm.skip >= 0 && tm.ns_t >= 0, "tile map");
    REQUIRE((int64_t)pl.n_splits * pl.tiles_per_split >= tm.ntiles, "pieces do not cover the workgroup's %d tiles (%d x %d)",
            tm.ntiles, pl.n_splits, pl.tiles_per_split);
    std::fill(seen.begin(), seen.end(), 0);
    for (int split = 0; split < pl.n_splits; ++split) {
      const KeyRange kr = key_range(tm, split, pl.tiles_per_split, len_prev, n_tokens, fused);
      if (kr.t_begin >= kr.t_end) continue;  // an empty piece touches nothing
      // (a piece that never reads the chunk as handed in ends below len_prev, so the clamp keeps it there too)
      const int64_t readable_cache = fused || work ? len_prev : len_after;
      REQUIRE((int64_t)kr.row_lim < len_after, "row_lim");
      Reader rd{cfg, n_tokens, len_prev, readable_cache, len_prev + rr.row_hi, row_bytes, fused, seen};
      if (cfg.dtype != KVFOLD_BF16 && pl.key_waves)
        walk_few_f32(rd, tm, kr, pl.key_waves, len_prev + rr.row_hi + 1, split, (split * 5 + ug) % cfg.n_kv_heads);
      else if (cfg.dtype != KVFOLD_BF16)
        walk_halves(rd, tm, kr, len_prev + rr.row_hi + 1);
      else if (pl.direct)
        walk_decode(rd, tm, kr, split, (split * 5 + ug) % cfg.n_kv_heads, work, appended);
      else if (pl.key_waves)
        walk_few(rd, tm, kr, pl.key_waves, len_prev + rr.row_hi + 1, split, (split * 5 + ug) % cfg.n_kv_heads, work, appended);
      else
        walk_ring(rd, tm, kr, ring_slots(cfg.head_dim, pl.units_per_wave, pl.n_wgs, n_cu));
    }
    // every key some row of the workgroup can see was fetched exactly once
    for (int r = rr.row_lo; r <= rr.row_hi; ++r) {
      const int64_t p = len_prev + r;
      for (int64_t j = 0; j <= p; ++j) {
        const bool vis = window <= 0 || j < n_sink || j > p - window;
        if (vis) REQUIRE(seen[(size_t)j] == 1, "key %lld visible to row %d fetched %d times (ug %d)", (long long)j, r, seen[(size_t)j], ug);
      }
    }
    for (int64_t j = 0; j < len_after; ++j) REQUIRE(seen[(size_t)j] <= 1, "key %lld fetched twice", (long long)j);
  }
  if (fused || work)  // (few rows: one workgroup per piece, so that the walk above has been through all)
    for (int r = 0; r < n_tokens; ++r) REQUIRE(appended[(size_t)r] == 1, "row %d appended %d times", r, appended[(size_t)r]);
}

static kvfold_config_t make_cfg(int Hq, int Hkv, int d, int C, int64_t cap, int dtype) {
  kvfold_config_t c{};
  c.struct_size = sizeof(c);
  c.n_layers = 1;
  c.n_q_heads = Hq;
  c.n_kv_heads = Hkv;
  c.head_dim = d;
  c.chunk_tokens = C;
  c.capacity_tokens = cap;
  c.dtype = dtype;
  return c;
}

static void model_sweep() {
  const int heads[][2] = {{4, 1}, {7, 1}, {6, 3}, {32, 8}, {2, 2}, {40, 1}};
  const int chunks[] = {1, 5, 16, 33, 64, 100, 256, 1000};
  const int64_t prefixes[] = {0, 63, 64, 500, 1024, 5000};
  const int64_t windows[][2] = {{0, 0}, {4, 1020}, {0, 1}, {4, 1}, {1, 33}, {70, 50}, {130, 129}, {0, 1 << 20}};
  long steps = 0;
  for (int d : {128, 64})
    for (auto& h : heads)
      for (int C : chunks)
        for (int64_t Lp : prefixes)
          for (auto& w : windows)
            for (int dtype : {(int)KVFOLD_BF16, (int)KVFOLD_F32}) {
              kvfold_config_t cfg = make_cfg(h[0], h[1], d, C, Lp + C, dtype);
              REQUIRE(validate_config(&cfg) == KVFOLD_OK, "config");
              for (int splits : {0, 2, 5})
                for (int upw : {0, 1, 2}) {
                  if (splits > 0 && (int64_t)splits * C * h[0] > workspace_rows(&cfg)) continue;
                  // (the widths differ in the plan's own choice, and in the kernel for 17 to 32 rows)
                  if (d == 64 && (upw > 0 || (splits > 0 && units_of_head(C, h[0] / h[1]) > 1))) continue;
                  walk_step(cfg, 256, C, Lp, (int)w[0], w[1], splits, upw);
                  ++steps;
                  // rows with work on their way: few rows of bf16, several units with the rotary embedding alone, and fp32 behind the append kernel
                  const bool few = dtype == KVFOLD_BF16 && units_of_head(C, h[0] / h[1]) == 1;
                  for (int work : {1, 2, 3}) {
                    if (w[1] > 0 || !(few || work == 1)) continue;
                    walk_step(cfg, 256, C, Lp, (int)w[0], w[1], splits, upw, (work & 1) != 0, work & 2 ? 8 : 0);
                    ++steps;
                  }
                }
            }
  // decoding: every place of the chunk's rows in their blocks and tiles
  for (int d : {128, 64})
    for (auto& h : {std::pair<int, int>{4, 1}, {2, 2}, {9, 1}})
      for (int C : {1, 2, 4, 7})
        for (int64_t Lp = 0; Lp < 200; ++Lp)
          for (int splits : {0, 1, 3})
            for (int work : {0, 1, 2}) {
              kvfold_config_t cfg = make_cfg(h.first, h.second, d, C, Lp + C, KVFOLD_BF16);
              if (splits > 0 && (int64_t)splits * C * h.first > workspace_rows(&cfg)) continue;
              walk_step(cfg, 256, C, Lp, 0, 0, splits, 0, work == 1, work == 2 ? 4 : 0);
              ++steps;
            }
  REQUIRE(g_met >= 200 && g_two_met >= 200, "%ld and %ld steps meet", g_met, g_two_met);
  REQUIRE(g_rotated >= 50, "%ld steps rotate the chunk's rows where they are read", g_rotated);
  // the benchmark's shapes at their real sizes, plain and with the streaming baseline's window
  struct { int Hq, Hkv, C; int64_t Lp; } big[] = {{32, 8, 2048, 14336}, {32, 8, 256, 130816}, {32, 8, 4096, 126976},
                                                 {28, 4, 128, 65408}, {28, 4, 8192, 57344}, {32, 8, 16, 131056}, {32, 8, 1, 131071}, {32, 8, 1, 4187},
                                                 {16, 2, 1, 90509}, {16, 1, 1, 60001}, {32, 8, 2, 30000}, {64, 32, 4, 9001}, {32, 8, 37, 32768}};
  for (auto& b : big)
    for (auto& w : {std::pair<int, int64_t>{0, 0}, {4, 1020}}) {
      kvfold_config_t cfg = make_cfg(b.Hq, b.Hkv, 128, b.C, b.Lp + b.C, KVFOLD_BF16);
      walk_step(cfg, 256, b.C, b.Lp, w.first, w.second, 0, 0);
      ++steps;
    }
  std::printf("host model: %ld steps walked\n", steps);
}

static void planner_sweep() {
  long n = 0;
  for (int Hkv : {1, 2, 4, 8, 64, 32767})
    for (int G : {1, 4, 7})
      for (int d : {64, 128})
        for (int64_t cap : {(int64_t)1, (int64_t)4096, (int64_t)131072, (int64_t)1 << 24, (int64_t)1 << 30})
          for (int C : {1, 64, 4096, 1 << 20})
            for (int dtype : {(int)KVFOLD_F32, (int)KVFOLD_BF16, 7}) {
              kvfold_config_t cfg = make_cfg(Hkv * G, Hkv, d, C, cap, dtype);
              const int rc = validate_config(&cfg);
              if (rc != KVFOLD_OK) {
                REQUIRE(kvfold_cache_bytes_required(&cfg) == 0, "bytes of an invalid config");
                continue;
              }
              REQUIRE(kvfold_cache_bytes_required(&cfg) == (size_t)2 * Hkv * cap * d * elem_size(dtype), "bytes");
              for (int64_t len_after : {(int64_t)C, cap})
                for (auto& w : {std::pair<int, int64_t>{0, 0}, {4, 1020}, {1 << 20, (int64_t)1 << 30}}) {
                  if (len_after < C || len_after > cap) continue;
                  kvfold_plan_t out;
                  const int prc = kvfold_plan_for(&cfg, 256, C, len_after, w.first, w.second, &out);
                  REQUIRE(prc == KVFOLD_OK, "plan_for rc %d", prc);
                  REQUIRE(out.n_workgroups >= 1 && out.n_splits >= 1 && out.tiles_per_split >= 1, "plan_for values");
                  REQUIRE((int64_t)out.n_splits * out.tiles_per_split * kTileKeys >= (w.second ? 1 : len_after), "plan_for tiles");
                  ++n;
                }
            }
  std::printf("planner: %ld plans\n", n);
}

// One query head per KV head: each of eight wavefronts would load the rotary angles of 32 tokens (13.0 us before, 14.7 with eight, and the like).
static void plans_of_single_heads() {
  struct { int heads, n; int64_t len_prev; } slow[] = {{8, 38, 152}, {8, 36, 102}, {8, 40, 391}};
  for (auto& t : slow) {
    PlanCtx pc{};
    pc.cfg = make_cfg(t.heads, t.heads, 128, 256, 131072, KVFOLD_BF16);
    pc.ws_rows = workspace_rows(&pc.cfg);
    pc.n_cu = 256;
    REQUIRE(make_plan(pc, t.n, t.len_prev + t.n, 0, 0).key_waves != 8, "%d tokens on %lld keys", t.n, (long long)t.len_prev);
  }
}

// Few rows 128 wide: long ranges of one or two KV heads belong to the kernel that fetches through LDS (us, it / keys straight into registers).
static void plans_of_few_rows() {
  struct { int Hq, Hkv, d, n; int64_t len_prev; bool direct; } steps[] = {
    {16, 2, 128, 1, 32625, false},   // 14.7 / 15.3
    {8, 2, 128, 1, 47946, false},    // 17.7 / 19.1
    {2, 2, 128, 1, 71723, false},    // 22.4 / 24.9
    {2, 2, 128, 16, 109066, false},  // 31.4 / 33.7
    {16, 1, 128, 1, 103038, false},  // 25.2 / 27.1
    {4, 1, 128, 1, 118893, false},   // 27.4 / 29.6
    {16, 2, 128, 1, 28572, true},    // 14.65 / 13.1
    {8, 2, 128, 1, 20021, true},     // 13.0 / 12.2
    {1, 1, 128, 1, 32576, true},     // 13.35 / 12.9
    {3, 3, 128, 1, 64336, true},     // 24.8 / 24.2
    {32, 8, 128, 1, 130941, true}, {2, 2, 64, 1, 109066, true}, {4, 1, 64, 8, 118893, true}, {17, 1, 128, 1, 1000, false}};
  for (auto& t : steps) {
    PlanCtx pc{};
    pc.cfg = make_cfg(t.Hq, t.Hkv, t.d, 256, 131072, KVFOLD_BF16);
    pc.ws_rows = workspace_rows(&pc.cfg);
    pc.n_cu = 256;
    pc.two_meet = true;
    const Plan pl = make_plan(pc, t.n, t.len_prev + t.n, 0, 0);
    REQUIRE(pl.few_rows && pl.direct == t.direct, "%d tokens on %lld keys, %d heads on %d", t.n, (long long)t.len_prev, t.Hq, t.Hkv);
  }
}

// 64 wide the one-unit kernel keeps two ring slots where it is alone on its CUs (14.7 us, 15.5 with three, and the like); the model walks with the
// launcher's depth.
static void ring_depths() {
  struct { int Hq, Hkv, d, n; int64_t len_prev; int slots; } steps[] = {
    {32, 8, 64, 551, 66, 2}, {28, 4, 64, 379, 3639, 2}, {32, 8, 64, 3570, 30, 2}, {32, 8, 128, 37, 32768, 3}, {28, 4, 128, 128, 32768, 3}, {32, 8, 128, 2048, 0, 2}};
  for (auto& t : steps) {
    PlanCtx pc{};
    pc.cfg = make_cfg(t.Hq, t.Hkv, t.d, 4096, 131072, KVFOLD_BF16);
    pc.ws_rows = workspace_rows(&pc.cfg);
    pc.n_cu = 256;
    pc.two_meet = true;
    const Plan pl = make_plan(pc, t.n, t.len_prev + t.n, 0, 0);
    REQUIRE(!pl.key_waves && pl.units_per_wave == 1 && ring_slots(t.d, 1, pl.n_wgs, 256) == t.slots, "%d tokens on %lld keys", t.n, (long long)t.len_prev);
  }
}

// No slot is in two hands, all are handed out before there is none, and one that was given back goes out again.
static void counter_slots() {
  CounterSlots slots;
  std::set<int> held;
  for (int i = 0; i < CounterSlots::kCount; ++i) {
    const int s = slots.take();
    REQUIRE(s >= 0 && s < CounterSlots::kCount && held.insert(s).second, "slot %d", s);
  }
  REQUIRE(slots.take() == -1, "none is free");
  for (int s : {17, 63, 0}) slots.give(s);
  for (int want : {0, 17, 63}) REQUIRE(slots.take() == want, "slot %d again", want);
  REQUIRE(slots.take() == -1, "none is free");
  for (int s = 0; s < CounterSlots::kCount; ++s) slots.give(s);
  std::vector<int> in_use(CounterSlots::kCount);
  std::vector<std::thread> threads;
  std::mutex m;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t]() {
      for (int i = 0; i < 2000; ++i) {
        const int s = slots.take();
        {
          std::lock_guard<std::mutex> lock(m);
          REQUIRE(s >= 0 && in_use[(size_t)s]++ == 0, "slot %d of thread %d", s, t);
        }
        {
          std::lock_guard<std::mutex> lock(m);
          --in_use[(size_t)s];
        }
        slots.give(s);
      }
    });
  for (auto& t : threads) t.join();
  REQUIRE(slots.taken == 0, "all given back");
}

static void oracle_tiny() {
  const int64_t Hq = 4, Hkv = 2, d = 8, cap = 40, C = 9, len_prev = 31;
  std::vector<double> K((size_t)Hkv * cap * d), V(K.size()), q((size_t)C * Hq * d);
  unsigned s = 12345;
  auto rnd = [&]() { s = s * 1664525u + 1013904223u; return (double)(s >> 8) / (1 << 24) - 0.5; };
  for (auto& x : K) x = rnd();
  for (auto& x : V) x = rnd();
  for (auto& x : q) x = rnd();
  std::vector<int64_t> rows = {0, 3, 8};
  std::vector<double> out(rows.size() * Hq * d), lse(rows.size() * Hq), w(rows.size() * Hq * (len_prev + C));
  REQUIRE(kvfold_oracle_attend_rows(K.data(), V.data(), Hkv, cap, d, q.data(), C, Hq, len_prev, 0.35, rows.data(),
                                    (int64_t)rows.size(), out.data(), lse.data(), w.data()) == 0, "oracle plain");
  std::vector<double> out2(out.size()), lse2(lse.size()), w2(w.size());
  REQUIRE(kvfold_oracle_attend_rows_window(K.data(), V.data(), Hkv, cap, d, q.data(), C, Hq, len_prev, 0.35, 0, 1000,
                                           rows.data(), (int64_t)rows.size(), out2.data(), lse2.data(), w2.data()) == 0, "oracle window");
  REQUIRE(std::memcmp(out.data(), out2.data(), out.size() * sizeof(double)) == 0, "an all-covering window is the plain step");
  REQUIRE(kvfold_oracle_attend_rows_window(K.data(), V.data(), Hkv, cap, d, q.data(), C, Hq, len_prev, 0.35, 2, 5,
                                           rows.data(), (int64_t)rows.size(), out2.data(), lse2.data(), w2.data()) == 0, "oracle window");
  for (size_t r = 0; r < rows.size(); ++r)
    for (int64_t h = 0; h < Hq; ++h) {
      int nz = 0;
      for (int64_t j = 0; j < len_prev + C; ++j) nz += w2[(r * Hq + h) * (len_prev + C) + j] > 0;
      REQUIRE(nz == 7, "2 sinks + 5 recent keys carry weight, got %d", nz);
    }
  REQUIRE(kvfold_oracle_attend_rows(K.data(), V.data(), Hkv, cap, d, q.data(), C, Hq, 32, 0.35, rows.data(), 3, out.data(),
                                    lse.data(), nullptr) == -1, "beyond capacity");
  // append: bytes land head-major at rows [len, len + C)
  std::vector<unsigned char> cache((size_t)Hkv * cap * d * 2, 0), chunk((size_t)C * Hkv * d * 2);
  for (size_t i = 0; i < chunk.size(); ++i) chunk[i] = (unsigned char)(i * 7 + 1);
  REQUIRE(kvfold_oracle_append_bytes(cache.data(), Hkv, cap, d, len_prev, chunk.data(), C, 2) == 0, "append");
  REQUIRE(cache[((size_t)1 * cap + len_prev + 2) * d * 2 + 3] == chunk[((size_t)2 * Hkv + 1) * d * 2 + 3], "append layout");
  REQUIRE(kvfold_oracle_append_bytes(cache.data(), Hkv, cap, d, len_prev, chunk.data(), C + 1, 2) == -1, "append beyond capacity");
  std::printf("oracle: tiny cases ok\n");
}

int main() {
  model_sweep();
  planner_sweep();
  plans_of_single_heads();
  counter_slots();
  plans_of_few_rows();
  ring_depths();
  oracle_tiny();
  std::printf("ok: %ld checks\n", g_checks);
  return 0;
}
