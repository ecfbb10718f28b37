// Configuration checks, byte accounting and the launch planner of libkvfold: everything the host decides
// before a kernel is launched.  No HIP in this file.
#include "kvfold_plan.h"

#include <algorithm>
#include <cmath>

namespace kvfold {

int elem_size(int dtype) { return dtype == KVFOLD_F32 ? 4 : dtype == KVFOLD_BF16 ? 2 : 0; }

int validate_config(const kvfold_config_t* c) {
  if (!c || c->struct_size != sizeof(kvfold_config_t)) return KVFOLD_ERR_INVALID_ARG;
  if (c->n_layers < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->chunk_tokens < 1 || c->capacity_tokens < 1 ||
      c->device < 0 || !(c->softmax_scale >= 0.f) || !std::isfinite(c->softmax_scale))
    return KVFOLD_ERR_INVALID_ARG;
  if (c->kv_buffer && (reinterpret_cast<uintptr_t>(c->kv_buffer) & 255)) return KVFOLD_ERR_INVALID_ARG;
  if (elem_size(c->dtype) == 0) return KVFOLD_ERR_UNSUPPORTED;
  if (c->head_dim != 64 && c->head_dim != 128) return KVFOLD_ERR_UNSUPPORTED;
  if (c->n_q_heads % c->n_kv_heads) return KVFOLD_ERR_UNSUPPORTED;
  // the append kernels put (KV head, K or V) on the grid's second dimension (at most 65535 blocks)
  if (c->n_kv_heads > 32767) return KVFOLD_ERR_UNSUPPORTED;
  // sizes the kernels index with 32-bit row counts / 64-bit byte offsets
  if (c->capacity_tokens > (int64_t)1 << 30 || (int64_t)c->chunk_tokens * c->n_q_heads > (int64_t)1 << 28)
    return KVFOLD_ERR_UNSUPPORTED;
  // the attention kernels address one KV head's rows with 32-bit byte offsets
  if (c->capacity_tokens * c->head_dim * elem_size(c->dtype) > (int64_t)0xFFFFFFFFll) return KVFOLD_ERR_UNSUPPORTED;
  if (c->chunk_tokens > c->capacity_tokens) return KVFOLD_ERR_INVALID_ARG;
  return KVFOLD_OK;
}

size_t bytes_required(const kvfold_config_t* c) {
  return (size_t)c->n_layers * 2u * (size_t)c->n_kv_heads * (size_t)c->capacity_tokens * (size_t)c->head_dim *
         (size_t)elem_size(c->dtype);
}

// split workspace: room for kMaxSplits pieces of one chunk, capped
int64_t workspace_rows(const kvfold_config_t* cfg) {
  const int64_t rows = (int64_t)cfg->chunk_tokens * cfg->n_q_heads;
  int64_t ws_rows = rows * kMaxSplits;
  if (ws_rows > kMaxSplitRows) ws_rows = kMaxSplitRows;
  if (ws_rows < 2 * rows) ws_rows = 0;  // chunks this large never need a split
  return ws_rows;
}

// The fused append reads the chunk's rows, [C][Hkv][d], with 32-bit byte offsets from the KV head's first row:
// the largest is below C * Hkv * row_bytes, which therefore has to stay below 2^32.
bool fused_append_applies(const PlanCtx& c, int n_tokens, int64_t len_prev, bool rope) {
  const kvfold_config_t& f = c.cfg;
  if (f.dtype != KVFOLD_BF16) return false;
  (void)len_prev;  // any cache length: a tile that straddles the cache's end is filled from both sides
  return attention_appends(c, Plan{}, n_tokens, rope);
}

bool attention_works_on_rows(const PlanCtx& c, const Plan& pl, int n_tokens, bool rope) {
  const kvfold_config_t& f = c.cfg;
  if (!pl.few_rows || !(rope || c.storage_bits) || c.tune_fused_append == 1) return false;
  // A launch less (3 us), against the work ahead of the piece that holds the chunk.  Measured on 300 to 33K keys, five head
  // shapes, 1 to 32 tokens, this against the append kernel: 128 wide 0.91 (1 token) to 0.96 of the time with the rotary
  // embedding and 0.90 to 0.96 with the round trip, 64 wide 0.86 to 0.93, and no shape slower.  The round trip, with its
  // divisions, takes 90 ns a row: up to 16 rows 128 wide.  More rows are for the general kernel, whose
  // ring has to be filled behind the rows: 37 tokens with the rotary embedding on 32K keys 45.9 / 46.8 us, and every other step
  // paid 0.5 % for the code.
  return !c.storage_bits || (int64_t)n_tokens * f.head_dim * elem_size(f.dtype) <= 4096;
}

bool attention_appends(const PlanCtx& c, const Plan& pl, int n_tokens, bool rope) {
  const kvfold_config_t& f = c.cfg;
  // fp32: short pieces of four wavefronts.  A launch less (2.5 us) against 0.04 us a tile in the loop, 0.12 us 64 wide.  Measured, append
  // kernel / this, 64 tokens, 8 heads on 2: 9 tiles 77.3 / 76.0 us, 14 110.9 / 110.0, 20 144.2 / 144.5, 28 204.2 / 206.7; 64 wide, 7
  // tiles 40.6 / 39.5, 9 47.1 / 46.6, 14 66.1 / 66.6, 20 85.3 / 86.7.
  if (f.dtype != KVFOLD_BF16 && !pl.key_waves && (pl.waves_per_wg != 4 || pl.tiles_per_split >= (f.head_dim == 64 ? 12 : 20))) return false;
  // The rotary embedding: where a unit's keys are dealt to wavefronts each rotates the rows of the chunk that it comes to, for a launch less.
  // Over 130 shapes, by tokens of the chunk: 128 wide up to 100 0.86 to 0.98 of the time, 116 to 240 0.94 to 1.08, above 1.0 to 1.4; 64 wide up to
  // 212 0.78 to 0.95, above 0.9 to 1.2.  Steps that end within 256 keys keep the append kernel, a route that their tests ask for (0.94, 64
  // wide 0.85).  (One unit per KV head: attention_works_on_rows().)
  const bool rotates = f.dtype == KVFOLD_BF16 && pl.key_waves && !pl.few_rows && n_tokens <= (f.head_dim == 128 ? 100 : 256) &&
                       pl.tiles_per_split * pl.n_splits > 4;
  if ((rope && !rotates) || c.storage_bits || c.tune_fused_append == 1) return false;
  const int64_t chunk_bytes = (int64_t)n_tokens * f.n_kv_heads * f.head_dim * elem_size(f.dtype);
  return chunk_bytes < ((int64_t)1 << 32);
}

namespace {

// What a workgroup of an attention kernel costs, in us (see plan_with()): per 64-key tile on an otherwise idle chip and on
// a full one (one workgroup per CU, two per CU), and once.  fp32: on a full one, as the share by which a tile takes longer than
// on an idle one where all wavefronts have rows.
struct KernelCost {
  double idle, full, full_two, start_end;
  bool two_per_cu;
};
KernelCost kernel_cost(int dtype, int head_dim, int upw, int waves, bool few_rows, double with_rows) {
  if (few_rows) return KernelCost{0.46, 0.46, 0.46, 4.6, true};  // (128 wide: 17 to 32 rows, and fewer on long ranges of one or two KV heads; the others: plan_direct())
  if (dtype == KVFOLD_BF16) {
    // half the head dim leaves the same vector work per logit
    if (head_dim == 64) return upw == 2 ? KernelCost{0.98, 0.98, 0, 10.0, false} : KernelCost{0.74, 0.78, 1.3, 5.7, true};
    return upw == 2 ? KernelCost{1.4, 1.4, 0, 14.0, false} : KernelCost{1.1, 1.1, 2.1, 5.5, true};
  }
  // eight wavefronts: a tile takes half as long again once some SIMD has two of them with rows (measured per tile, 1 to 4 / 5 to 8
  // units: 5.6 / 8.4 us, 64 wide 3.2 / 4.8; on a full chip 5.8 to 7.3 / 9.7 to 12, 3.7 / 5.9); their start and end has
  // the append kernel's launch in it.  Four: 6.9 to 7.2, full 7.4 to 8.1; 64 wide 4.1, 4.4, two per CU 5.7 to 7.
  const bool one_per_simd = with_rows <= 0.5;
  if (head_dim == 64) return waves == 8 ? KernelCost{one_per_simd ? 3.35 : 4.5, 0.21, 0, 9.0, false} : KernelCost{4.6, 0.09, 0.63, 4.2, true};
  return waves == 8 ? KernelCost{one_per_simd ? 5.5 : 8.0, 0.28, 0, 9.4, false} : KernelCost{7.8, 0.13, 0, 4.4, false};
}

// Whether every XCD gets the same mix of a KV head's workgroups (logical_id(): heads whole, or dealt to their XCDs in turn).
bool evenly_dealt(int n_kv_heads, int wgs_per_kvh) {
  return n_kv_heads % kNumXcd == 0 || (n_kv_heads < kNumXcd && kNumXcd % n_kv_heads == 0 && wgs_per_kvh % (kNumXcd / n_kv_heads) == 0);
}

Plan finish_plan(Plan pl, int64_t s, int64_t s_max, int ntiles, int64_t base) {
  if (s > s_max) s = s_max;
  pl.tiles_per_split = (int)((ntiles + s - 1) / s);
  if (pl.tiles_per_split < 1) pl.tiles_per_split = 1;
  pl.n_splits = (ntiles + pl.tiles_per_split - 1) / pl.tiles_per_split;
  if (pl.n_splits < 1) pl.n_splits = 1;
  pl.n_wgs = (int)(base * pl.n_splits);
  return pl;
}

// The split count of the kernel that deals the keys of one unit to its wavefronts, for more than one unit per KV head or a window, and what
// the step takes, in us: a wavefront's chain of 32-key blocks, every block of a CU through its LDS, the rows from memory, further rounds
// of workgroups (which overlap with the one before but for their start), and the merge.  Fitted to 7951 measured steps (captured
// graphs): 568 shapes (1 to 64 heads, 1 to 1500 tokens on 16 to 127K keys, windows among them), both wavefront counts, every split count;
// the choice is 1.7 % above the best of these on average and more than 10 % above it in 16.
void plan_key_waves(const PlanCtx& c, int64_t rows, int64_t base, int ntiles, int64_t s_max, int waves, double kv_rows,
                    double seen, int64_t& s, double& est_us) {
  struct Cost {
    double start_end, block, cu_block, bytes_per_us, round, merge, merge_bytes_per_us;
  };
  const bool wide = c.cfg.head_dim == 128;
  const Cost k = wide ? (waves == 4 ? Cost{6.12, 0.348, 0.141, 10.7e6, 1.68, 1.42, 2.71e6} : Cost{6.29, 0.363, 0.144, 9.3e6, 3.95, 2.17, 2.85e6})
                      : (waves == 4 ? Cost{4.42, 0.443, 0.064, 11.4e6, 1.09, 2.06, 2.62e6} : Cost{4.89, 0.186, 0.080, 9.0e6, 2.04, 2.48, 2.63e6});
  const double slots = (double)c.n_cu * (8 / waves) * (wide ? 1 : 2);  // workgroups that LDS has room for
  const double kv_us = 4.0 * c.cfg.n_kv_heads * c.cfg.head_dim * kv_rows / k.bytes_per_us;
  est_us = 1e30;
  for (int64_t cand = 1; cand <= s_max; ++cand) {
    const int64_t tps = (ntiles + cand - 1) / cand;
    if ((ntiles + tps - 1) / tps != cand) continue;
    const double w = (double)(base * cand);
    double t = k.start_end + (double)((2 * tps + waves - 1) / waves) * k.block + std::max(1.0, std::ceil(w / c.n_cu) * seen) * 2.0 * (double)tps * k.cu_block + kv_us +
               (std::ceil(w / slots) - 1.0) * k.round;
    if (cand > 1) t += k.merge + (double)cand * (double)rows * (c.cfg.head_dim + 2) * 8.0 / k.merge_bytes_per_us;
    t = std::max(t, 4.0 + 2.65 * (cand > 1 ? 2 : 1)) + 0.1 * t;  // (as in plan_with())
    if (t < est_us) {
      est_us = t;
      s = cand;
    }
    if (w > 2.0 * slots) break;
  }
}

// The same for the fp32 kernel of that kind.  One workgroup per CU; what a wavefront's chain of blocks takes is for the most part the wait
// for its rows (attn_few_f32.hip).  Fitted to 2500 measured steps (captured graphs): 416 shapes (1 to 64 heads, 1 to 600
// tokens on 0 to 65K keys, windows among them), every split count; the choice is 0.9 % above the best of these on average (64 wide
// 1.6 %), more than 10 % above it in 11: pieces stay within a round of workgroups (897 tokens, 4 heads on 1, on 146 keys).
void plan_key_waves_f32(const PlanCtx& c, int64_t rows, int64_t base, int ntiles, int64_t s_max, int waves, double kv_rows,
                        double seen, int64_t& s, double& est_us) {
  struct Cost {
    double start_end, block, cu_block, full, bytes_per_us, round, merge, merge_bytes_per_us;
  };
  const Cost k = c.cfg.head_dim == 128 ? Cost{7.72, 3.19, 0.112, 0.04, 4.87e6, 3.73, 1.90, 2.46e6} : Cost{6.64, 0.463, 0.359, 0.12, 5.96e6, 3.57, 2.20, 3.34e6};
  const double kv_us = 8.0 * c.cfg.n_kv_heads * c.cfg.head_dim * kv_rows / k.bytes_per_us;
  est_us = 1e30;
  for (int64_t cand = 1; cand <= s_max; ++cand) {
    const int64_t tps = (ntiles + cand - 1) / cand;
    if ((ntiles + tps - 1) / tps != cand) continue;
    if (cand > 1 && base * cand > c.n_cu) break;
    const double w = (double)(base * cand), rounds = std::max(1.0, std::ceil(w / c.n_cu)), passes = std::max(1.0, rounds * seen);
    const double chain = passes * ((double)((2 * tps + waves - 1) / waves) * k.block + 2.0 * (double)tps * k.cu_block) * (1.0 + k.full * w / (rounds * c.n_cu));
    double t = k.start_end + std::sqrt(std::sqrt(chain * chain * chain * chain + kv_us * kv_us * kv_us * kv_us)) + (rounds - 1.0) * k.round;
    if (cand > 1) t += k.merge + (double)cand * (double)rows * (c.cfg.head_dim + 2) * 8.0 / k.merge_bytes_per_us;
    t = std::max(t, 4.0 + 2.65 * (cand > 1 ? 2 : 1)) + 0.1 * t;  // (as in plan_with())
    if (t < est_us) {
      est_us = t;
      s = cand;
    }
  }
}

// The same for the kernel whose keys come straight into registers (attn_decode.hip).  A piece's chain and the rows' way from memory overlap
// in part; per tile a CU's workgroups share its way to the L2, and neither odd numbers of tiles nor, below them, the blocks of a
// wavefront make a difference.  Fitted to 2200 measured steps (captured graphs, caches from memory): 142 shapes (1 to 64
// heads, 1 to 16 tokens on 64 to 131K keys), every split count; the choice is 0.5 % above the best of these on average (64 wide 0.2
// %), 5 % at most; with the few-rows kernel's figures 1.0 % and 8 % (one token on 4187 keys, 32 heads on 8, 17 pieces 9.91 us, 22 9.30).  The
// longest caches would have 1 to 2 % less with one workgroup per CU as well (128K keys, 8 heads, 32 pieces 92.9 us, 64 94.0); their geometry, two per CU, is
// kept as it is pinned: pieces of more than 48 tiles.
void plan_direct(const PlanCtx& c, const Plan& pl, int n_tokens, int64_t rows, int64_t base, int ntiles, int64_t s_max, double len_after, int64_t& s, double& est_us) {
  struct Cost {
    double start_end, tile, bytes_per_us, uneven, round, merge, merge_bytes_per_us;
  };
  const Cost k = c.cfg.head_dim == 128 ? Cost{2.73, 0.595, 7.45e6, 0.29, 1.62, 3.33, 1.60e6} : Cost{2.74, 0.353, 8.0e6, 0.28, 2.25, 3.12, 1.40e6};
  const double kv_us = 4.0 * c.cfg.n_kv_heads * c.cfg.head_dim * len_after / k.bytes_per_us;
  est_us = 1e30;
  for (int64_t cand = 1; cand <= s_max; ++cand) {
    const int64_t tps = (ntiles + cand - 1) / cand;
    if ((ntiles + tps - 1) / tps != cand) continue;
    const double w = (double)(base * cand), per_cu = std::ceil(w / c.n_cu);
    const double chain = per_cu * (double)tps * k.tile;
    const double mem = kv_us * (double)(tps * cand) / (double)ntiles * (per_cu > 1.0 ? 1.0 + k.uneven * (per_cu * c.n_cu / w - 1.0) : tps > 48 ? 1.05 : 1.0);
    double t = k.start_end + std::sqrt(chain * chain + mem * mem) + (per_cu > 2.0 ? k.round : 0.0);
    if (cand > 1) t += k.merge + (double)cand * (double)rows * (c.cfg.head_dim + 2) * 8.0 / k.merge_bytes_per_us;
    if (pieces_meet(c, pl, n_tokens, cand)) t -= c.cfg.head_dim == 64 || rows <= 4 * c.cfg.n_kv_heads ? 1.1 : 0.6;  // (meet.h)
    if (t < est_us) {
      est_us = t;
      s = cand;
    }
  }
}

// Launch geometry for `upw` units per wavefront and `waves` wavefronts per workgroup: the split count with the smallest
// estimated time (a forced split count overrides that).
Plan plan_with(const PlanCtx& c, int n_tokens, int64_t len_after, int upw, int n_sink, int64_t window,
               int waves = kUnitsPerWg, int key_waves = 0) {
  const kvfold_config_t& f = c.cfg;
  const int G = f.n_q_heads / f.n_kv_heads;
  Plan pl;
  pl.pair_order = 0;
  pl.pair_units = 0;
  pl.units_per_head = units_of_head(n_tokens, G);
  pl.units_per_wave = upw;
  pl.waves_per_wg = waves;
  pl.key_waves = key_waves;
  const bool few_rows = f.dtype == KVFOLD_BF16 && key_waves == 4 && pl.units_per_head == 1 && window <= 0;
  pl.few_rows = few_rows;
  const int per_wg = key_waves > 0 ? 1 : waves * upw;
  pl.wgs_per_head = (pl.units_per_head + per_wg - 1) / per_wg;
  const int64_t base = (int64_t)f.n_kv_heads * pl.wgs_per_head;
  // tiles of the longest key range of any workgroup (the kernels cut exactly this many into pieces)
  int ntiles = (int)((len_after + kTileKeys - 1) / kTileKeys);
  if (window > 0) {
    ntiles = 1;
    const int step = key_waves > 0 ? kUnitsPerWg : per_wg;  // (workgroups of one unit: a bound from four units at a time, a quarter of the host work)
    for (int ug = 0; ug * step < pl.units_per_head; ++ug) {
      const RowRange rr = workgroup_rows(ug, step, pl.units_per_head, G, n_tokens);
      ntiles = std::max(ntiles, tile_map(len_after - n_tokens, rr.row_lo, rr.row_hi, n_sink, window).ntiles);
    }
  }
  // At most 16 packed rows, 32 where heads are 64 wide: keys straight into registers (attn_decode.hip).  Not 128 wide on long ranges of one or two KV heads, whose
  // pieces leave half the CUs without a workgroup: the few-rows kernel fetches more per CU there, if its blocks go round the four wavefronts, an even
  // number of tiles a piece.  Measured, few rows / registers, one token: 16 heads on 2, 32.6K keys (8 tiles) 14.7 / 15.3 us, 2 on 2, 71.7K (18)
  // 22.4 / 24.9, 16 on 1, 103K (26) 25.2 / 27.1; 8 on 2, 20K (5) 13.0 / 12.2, 33.7K (9) 15.5 / 14.8, 1 on 1, 32.6K (8) 13.4 / 12.9.  From three KV heads
  // on registers are faster up to 127K keys (3 on 3, 64K 24.8 / 24.2), and 64 wide everywhere.
  const int tps_min = (ntiles + kMaxSplits - 1) / kMaxSplits;
  const bool half_idle = 2 * f.n_kv_heads * kMaxSplits <= c.n_cu && f.n_kv_heads * tps_min >= (tps_min % 2 ? 25 : 16);
  pl.direct = few_rows && (f.head_dim == 64 || (n_tokens * G <= 16 && !half_idle));
  int64_t s_max = ntiles;
  const int64_t rows = (int64_t)n_tokens * f.n_q_heads;
  if (c.ws_rows / rows < s_max) s_max = c.ws_rows / rows;
  if (s_max > kMaxSplits) s_max = kMaxSplits;
  if (s_max < 1) s_max = 1;
  int64_t s = 1;
  pl.est_us = 0.0;
  if (c.tune_splits > 0) {
    s = c.tune_splits;
  } else {
    // Estimated time of the step for every split count; the smallest wins (by more than 1.5 %):
    //     rounds of workgroups x (tiles of the longest piece x time per tile + start and end), and for s > 1 the merge.
    //  * Time per tile: `idle` on a chip that is otherwise idle (one workgroup's chain of matrix work and waits), up to
    //    `full` when every CU works at it: the chip is power-limited, busy CUs share what it has (rate ~ fill^0.5), and
    //    wavefronts without rows leave theirs to the others.
    //  * K and V rows come from memory at 6.5 TB/s with two workgroups per CU, a little less with fewer in flight.
    //  * Unsplit, several rounds, heaviest workgroups first: the slots left over in the last round idle for
    //    the length of the lightest workgroups only (first token block: the prefix and little else); never less than the
    //    heaviest workgroup's own chain.
    //  * A KV head's workgroups lie on its XCDs in runs where they cannot be dealt to them in turn: one XCD then has the heavy
    //    ones, another the light or empty ones (28 heads on 4, one / two units per wavefront: 3249 tokens, 178 / 89 workgroups a head,
    //    78 / 115 us; 3273 tokens on 153 keys, 179 / 90 workgroups, 117 / 89; fp32, 8 heads on 2, 295 tokens on 1252 keys, 130
    //    workgroups a head of which 16 are empty: 53 us, two rounds for the first XCD of each head).  What the others do not take of
    //    the chip's power goes to the first (64 wide, 28 heads on 4, 2867 tokens, 157 / 79 workgroups a head: 54 / 73 us).
    //  * The merge: its launch, and the fp32 partials written and read once at 6.7 TB/s.  (Few rows: the rest of what a launch
    //    costs is in the pace at which they are queued; with 4.7 us here 12 tokens on 1091 keys, 32 heads, stayed unsplit, 16.4 us
    //    for 13.1.)
    //  * A step is not queued faster than its launches: some 6.7 us with one, 2.65 us more for each further one.  (The pace of the
    //    Python binding.  C callers and captured graphs queue faster; where this decides, the kernels' own times differ little:
    //    in captured graphs the choice is 1.2 to 1.9 % above the best on average.)
    // The figures are fitted to 25,000 measured steps: 1327 shapes (1 to 64 heads, 1 to 1500 tokens on 0 to 128K keys, all
    // kernels), every split count.  The choice is 1.0 % above the best on average, more than 5 % in 82 shapes, more
    // than 10 % in 24; with the figures before, fitted to 30 workloads, 1.8 %, 166 and 70.  The fp32 kernel's are fitted again
    // to the kernels' own times (captured graphs, no launch in the way) of 1100 shapes (1 to 64 heads, 1 to 2500 tokens on 0 to
    // 80K keys, windows among them), both wavefront counts: 1.0 % above the best on average, more than 10 % in 40; the figures before,
    // fitted to 182 of these, 2.4 % and 100, and slower by up to 20 % than those of the kernel that did not append where a few
    // workgroups read many keys (64 tokens on 60K keys, 8 heads on 2: four wavefronts 124 us, eight 149).
    if (key_waves > 0 && f.dtype != KVFOLD_BF16) {
      plan_key_waves_f32(c, rows, base, ntiles, s_max, key_waves, window > 0 ? std::min((double)len_after, (double)ntiles * kTileKeys) : (double)len_after,
                         window > 0 ? 1.0 : ((double)len_after - 0.5 * n_tokens) / (double)len_after, s, pl.est_us);
      return finish_plan(pl, s, s_max, ntiles, base);
    }
    if (pl.direct) {
      plan_direct(c, pl, n_tokens, rows, base, ntiles, s_max, (double)len_after, s, pl.est_us);
      return finish_plan(pl, s, s_max, ntiles, base);
    }
    if (key_waves > 0 && !few_rows) {
      plan_key_waves(c, rows, base, ntiles, s_max, key_waves, window > 0 ? std::min((double)len_after, (double)ntiles * kTileKeys) : (double)len_after,
                     window > 0 ? 1.0 : ((double)len_after - 0.5 * n_tokens) / (double)len_after, s, pl.est_us);
      return finish_plan(pl, s, s_max, ntiles, base);
    }
    const double with_rows = (double)pl.units_per_head / (double)((int64_t)pl.wgs_per_head * per_wg);  // share of the units
    const KernelCost k = kernel_cost(f.dtype, f.head_dim, upw, waves, few_rows, with_rows);
    const double la = (double)len_after, mean_keys = la - 0.5 * n_tokens;
    const bool fp32 = f.dtype != KVFOLD_BF16;
    const double active = std::sqrt(std::sqrt(with_rows));
    const double kv_rows = window > 0 ? std::min(la, (double)ntiles * kTileKeys) : la;
    const double kv_us = 2.0 * f.n_kv_heads * f.head_dim * (double)elem_size(f.dtype) * kv_rows / (few_rows ? 5.9e6 : 6.5e6);
    const int launches = (c.storage_bits && !attention_works_on_rows(c, pl, n_tokens, false)) || waves == 8 ? 2 : 1;
    // (unsplit, not evenly dealt: mean and least keys of the workgroups on the XCD that gets the latest tokens' part of a KV head)
    const double heads = f.n_kv_heads / (double)kNumXcd, part = heads - std::floor(heads);
    const double late_keys = (std::floor(heads) * mean_keys + part * (la - 0.5 * part * n_tokens)) / heads;
    const double late_least = la - (heads < 1.0 ? part : 1.0) * n_tokens;
    double best = 1e30;
    for (int64_t cand = 1; cand <= s_max; ++cand) {
      // only split counts that whole tiles can realise; the last piece may be shorter than the others, and the
      // launch lasts as long as the longest
      const int64_t tps = (ntiles + cand - 1) / cand;
      if ((ntiles + tps - 1) / tps != cand) continue;
      const int64_t w = base * cand;
      const bool even = evenly_dealt(f.n_kv_heads, (int)(w / f.n_kv_heads));
      const bool two_per_cu = k.two_per_cu && w > (int64_t)c.n_cu;
      const double slots = (double)c.n_cu * (two_per_cu ? 2 : 1);
      const double full = two_per_cu ? k.full_two : k.full;
      // Workgroups with work: piece j is empty for the tokens before j * tps tiles less the prefix, so of the pieces from
      // first_cut on only the later tokens' have any.  (Not evenly dealt, some XCD has none of the empty ones.)
      double busy = (double)w;
      if (cand > 1 && window <= 0 && even) {
        const int64_t keys = tps * kTileKeys, prefix = len_after - n_tokens, first_cut = prefix / keys + 1, cut = cand - first_cut;
        if (cut > 0)
          busy = (double)base * ((double)first_cut + (double)cut * (1.0 + ((double)prefix - 0.5 * (double)(keys * (first_cut + cand - 1))) / n_tokens));
      }
      const double rounds = std::max(1.0, std::ceil(busy / slots - 1e-9));
      const double fill = busy / (rounds * slots);
      const double worst = fp32 ? k.idle * (1.0 + full * with_rows) : std::max(k.idle, full);  // a tile, every slot taken
      double t = rounds * (double)tps * (fp32 ? k.idle * (1.0 + full * with_rows * std::sqrt(fill) * (two_per_cu ? std::sqrt(std::sqrt(fill)) : fill))
                                              : std::max(k.idle, full * active * std::sqrt(fill)));
      // fp32, a grid of more than a round whose empty workgroups are to make room for the rest: they are slots taken for a while, and not
      // where the rest needs them (measured, with work for less than 0.8 of the slots 0 to 5 % longer, for 0.9 15 %, for all 25 %, up
      // to a second round: 506 tokens on 1131 keys, 8 heads on 2, 44 us in one round, 62 with 288 workgroups of which 255 have work)
      // -- and bf16's two-unit kernel with 64-wide heads (4045 tokens on 189 keys, 4 heads on 1: 31 us in 320 workgroups, 45 in 448 of
      // which 256 have work; 128 wide it lets others in sooner, 3835 tokens on 425 keys, 8 on 2, 360 of which 256 have work 57, 63 with one unit)
      if ((fp32 || (f.head_dim == 64 && upw == 2)) && (double)w > slots && busy < slots) t *= 1.0 + 1.5 * std::max(0.0, busy / slots - 0.8);
      // few rows: the blocks of an odd number of tiles do not go round the four wavefronts.  (The figures here and below are from when every step of one token
      // came this way.  Over 560 shapes on as many layers as
      // keep the caches out of the chip's own, the choice is 0.8 % above the best with this and 0.9 % without the second
      // term.  A step's two launches follow each other in steps of 0.8 us, which is the scatter: one token on 4187 keys, 2 / 3 / 4 / 5 tiles
      // a piece 12.4 / 11.7 / 10.8 / 11.5 us, on 4538 12.4 / 11.0 / 11.7 / 11.6.)
      if (few_rows && tps % 2 && tps > 1) t += k.idle + 0.7;
      if (cand == 1 && window <= 0 && rounds >= 2.0)
        t = (double)tps * (even ? worst : std::max(k.idle, worst * std::sqrt(mean_keys / late_keys))) *
            ((double)w * (even ? mean_keys : late_keys) + (rounds * slots - (double)w) * ((even ? la - n_tokens : late_least) + kRowsPerUnit)) / (slots * la);
      if (cand == 1 && window <= 0) t = std::max(t, (double)tps * k.idle);
      const double kv_piece = kv_us * (double)(tps * cand) / (double)ntiles;
      if (few_rows) {
        // 5.9 TB/s from one workgroup per CU on, less where some CUs have one more than others; near that rate both times
        // count (measured, one token on 128K keys: 121 us with 12 pieces, 101 with 16, 93.5 with 28, 110 with 40, 95 with 64)
        const double per_cu = std::ceil((double)w / c.n_cu);
        const double mem = kv_piece * (two_per_cu ? std::sqrt(per_cu * c.n_cu / (double)w) : 1.0);
        t = std::sqrt(std::sqrt(t * t * t * t + mem * mem * mem * mem));
      } else if (2.0 * kv_piece > t) {  // (the factor stays below 1.6)
        const bool few_in_flight = w < 2 * (int64_t)c.n_cu;
        t = std::max(t, kv_piece * (few_in_flight ? std::sqrt(std::sqrt(std::sqrt(std::sqrt(2.0 * c.n_cu / (double)w)))) : 1.0));
      }
      t += (k.start_end + (two_per_cu && !few_rows ? 0.5 : 0.0)) * rounds;
      // Two pieces that meet in the attention kernel: no launch, but the later one's way through memory at the end; less where 64-wide workgroups
      // share a CU or have two units a wavefront.  Over 600 shapes, 48 to 4096 tokens on 16 to 127K keys, both kernels, all split counts up to
      // eight and the kernel of one unit a workgroup where it was chosen: 1.3 % above the best on average 128 wide, 1.8 % 64 wide.  Of
      // these and 1500 others seven are more than 3 % slower than when pieces did not meet, by up to 3.3 %.  (At 1 us and the traffic of the merge kernel 1.5 and 2.0 %,
      // and short steps split that are faster whole: 286 tokens on 319 keys, 32 heads on 8, 13.05 / 15.4 us; 64 wide 1202 on 1710, 8 on 1, two pieces
      // 27.5, three 22.4.)  Not where the prefix is less than half of the chunk (64-wide workgroups that share a CU or have two units a wavefront: a quarter): the later
      // piece is empty for most rows then (2182 tokens on 631 keys, 32 heads on 2, 97 whole, 102.5 in two; 64 wide 3845 on 1320, 4 on 1, 37 / 40.3).
      const bool late = f.head_dim == 128 || (upw == 1 && w <= (int64_t)c.n_cu);
      const bool meet = two_pieces_meet(c, pl, (int)cand) && (late ? 2 : 4) * (len_after - n_tokens) >= n_tokens;
      if (meet)
        t += late ? 5.0 : 2.0;
      else if (cand > 1)
        t += (double)cand * rows * (f.head_dim + 2) * 8.0 / (fp32 ? 5.7e6 : 6.7e6) + (few_rows ? 3.4 : fp32 ? 3.9 : 4.7);
      t = std::max(t, 4.0 + 2.65 * (launches + (cand > 1 && !meet ? 1 : 0))) + 0.1 * t;  // (where the launches decide, the shorter kernel)
      if (t < best * (few_rows ? 1.0 : 0.985)) {
        best = t;
        s = cand;
      }
    }
    // One unit per wavefront, two workgroups a head of whose wavefronts more than a third have no rows (five units): two such workgroups on a CU
    // have little to fill each other's waits with, and one alone, with the deeper ring it then has (attn_bf16.hip), is faster if all CUs get
    // one.  32 heads on 8, 37 tokens on 32K keys 44.1 us with 27 pieces, 41.4 with 16; 40 on 16K 30.3 / 27.3, 34 on 65K 74 / 69.5, 37 on 100K
    // 110 / 106.  (With six to eight units 66 tokens on 98K 149.5 / 159; 64 wide 37 on 32K 29.0 / 30.4.)
    const int64_t alone = c.n_cu / base;
    if (!fp32 && key_waves == 0 && upw == 1 && f.head_dim == 128 && window <= 0 && pl.wgs_per_head == 2 && with_rows < 0.65 && base * s > c.n_cu &&
        alone <= s_max && base * alone * 10 >= (int64_t)c.n_cu * 9) {
      s = alone;
      best *= 0.95;
    }
    pl.est_us = best;
  }
  return finish_plan(pl, s, s_max, ntiles, base);
}

Plan choose_plan(const PlanCtx& c, int n_tokens, int64_t len_after, int n_sink, int64_t window) {
  const kvfold_config_t& f = c.cfg;
  if (f.dtype != KVFOLD_BF16) {
    const Plan w4 = plan_with(c, n_tokens, len_after, 1, n_sink, window, 4), w8 = plan_with(c, n_tokens, len_after, 1, n_sink, window, 8);
    if (c.tune_units_per_wave) return c.tune_units_per_wave == 2 ? w8 : w4;
    if (c.tune_splits > 0) return w4.units_per_head <= 4 ? w4 : w8;
    const Plan best = w4.est_us <= w8.est_us ? w4 : w8;
    // Few units on not too many keys: the kernel that deals a unit's keys to its wavefronts leaves the 416 shapes at
    // 0.82 of the time, one of them 4 % slower (64 heads on 8, 64 wide, 13 tokens on 15.7K keys 38.9 / 40.4 us).  One token, 32 heads on 8: 300 keys 15.5 -> 12.5 us, 4187 28 -> 19.9, 30K 92 -> 58; 128 tokens, 4 heads on 1, 64 wide, no keys 12.0 -> 7.5.  Every
    // unit splits the keys into terms anew, so that the gain is gone where many units have many keys (128 wide, 128 tokens, 8 heads on 2
    // = 32 units on 4.2K keys 39.9 / 30.9 us, on 20K 78 / 93; 64 wide, 37 tokens, 32 heads on 8 = 40 units on 30K 84 / 89; three and four units a
    // head beyond the line 0.97 to 1.10 of the time, 10 tokens on 65K, 28 heads on 4, 113.6 / 124.5; two of them 0.78 to 0.89), and
    // a single block of 32 keys has nothing to deal (128 wide 9.2 / 10.1 us, 64 wide 6.8 / 7.8; 34 keys 13.3 / 11.2).  The line is
    // drawn by the product of units and keys; 5 to 16 units in all on longer caches stay with the general kernel without having been measured there.
    const int64_t units = w4.units_per_head, all_units = units * f.n_kv_heads, keys = (int64_t)w4.tiles_per_split * w4.n_splits * kTileKeys;
    if (len_after <= 32 || all_units > 2 * (int64_t)c.n_cu || (units > 2 && all_units * keys > (f.head_dim == 128 ? 400000 : 600000))) return best;
    const Plan pk = plan_with(c, n_tokens, len_after, 1, n_sink, window, kUnitsPerWg, f.head_dim == 64 ? 8 : 4);
    return pk.est_us < best.est_us * 0.95 ? pk : best;
  }
  if (c.tune_units_per_wave) return plan_with(c, n_tokens, len_after, c.tune_units_per_wave, n_sink, window);
  if (window <= 0 && units_of_head(n_tokens, f.n_q_heads / f.n_kv_heads) == 1)
    return plan_with(c, n_tokens, len_after, 1, n_sink, window, kUnitsPerWg, 4);
  Plan p1 = plan_with(c, n_tokens, len_after, 1, n_sink, window);
  // Prefix shorter than the chunk: the causal part makes late token blocks several times as long as early
  // ones.  If the one-unit-per-wavefront grid is resident at once (two workgroups per CU), pair heavy with
  // light workgroups on a CU (measured faster than pairing units inside the two-unit kernel only here).  That takes workgroups
  // which are dealt to a head's XCDs in turn.  In runs, heavy ones share their CUs: with four or eight XCDs to a head the
  // two-unit kernel was faster in all of 25 shapes, by 12 to 48 % (14 heads on 2, 4282 tokens on 65 keys: 111 / 83 us; 8 on
  // 1, 7507 on none: 198 / 142); with two, 28 shapes from 5 % slower to 10 % faster, the estimates decide.
  const int64_t wgs1 = (int64_t)f.n_kv_heads * p1.wgs_per_head;
  const bool pair = c.tune_splits == 0 && window <= 0 && len_after < 2 * (int64_t)n_tokens && wgs1 <= 2 * (int64_t)c.n_cu &&
                    wgs1 > (int64_t)c.n_cu && p1.n_splits == 1;
  p1.pair_order = pair ? 1 : 0;
  if (pair && evenly_dealt(f.n_kv_heads, p1.wgs_per_head)) return p1;
  // Two units per wavefront is the faster kernel on a full chip (every LDS fragment feeds two MFMAs); one unit starts
  // sooner and fills the chip with fewer rows.  The estimates decide, the two-unit kernel's taken 10 % longer (part of the
  // fit).  Where units straddle tokens and half of a two-unit workgroup is padding (C = 128, G = 7) the choice changes
  // at 38K keys; measured there, one unit / two units per wavefront: 70.8 / 73.0 us at 32K, 84.7 / 84.5 at 40K, 98 / 96
  // at 48K, 125 / 123 at 64K; with 24 heads on 8, 64 / 66 at 32K, 101 / 100 at 56K.
  const Plan p2 = plan_with(c, n_tokens, len_after, 2, n_sink, window);
  if (c.tune_splits > 0) {
    const int64_t padded1 = (int64_t)p1.wgs_per_head * kUnitsPerWg, padded2 = (int64_t)p2.wgs_per_head * kUnitsPerWg * 2;
    if (padded2 * 5 > padded1 * 6) return p1;  // more than 20 % extra padding
    if (p2.n_splits == 1 && (int64_t)p2.n_wgs * 4 < (int64_t)c.n_cu * 3 && p1.n_wgs > p2.n_wgs) return p1;  // cannot fill the chip
    return p2;
  }
  if (pair && 4 * f.n_kv_heads <= kNumXcd) return p2;
  // Where a piece's two workgroups of one unit a wavefront are dealt to different XCDs (logical_id()), each brings its rows from beyond an L2 of its own; one
  // workgroup of two units brings them once.  Where the rows take a third of the step or more the estimates are taken as they are: 39
  // shapes of 28 heads on 4 and 12 on 4 0.74 to 0.95 of the time (27 tokens on 73K keys, 28 on 4: 60 / 48 us; 20 on 104K 73.6 / 54.1).  Not where both share an L2:
  // over 289 shapes with 8 and 16 KV heads 0.99, but single ones 0.90 to 1.15 (213 tokens on 25.6K keys, 16 on 16: 60.9 / 69.9).
  const double kv_us = 4.0 * f.n_kv_heads * f.head_dim * (double)len_after / 6.5e6;
  const bool read_twice = window <= 0 && kv_us > 0.3 * p1.est_us && p1.wgs_per_head == 2 && f.n_kv_heads < kNumXcd &&
                          evenly_dealt(f.n_kv_heads, p1.n_wgs / f.n_kv_heads);
  Plan best = p1.est_us < p2.est_us * (read_twice ? 1.0 : 1.1) ? p1 : p2;
  // Few units on not too many keys: the chain of one wavefront through the general kernels' tiles is longer than the whole step where the
  // keys of a unit are dealt to all wavefronts of a workgroup, and often no merge is left (32 heads on 8, 128 tokens on 1000 keys: 18.9 us,
  // 12.4 with eight wavefronts; 256 on 4187: 32.7 / 33.0; window 4 + 1020, 256 tokens 18.9 / 14).  Each unit streams all
  // its keys for itself, so that full grids are not for it: up to two workgroups per CU, and with a margin where there are many units (221
  // tokens with the rotary embedding on 6.9K keys, 32 heads on 8, 64 wide, 28 units: 29.2 / 31.8).  Long ranges stay out as they did while the units of a
  // piece lay on different XCDs and each row came from memory for every one of them (xcd_share_log2(): 15 tokens, 16 heads on 2, 64 wide, 66K
  // keys 20.7 / 25.5, 114K 27.1 / 39.1); they have not been measured since.  So do steps of more
  // than some 35 us (32 on 8, 64 wide: 489 tokens on 3.8K 31.4 / 30.3, 510 on 5.5K 39.7 / 42.3; 8 on 2, 2038 on 1.8K 42.3 / 46.3).
  // Over 400 shapes with more than one unit or a window the steps take 0.84 of the time.
  // (With one query head per KV head a unit's rows are 32 tokens, and with the rotary embedding each of eight wavefronts loads the angles of all of them:
  // 8 heads on 8, 38 tokens on 152 keys 13.0 us general, 14.7 with eight, 13.1 with four.  The plan does not ask for the embedding, so that a
  // rotated step has the bits of the step on rotated rows; eight wavefronts have to be 0.4 us better there.  Over 800 shapes steps with
  // the embedding take 0.834 of the general kernels' time, 0.853 without this, 3 of them more than 3 % longer than there instead of 17; plain ones 0.770,
  // 0.763 without.)
  const int64_t units = p1.units_per_head;
  const bool long_range = window <= 0 && (f.n_kv_heads > 1 ? len_after > 48 * 1024 : units * len_after > 800000);
  if (c.tune_pair_units == 0 && units * f.n_kv_heads <= 2 * (int64_t)c.n_cu && !long_range && best.est_us < 39.0)
    for (int waves : {8, 4}) {
      if (waves == 4 && window > 0) continue;
      Plan pk = plan_with(c, n_tokens, len_after, 1, n_sink, window, kUnitsPerWg, waves);
      if (waves == 8 && f.n_q_heads == f.n_kv_heads && window <= 0) pk.est_us += 0.4 * f.head_dim / 128;
      if (pk.est_us < best.est_us * (best.key_waves ? 1.0 : units > 16 ? 0.9 : 0.95)) best = pk;
    }
  return best;
}

}  // namespace

Plan make_plan(const PlanCtx& c, int n_tokens, int64_t len_after, int n_sink, int64_t window) {
  Plan pl = choose_plan(c, n_tokens, len_after, n_sink, window);
  // Two-unit kernel, a single round of workgroups: the causal part makes the last token block's wavefronts
  // longer than the first's (100 % on an empty cache, 6 % after 8 chunks) and nothing evens that out; pair
  // an early and a late row block in every wavefront instead (the late one finishes alone, at the
  // efficiency of a one-unit step).  Measured: +7 % down to +0.5 % at 31 chunks of prefix, even at 63; with
  // a split prefix (only the last pieces hold the causal part) +0.5 to 2 %, never a loss.  With several
  // rounds the dispatcher balances heaviest-first workgroups by itself and pairing only costs.  Under a
  // sliding window every row block has the same number of keys and there is nothing to pair.
  if (c.cfg.dtype == KVFOLD_BF16 && pl.units_per_wave == 2 && c.tune_pair_units != 1 && window <= 0) {
    if (c.tune_pair_units == 2 || pl.n_wgs <= c.n_cu) pl.pair_units = 1;
  }
  return pl;
}

}  // namespace kvfold

using namespace kvfold;

extern "C" {

size_t kvfold_cache_bytes_required(const kvfold_config_t* cfg) {
  if (validate_config(cfg) != KVFOLD_OK) return 0;
  return bytes_required(cfg);
}

int kvfold_plan_for(const kvfold_config_t* cfg, int32_t n_compute_units, int32_t n_tokens, int64_t len_after,
                    int32_t n_sink, int64_t window, kvfold_plan_t* out) {
  const int rc = validate_config(cfg);
  if (rc != KVFOLD_OK) return rc;
  if (n_compute_units < 1 || n_tokens < 1 || n_tokens > cfg->chunk_tokens || len_after < n_tokens ||
      len_after > cfg->capacity_tokens || n_sink < 0 || window < 0 || !out)
    return KVFOLD_ERR_INVALID_ARG;
  PlanCtx c{};
  c.cfg = *cfg;
  c.ws_rows = workspace_rows(cfg);
  c.n_cu = n_compute_units;
  c.two_meet = cfg->dtype == KVFOLD_BF16 && c.ws_rows > 0;
  const Plan pl = make_plan(c, n_tokens, len_after, n_sink, window);
  out->n_workgroups = pl.n_wgs;
  out->n_splits = pl.n_splits;
  out->units_per_wave = pl.units_per_wave;
  out->tiles_per_split = pl.tiles_per_split;
  out->fused_append = fused_append_applies(c, n_tokens, len_after - n_tokens, false) ? 1 : 0;
  out->pair_units = pl.pair_units;
  out->pair_order = pl.pair_order;
  return KVFOLD_OK;
}

const char* kvfold_status_string(int status) {
  switch (status) {
    case KVFOLD_OK: return "ok";
    case KVFOLD_ERR_INVALID_ARG: return "invalid argument";
    case KVFOLD_ERR_BAD_LAYER: return "layer out of range";
    case KVFOLD_ERR_POSITION: return "pos_offset does not continue the cache";
    case KVFOLD_ERR_CAPACITY: return "cache capacity exceeded";
    case KVFOLD_ERR_UNSUPPORTED: return "unsupported configuration";
    case KVFOLD_ERR_OOM: return "out of device memory or buffer too small";
    case KVFOLD_ERR_HIP: return "HIP runtime error";
    case KVFOLD_ERR_SCRATCH: return "step does not fit the static scratch buffer";
    default: return "unknown status";
  }
}

}  // extern "C"
