// Host-only part of libkvfold that needs no HIP: configuration checks, byte accounting and the launch
// planner.  Built into the library and, as plain C++ with the host sanitizers, into a test program.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>

#include "../../include/kvfold.h"
#include "kvfold_consts.h"

namespace kvfold {

constexpr int64_t kMaxSplitRows = 1 << 19;  // cap on S * C * Hq rows held in a cache's split workspace
constexpr int64_t kStaticScratchRows = 1 << 17;  // (row, split) pairs of the static array of steps that allocate nothing
constexpr int kMaxSplits = 64;

// What the planner needs to know of a cache (all host values).
struct PlanCtx {
  kvfold_config_t cfg;
  int64_t ws_rows;  // (row, split) pairs the split workspace in use can hold
  int n_cu;
  int tune_splits, tune_units_per_wave, tune_pair_units, tune_fused_append;
  int storage_bits;
  bool two_meet;  // a step's pieces may meet in the attention kernel (bf16, a cache with counters, whichever array holds the partial results)
};

struct Plan {
  bool few_rows;     // a bf16 kernel for at most 32 packed rows per KV head
  bool direct;       // of these, the one whose keys come straight into registers: at most 16 rows (not on long ranges of one or two KV heads), 32 where heads are 64 wide
  int key_waves;     // the kernel whose workgroups deal the keys of one unit to their wavefronts: 4 or 8 of them (0: another kernel)
  int waves_per_wg;  // 4, or 8 in the fp32 kernel's large form
  int units_per_wave, units_per_head, wgs_per_head, n_splits, tiles_per_split, n_wgs, pair_order, pair_units;
  double est_us;  // the planner's time estimate of the step (0 when the split count was forced)
};

// Counters of a cache (AttnParams::merge_count), and whether the two pieces of a step with this plan meet in the attention kernel, through
// them and the workspace, which holds whole units then, a lane's own (m, l) for each of the two lanes of a row.
constexpr int kMergeCounters = 8192;
inline bool two_pieces_meet(const PlanCtx& c, const Plan& pl, int n_splits) {
  const int64_t waves = (int64_t)c.cfg.n_kv_heads * pl.wgs_per_head * kUnitsPerWg;
  return c.two_meet && n_splits == 2 && !pl.key_waves && waves <= kMergeCounters && 2 * waves * pl.units_per_wave * 64 <= c.ws_rows;
}

// The kernel whose pieces may meet in the last one's workgroup (meet.h), and whether they do: at most four rows, one a wavefront, or eight, then
// 128 wide at most twelve pieces.
constexpr int kMeetUnits = 1024, kMeetSplits = 32, kMeetSplitsFew = 12;
constexpr int kMeetStride = 64;  // words of a KV head, its counter for every number of pieces among them
inline bool pieces_meet(const PlanCtx& c, const Plan& pl, int n_tokens, int64_t n_splits) {
  const int rows = n_tokens * (c.cfg.n_q_heads / c.cfg.n_kv_heads);
  return c.two_meet && pl.direct && n_splits > 1 && n_splits <= (rows <= 4 || c.cfg.head_dim == 64 ? kMeetSplits : kMeetSplitsFew) && rows <= 8 &&
         c.cfg.n_kv_heads <= kMeetUnits;
}

// The caches' places among the static counters of a GPU: each in one cache's hands at a time.
struct CounterSlots {
  static constexpr int kCount = 64;
  std::mutex mutex;
  uint64_t taken = 0;
  int take() {  // -1: none is free
    std::lock_guard<std::mutex> lock(mutex);
    for (int i = 0; i < kCount; ++i)
      if (!(taken >> i & 1)) {
        taken |= uint64_t{1} << i;
        return i;
      }
    return -1;
  }
  void give(int i) {
    std::lock_guard<std::mutex> lock(mutex);
    taken &= ~(uint64_t{1} << i);
  }
};

int elem_size(int dtype);
int validate_config(const kvfold_config_t* c);
size_t bytes_required(const kvfold_config_t* c);
// (row, split) pairs of the workspace that kvfold_cache_create reserves
int64_t workspace_rows(const kvfold_config_t* cfg);
// Launch geometry of one step of n_tokens rows that leaves the cache at len_after rows; window > 0 selects the
// sink + sliding-window step (n_sink first keys plus the last `window` keys of every row).
Plan make_plan(const PlanCtx& c, int n_tokens, int64_t len_after, int n_sink, int64_t window);
// Whether the rows of a step with this plan, which need work on their way into the cache, are appended by the workgroups of
// the few-rows kernel that read them.
bool attention_works_on_rows(const PlanCtx& c, const Plan& pl, int n_tokens, bool rope);
// Whether the attention kernel of a step with this plan does the append itself, and whether it is a bf16 kernel that does
// (kvfold_plan_t::fused_append, which has always been about these).
bool attention_appends(const PlanCtx& c, const Plan& pl, int n_tokens, bool rope);
bool fused_append_applies(const PlanCtx& c, int n_tokens, int64_t len_prev, bool rope);

}  // namespace kvfold
