// Internal declarations shared by the HIP translation units of libkvfold (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kvfold_consts.h"
#include "kvfold_plan.h"

namespace kvfold {

struct AppendParams {
  const void* k_new;  // [C][Hkv][d]
  const void* v_new;  // [C][Hkv][d]
  void* k_cache;      // layer base, [Hkv][cap][d]
  void* v_cache;
  int32_t n_tokens;   // C
  int32_t n_kv_heads;
  int32_t row_bytes;  // d * elem_size, multiple of 16
  int64_t capacity;   // rows per head
  int64_t len_prev;   // first destination row
  // Rotary embedding of the K rows on their way into the cache (nullptr: plain bit copy): angles of the
  // rows' absolute positions, [C][d/2] fp32 each; V is never rotated.
  const float* rope_cos;
  const float* rope_sin;
  int32_t elem_is_bf16;
};

struct AttnParams {
  const void* q;         // [C][Hq][d]
  const void* k_cache;   // layer base, [Hkv][cap][d]; rows [0, len_prev + C) valid
  const void* v_cache;
  void* out;             // [C][Hq][d]
  float* lse;            // [Hq][C] or nullptr
  float* part_o;         // [S][C*Hq][d]  unnormalised partial outputs (split mode)
  float* part_ml;        // [S][C*Hq][2]  (running max in log2 units, partial sum)
  int32_t n_tokens;      // C
  int32_t n_q_heads;     // Hq
  int32_t n_kv_heads;    // Hkv
  int32_t group;         // G = Hq / Hkv
  int64_t capacity;      // rows per head in the cache
  int64_t len_prev;      // cache length before this chunk
  int32_t n_splits;      // S >= 1; S == 1 writes out/lse directly
  int32_t tiles_per_split;
  int32_t units_per_head;  // ceil(C * G / 32): units of 32 packed rows
  int32_t wgs_per_head;    // ceil(units_per_head / units per workgroup)
  int32_t n_wgs;           // Hkv * wgs_per_head * S (the grid is padded to a multiple of 8)
  int32_t pair_order;      // 1: every workgroup is resident at once, two per CU; order them heaviest-first for the
                           // first half and lightest-first for the second so each CU gets a balanced pair
  int32_t pair_units;      // two-unit bf16 kernel: a wavefront owns an early and a late unit of the chunk (see the kernel)
  uint32_t* merge_count;   // bf16 general kernel, two pieces: one counter per KV head and wavefront of its rows, even between steps (nullptr: the
                           // partial results are for the combine kernel)
  uint32_t* meet_count;    // the last of a KV head's pieces merges them, by these counters (see meet.h; nullptr: the combine kernel)
  float scale_log2e;       // softmax scale * log2(e)
  // Rotary embedding of the queries as they are loaded (nullptr: q is used as handed in): angles of the
  // chunk's absolute positions, [C][d/2] fp32 each
  const float* rope_cos;
  const float* rope_sin;
  // Append fused into the attention kernel (nullptr: the cache already holds the chunk's rows): the
  // chunk's K / V rows as handed in, [C][Hkv][d].  Tiles of the chunk are then streamed from here, and every
  // workgroup copies its share of the rows into the cache for the steps to come.
  const void* k_new;
  const void* v_new;
  // Few-rows kernel, rows that need work on their way into the cache (nullptr: not this step): the chunk's K / V rows as handed
  // in.  Every workgroup appends the rows of its piece (rotated if rope_cos, through the storage round trip if
  // work_qmax > 0) and then reads them from the cache like all others.
  const void* work_k;
  const void* work_v;
  float work_qmax;
  // Sink + sliding-window step (window > 0; 0: every key up to the row's own position is visible): the row at
  // absolute position p sees keys j < n_sink and p - window < j <= p.  Tiles between the sink tiles and the
  // window are skipped (see tile_map()).
  int32_t n_sink;
  int32_t window;
  // Quotients the workgroups need, prepared by finish_attn_params()
  FastDiv by_group, by_wgs_per_head, by_wgs_per_kvh;
  int32_t group_inv16;      // floor(2^16 / G) + 1
  int32_t copy_rows;        // fused append: chunk rows that one workgroup copies, ceil(C / (wgs_per_head * S))
  int32_t xcd_share_log2;   // log2 of the XCDs that a KV head's workgroups are dealt to, -1: contiguous runs (see logical_id())
};

// Fills in what follows from the launch geometry (one_unit_wgs: see xcd_share_log2()).
inline void finish_attn_params(AttnParams& p, bool one_unit_wgs) {
  const int per_kvh = p.wgs_per_head * p.n_splits;
  p.by_group = fast_div(p.group);
  p.by_wgs_per_head = fast_div(p.wgs_per_head);
  p.by_wgs_per_kvh = fast_div(per_kvh);
  p.group_inv16 = 65536 / p.group + 1;
  p.copy_rows = (p.n_tokens + per_kvh - 1) / per_kvh;
  p.xcd_share_log2 = xcd_share_log2(p.n_kv_heads, p.wgs_per_head, p.n_splits, one_unit_wgs);
}

struct CombineParams {
  const float* part_o;
  const float* part_ml;
  void* out;
  float* lse;          // [Hq][C] or nullptr
  int32_t n_rows;      // C * Hq
  int32_t n_tokens;    // C
  int32_t n_q_heads;
  int32_t head_dim;
  int32_t n_splits;
  int32_t out_is_bf16;
};

// storage_bits 4 or 8 (bf16 only): the rows take the storage round trip bf16 -> intN -> bf16 on their way; 0: they do not.
hipError_t launch_append(const AppendParams& p, int storage_bits, hipStream_t s);
hipError_t launch_attn_bf16(const AttnParams& p, int head_dim, int units_per_wave, int n_cu, hipStream_t s);
// Sets the LDS size attribute of every bf16 attention kernel variant of this head dimension on the current
// device (once per device; launches then have nothing left that could fail for a valid configuration).
hipError_t prepare_attn_bf16(int head_dim);
// The kernel whose workgroups deal the keys of one unit to key_waves wavefronts (4, or 8, which a window asks for); prepare as above.
hipError_t launch_attn_few(const AttnParams& p, int head_dim, int key_waves, hipStream_t s);
hipError_t prepare_attn_few(int head_dim);
// One unit per KV head, no window: at most 16 packed rows, 32 where heads are 64 wide (Plan::direct).
hipError_t launch_attn_decode(const AttnParams& p, int head_dim, hipStream_t s);
// The same as launch_attn_few in fp32: four wavefronts, eight where heads are 64 wide.
hipError_t launch_attn_few_f32(const AttnParams& p, int head_dim, hipStream_t s);
hipError_t launch_attn_f32(const AttnParams& p, int head_dim, int waves_per_wg, hipStream_t s);
hipError_t launch_combine(const CombineParams& p, hipStream_t s);

__device__ __forceinline__ int logical_workgroup(unsigned b, unsigned grid, const AttnParams& p) {
  return logical_id(b, grid, (unsigned)(p.wgs_per_head * p.n_splits), p.xcd_share_log2);
}

// Packed rows of one unit (row j of unit u: packed row 32 u + j of the KV head, j < 32): token and head of the group.
// One scalar quotient per unit; the lanes add rem0 + j < G + 32, whose quotient by G is a multiplication for G < 32
// (x < 64 and inv * G - 2^16 <= G, so x * inv / 2^16 never reaches the next whole number) and 0 or 1 above.
struct UnitRows {
  int tok0, rem0, G, inv;
  __device__ __forceinline__ UnitRows(int u, const AttnParams& p) : G(p.group), inv(p.group_inv16) {
    const unsigned r0 = (unsigned)u * kRowsPerUnit;
    tok0 = (int)quot(r0, p.by_group);
    rem0 = (int)(r0 - (unsigned)tok0 * (unsigned)G);
  }
  __device__ __forceinline__ int step(int j) const {
    const int x = rem0 + j;
    return G < kRowsPerUnit ? (x * inv) >> 16 : (int)(x >= G);
  }
  __device__ __forceinline__ int tok(int j) const { return tok0 + step(j); }
  __device__ __forceinline__ int head(int j) const { return rem0 + j - step(j) * G; }
};

}  // namespace kvfold
