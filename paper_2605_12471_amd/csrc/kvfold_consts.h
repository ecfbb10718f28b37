// Tile geometry shared by the kernels and the host-side planner (no HIP types here: the planner is built
// as plain C++ as well, for host-only tests).
#pragma once

namespace kvfold {

// Rows of a unit, the work of one wavefront: 32 consecutive rows of a KV head's (token, query head of the group)
// rows, token-major -- packed row r of the KV head is token r / G, head r % G of its group.
constexpr int kRowsPerUnit = 32;
// Wavefronts (units) per workgroup of the attention kernels.
constexpr int kUnitsPerWg = 4;
// Keys per K/V tile staged through LDS.
constexpr int kTileKeys = 64;
// The hardware hands workgroup b to XCD b % 8.
constexpr int kNumXcd = 8;


#if defined(__HIP__)
#define KVFOLD_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define KVFOLD_HD inline
#endif

// Which workgroup the hardware's block b of `grid` is: logical ids run KV head major, then split, then workgroup of the head, heaviest
// first; per_kvh of them belong to a KV head.  Dealt out in 8 contiguous runs, one per XCD, they keep the workgroups of a KV head, and of
// a piece of its keys, on one XCD's L2 (share_log2 < 0).  A KV head that spans k = 8 / Hkv = 2^share_log2 XCDs may have its
// workgroups dealt to those XCDs in turn instead: every XCD then gets the same mix of heavy and light workgroups and of prefix splits (a
// contiguous run would put all late token blocks, or a whole split, on one XCD and the light rest on its neighbour).
KVFOLD_HD int logical_id(unsigned b, unsigned grid, unsigned per_kvh, int share_log2) {
  const unsigned x = b % kNumXcd, j = b / kNumXcd;
  if (share_log2 >= 0) return (int)((x >> share_log2) * per_kvh + (j << share_log2) + (x & ((1u << share_log2) - 1)));  // grid = Hkv * per_kvh
  return (int)(x * (grid / kNumXcd) + j);
}
inline int padded_grid(int n_wgs) { return (n_wgs + kNumXcd - 1) / kNumXcd * kNumXcd; }
// share_log2 of a launch.  one_unit_wgs: workgroups of one unit, whose keys are dealt to their wavefronts.  Each of these streams all the keys of
// its piece, so that the units of a piece belong on one XCD, where the first to ask brings a row into the L2 for all: dealt in turn, every
// row came from beyond an L2 as many times as the piece has units on different XCDs.  57 tokens on 36K keys, 4 heads on 1, 28.5 us where the general
// kernel takes 20.5; 19 on 43K, 8 heads on 2, 26.4 dealt, 18 in runs (a split count that does not deal evenly).
inline int xcd_share_log2(int n_kv_heads, int wgs_per_head, int n_splits, bool one_unit_wgs) {
  if (one_unit_wgs && wgs_per_head > 1 && n_splits > 1) return -1;
  if (n_kv_heads >= kNumXcd || kNumXcd % n_kv_heads || wgs_per_head * n_splits % (kNumXcd / n_kv_heads)) return -1;
  int lk = 0;
  while ((n_kv_heads << lk) < kNumXcd) ++lk;
  return lk;
}

// V ring slots of the general bf16 kernels (the K ring has one more): three for the two-unit kernel, and 128 wide for the one-unit kernel in grids
// that leave no CU two workgroups, where one has 112 KB of the CU's LDS to itself; two for the one-unit kernel else, so that two workgroups share the
// 160 KB (64 wide three).  With two slots a tile is asked for one tile's time ahead of its use, which a workgroup alone on its CU spends waiting: 37
// tokens, 32 heads on 8, on 32K keys, 16 pieces 49.8 -> 41.1 us, 64 tokens 53.6 -> 48.0, 64 workgroups with 128 tiles each 130 -> 105.  Four
// slots 41.6, 48.6 and 106: the longer fill is not won back.  Where two share a CU a deeper ring bought nothing.  64 wide a tile is half the rows, and
// 45 steps alone on their CUs take 0.962 of the time with two slots where they do not split the keys and 0.992 where they do (551 tokens on 66 keys, 32
// heads on 8, 15.5 -> 14.7 us; 379 on 3639, 28 on 4, 26.9 -> 26.0).
constexpr int kRingAlone = 3, kRingShared = 2;
inline int ring_slots(int head_dim, int units_per_wave, int n_wgs, int n_cu) {
  return units_per_wave == 2 || (head_dim == 128 && n_wgs <= n_cu) ? kRingAlone : kRingShared;
}

// Quotients by a divisor that the host knows: n / d = (n * mul) >> shift for every n < 2^31.  With l = ceil(log2 d),
// mul = ceil(2^(31+l) / d) < 2^32 overshoots by e = mul * d - 2^(31+l) < 2^l, and n * e < 2^(31+l).  Integer division
// has no instruction on the GPU; the half dozen that a workgroup needs to find its place took 1 us of its start.
struct FastDiv {
  unsigned mul;
  int shift;
};
inline FastDiv fast_div(int d) {
  int l = 0;
  while ((1ll << l) < d) ++l;
  FastDiv f;
  f.shift = 31 + l;
  f.mul = (unsigned)(((1ull << f.shift) + (unsigned)d - 1) / (unsigned)d);
  return f;
}
KVFOLD_HD unsigned quot(unsigned n, int d) { return n / (unsigned)d; }
// (in two 32-bit steps: the high word of 2 n mul, which is (n mul) >> 31, then the rest of the shift)
KVFOLD_HD unsigned quot(unsigned n, const FastDiv& d) { return (unsigned)(((unsigned long long)(2 * n) * d.mul) >> 32) >> (d.shift - 31); }

// 32-row units of one KV head: its n_tokens * G packed rows, the last unit filled up.
KVFOLD_HD int units_of_head(int n_tokens, int G) { return (int)(((long long)n_tokens * G + kRowsPerUnit - 1) / kRowsPerUnit); }
// First and last token (of the chunk) with a row in unit u; units are token-major, so they ascend with u.
// (DIV: the group size G itself, or its FastDiv.)
template <class DIV>
KVFOLD_HD int unit_first_token(int u, const DIV& G) {
  return (int)quot((unsigned)(u * kRowsPerUnit), G);
}
template <class DIV>
KVFOLD_HD int unit_last_token(int u, const DIV& G, int n_tokens) {
  const int t = (int)quot((unsigned)(u * kRowsPerUnit + kRowsPerUnit - 1), G);
  return t < n_tokens - 1 ? t : n_tokens - 1;
}

// Tokens [row_lo, row_hi] of the chunk with rows in workgroup `ug` of a KV head: its `upw_wg` consecutive units.
struct RowRange {
  int row_lo, row_hi;
};
template <class DIV>
KVFOLD_HD RowRange workgroup_rows(int ug, int upw_wg, int units_per_head, const DIV& G, int n_tokens) {
  int ufirst = ug * upw_wg, ulast = ufirst + upw_wg - 1;
  if (ulast > units_per_head - 1) ulast = units_per_head - 1;
  if (ufirst > ulast) ufirst = ulast;
  if (ufirst < 0) ufirst = 0;
  if (ulast < 0) ulast = 0;
  RowRange r;
  r.row_lo = unit_first_token(ufirst, G);
  r.row_hi = unit_last_token(ulast, G, n_tokens);
  if (r.row_lo > r.row_hi) r.row_lo = r.row_hi;
  return r;
}

// Key tiles a workgroup walks.  Plain step (window <= 0): physical tiles [0, ntiles) cover keys
// [0, len_prev + row_hi].  Sink + sliding-window step: the row at absolute position p sees keys j < n_sink and
// p - window < j <= p, so the workgroup needs the sink tiles [0, ns_t) and the tiles from the one that holds key
// len_prev + row_lo - window + 1 on; the `skip` tiles in between are never touched.  The kernels count LOGICAL
// tiles 0 .. ntiles-1; logical tile t is physical tile t + (t >= ns_t ? skip : 0).
struct TileMap {
  int ns_t, skip, ntiles;
};
KVFOLD_HD TileMap tile_map(long long len_prev, int row_lo, int row_hi, int n_sink, long long window) {
  const int nt_phys = (int)((len_prev + row_hi + 1 + kTileKeys - 1) / kTileKeys);
  TileMap tm;
  tm.ns_t = 0;
  tm.skip = 0;
  tm.ntiles = nt_phys;
  if (window <= 0) return tm;
  long long lb = len_prev + row_lo - window + 1;
  if (lb < 0) lb = 0;
  int ns_t = (n_sink + kTileKeys - 1) / kTileKeys;
  if (ns_t > nt_phys) ns_t = nt_phys;
  int tw0 = (int)(lb / kTileKeys);
  if (tw0 < ns_t) tw0 = ns_t;
  tm.ns_t = ns_t;
  tm.skip = tw0 - ns_t;
  tm.ntiles = nt_phys - tm.skip;
  return tm;
}


// Piece `split` of a workgroup's logical tiles, [t_begin, t_end), and what the DMA of its K/V tiles may touch.
// The LDS ring runs a few tiles ahead and knows no end, so every source row is clamped to row_lim, the last row
// of the piece that exists (the cache holds rows [0, len_prev + n_tokens)).  With the append fused into the
// attention kernel the chunk's rows are not in the cache yet: rows from chunk_row0 = len_prev on are read from the
// rows as handed in, [n_tokens][Hkv][d], counted from the chunk's first row -- unless the piece ends before the
// chunk begins, in which case nothing is ever read from there.  Physical tiles from t_new on lie wholly in the
// chunk; when len_prev is not a multiple of the tile, tile t_straddle = t_new - 1 holds rows of both.
struct KeyRange {
  int t_begin, t_end;   // logical tiles
  unsigned row_lim;     // last row (cache numbering) a DMA of this piece may read
  unsigned chunk_row0;  // first row that comes from the chunk as handed in (0xffffffff: none does)
  int t_new;            // first physical tile that lies wholly in the chunk (INT_MAX: none)
  int t_straddle;       // physical tile with rows on both sides of chunk_row0 (-1: none)
};
KVFOLD_HD KeyRange key_range(const TileMap& tm, int split, int tiles_per_split, long long len_prev, int n_tokens, bool fused) {
  KeyRange k;
  k.t_begin = split * tiles_per_split;
  k.t_end = k.t_begin + tiles_per_split;
  if (k.t_end > tm.ntiles) k.t_end = tm.ntiles;
  // (32 bits: a cache has at most 2^30 rows, and this is part of what a workgroup does before its first fetch)
  const int last = k.t_end - 1;  // (only used when the piece is not empty)
  const int row_end = (last + (last >= tm.ns_t ? tm.skip : 0)) * kTileKeys + kTileKeys - 1;
  const int Lm1 = (int)len_prev + n_tokens - 1;
  const int lim = row_end < Lm1 ? row_end : Lm1;
  k.row_lim = (unsigned)(lim < 0 ? 0 : lim);
  const bool reaches_chunk = fused && lim >= (int)len_prev;
  const unsigned row0 = (unsigned)len_prev;
  k.chunk_row0 = reaches_chunk ? row0 : 0xffffffffu;
  k.t_new = reaches_chunk ? (int)((row0 + kTileKeys - 1) / kTileKeys) : 0x7fffffff;
  k.t_straddle = reaches_chunk && row0 % kTileKeys ? (int)(row0 / kTileKeys) : -1;
  return k;
}

// Source of ring row `row_in_tile` (0 .. 63) of physical tile t_phys: a cache row of the KV head, or a row of the
// chunk as handed in (counted from its first row), clamped as described above.
struct DmaRow {
  bool from_chunk;
  unsigned row;
};
KVFOLD_HD DmaRow dma_row(const KeyRange& k, int t_phys, int row_in_tile) {
  unsigned r = (unsigned)(t_phys * kTileKeys + row_in_tile);
  r = r < k.row_lim ? r : k.row_lim;
  DmaRow d;
  d.from_chunk = r >= k.chunk_row0;
  d.row = d.from_chunk ? r - k.chunk_row0 : r;
  return d;
}

}  // namespace kvfold
