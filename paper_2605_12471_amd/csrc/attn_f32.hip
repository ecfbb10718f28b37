// Chunk-prefix attention of the fold step in fp32 (the precision-ablation mode of the paper's Sec. 3; here the 1e-5
// correctness mode).  Same decomposition as the bf16 kernel: a wavefront owns one unit of 32 packed (token, head of the
// group) rows, the wavefronts of a workgroup share the K/V tiles of one KV head through LDS, logits are formed transposed
// (S^T = K Q^T, keys as MFMA rows) so that a lane holds logits of one query only, and S^T feeds O^T = V^T P^T directly.
//
// The products run on the bf16 matrix instructions, on operands split into three bf16 terms: x = x0 + x1 + x2, each term what
// is left of x rounded to nearest (sums of shorter floats: Dekker 1971; of bf16 numbers: Henry, Tang and Heinecke 2019), so that
// |x1| <= 2^-8 |x| and |x2| <= 2^-17 |x|, and
//     x y = x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0) + (x1 y2 + x2 y1, each at most 2^-25) + x2 y2 (2^-34),
// summed in fp32 like the fp32 instruction's own products.  Logits take all but the last: an error of a logit is one of its
// weight, and a logit may be a single large product.  P V takes the first six: what the others add is less than the row sums'
// rounding.  Seven bf16 32x32x16 instructions on average take 224 cycles where the eight 32x32x2 fp32 ones that they replace
// take 512, and round the sums less often.  Error against 64 bits, relative to what the fp32 instructions left (60 pairs of
// shape and distribution, N(0,1), larger, sparse and tiny values, geometric means): outputs 0.57 (2-norm) and 0.56 (largest),
// log-sum-exp 0.79; log-sum-exp of a single product 3.76e-8 against 3.76e-8 (with six products 3.80e-8, and with terms rounded
// towards zero 4.32e-8), output of a single product 7.5e-8 against 13.3e-8.
// 512 tokens on 16K keys, 28 heads: 1145 us with the fp32 instructions (108 TFLOP/s, of 157), 663 us now (187); six
// products everywhere would take 585, eight 730.
// What bounds it: 187 TFLOP/s are 1.31 PFLOP/s of bf16 products, near the 1.4 that the bf16 kernel reaches on the
// power-limited chip; the split and the softmax take a third of the issue slots.
// The terms are exact for every value that fp32 holds below 2^60 (see kProbe and kValueScale).
// K and V are split once per workgroup, on their way into LDS, where a tile's terms lie in the order in which the matrix
// instructions read their fragments: V is transposed by the split (a lane gathers 8 keys of one column), so that all
// fragment reads are 16 bytes per lane.  P is split in registers.
//
// The terms of an infinity would be NaN, and sums of terms of values above 2^60 could overflow.  A key whose K or V row holds
// such a number is left out of its tile and added after the piece's end with the fp32 instructions, operands straight from
// memory: rows that do not see it keep their bits.  A workgroup that met more such tiles than it can list, and the rows
// of a wavefront with such a query, take the whole piece that way.  Measured on 512 tokens on 16K keys (677 us): one NaN key
// 700 us, 24 infinite values 765, one in every tile 2350 (which the fp32 instructions alone did in 1142), a NaN query 1594;
// with the whole piece done again for one such key it was 5100.
#include <type_traits>

#include "f32_terms.h"
#include "kvfold_internal.h"
#include "wave_ops.h"

namespace kvfold {

// NW wavefronts per workgroup, one workgroup per CU at D = 128 (96 KB of LDS).  Eight (two per SIMD) share the split of a
// tile among twice the rows and have one wavefront's vector work behind the other's matrix work; four are for chunks that
// leave half of the eight without rows.  WIN: the sink + sliding-window step.  FUSED (four wavefronts): for short pieces, and the
// kernel may append the chunk's rows itself.
template <int D, bool WIN, int NW, bool FUSED>
__global__ void __launch_bounds__(NW * 64, NW / 4) attn_f32_kernel(AttnParams p) {
  constexpr int NT = NW * 64;
  constexpr int ROWB = D * 4;       // bytes per row of the cache
  constexpr int BN = 32;            // keys per step; the planner's tiles hold two
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int TERMB = BN * D * 2;          // one term of a K or V tile
  constexpr int BUFB = 2 * kTerms * TERMB;   // a K tile, a V tile
  constexpr int ITEMS = BN * D / 8;          // vectors of 8 values per tensor and tile
  constexpr int PER = ITEMS >= NT ? ITEMS / NT : 1;
  constexpr float kThresh = 8.0f;
  // The next tile's values on their way together with its keys, a step ahead of their use, where there are registers for it
  // (D = 128 has none left); 32 keys of half the width are worked off faster than memory answers.
  constexpr bool kBothAhead = D == 64 && (FUSED || NW == 8);

  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BUFB];
  // keys with a number that the terms cannot hold: by tile, for the two tiles in flight and one being cleared, and the list
  // of tiles with such keys
  constexpr int kOddList = 32;
  __shared__ unsigned odd_keys[3];
  __shared__ int odd_tiles;
  __shared__ struct { int h; unsigned keys; } odd_list[kOddList];

  const int wgs_per_kvh = p.wgs_per_head * p.n_splits;
  const int lid = logical_workgroup(blockIdx.x, gridDim.x, p);
  if (lid >= p.n_wgs) return;
  const int g = (int)quot((unsigned)lid, p.by_wgs_per_kvh);
  const int rem = lid - g * wgs_per_kvh;
  const int split = (int)quot((unsigned)rem, p.by_wgs_per_head);
  // Later token blocks see more keys: heaviest first (longest-processing-time first over several rounds of workgroups).
  const int ug = p.wgs_per_head - 1 - (rem - split * p.wgs_per_head);

  const int tid = threadIdx.x, l = tid & 63, hi = l >> 5, m = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: what depends on it alone stays in scalar registers
  const int C = p.n_tokens, Hq = p.n_q_heads, G = p.group;
  const int L = (int)p.len_prev + C;  // (row counts fit 32 bits: the host limits the capacity to 2^30 rows)

  const int u = ug * NW + w;
  const int uc = u < p.units_per_head ? u : p.units_per_head - 1;
  const bool idle = u >= p.units_per_head;  // no rows: this wavefront only moves its share of the tiles
  const UnitRows ur(uc, p);
  const bool inside = ur.tok(m) < C;
  const int tok = inside ? ur.tok(m) : C - 1;  // of this lane's row (the chunk's last row where the unit runs past it)
  const int head = g * G + (inside ? ur.head(m) : G - 1);
  const bool store_ok = !idle && inside;
  const int my_vis = (int)p.len_prev + tok + 1;
  const int vis_first = (int)p.len_prev + ur.tok0 + 1;
  // Sink + sliding-window step (Sec. 6 of the paper, the streaming baseline's mask): of the keys [0, vis) a row
  // sees only j < n_sink and j >= vis - window; lb_last is the largest such lower bound among the unit's rows
  constexpr bool win = WIN;
  const int vis_last = (int)p.len_prev + unit_last_token(uc, p.by_group, C) + 1;
  const int lb_last = vis_last - p.window;

  int nkeys_wg;
  {
    int ulast = ug * NW + NW - 1;
    if (ulast > p.units_per_head - 1) ulast = p.units_per_head - 1;
    nkeys_wg = (int)p.len_prev + unit_last_token(ulast, p.by_group, C) + 1;
  }
  // logical tiles 0 .. ntiles-1; under a window the tiles between the sinks and the window are left out:
  // logical tile t is physical tile t + (t >= ns_t ? skip : 0)
  TileMap tm;
  if (win) {
    const RowRange rr = workgroup_rows(ug, NW, p.units_per_head, p.by_group, C);
    tm = tile_map(p.len_prev, rr.row_lo, rr.row_hi, p.n_sink, p.window);
  } else {
    tm.ns_t = 0;
    tm.skip = 0;
    tm.ntiles = (nkeys_wg + kTileKeys - 1) / kTileKeys;
  }
  const int t_begin = split * p.tiles_per_split;
  int t_end = t_begin + p.tiles_per_split;
  if (t_end > tm.ntiles) t_end = tm.ntiles;
  const int h_begin = 2 * t_begin;
  int h_end = 2 * t_end;  // steps: half tiles
  auto first_key = [&](int h) __attribute__((always_inline)) -> int {
    const int t = h >> 1;
    return (2 * (t + (t >= tm.ns_t ? tm.skip : 0)) + (h & 1)) * BN;
  };
  if (h_end > h_begin && first_key(h_end - 1) >= nkeys_wg) --h_end;  // the piece's last half lies beyond every row

  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(p.k_cache) + (int64_t)g * p.capacity * ROWB;
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(p.v_cache) + (int64_t)g * p.capacity * ROWB;

  // ---- fused append (paper Sec. 2: the chunk's K/V rows join the cache): rows from chunk0 on are read as handed in,
  // [C][Hkv][d], so that no workgroup waits for another's copy; the copy into the cache, for the steps to come, is shared
  // out over the workgroups of the KV head.  As a kernel of its own it was one launch of the three that a short step took:
  // a fold of 4 x 128 tokens, 4 heads on 1, D = 64, 63.4 us with it, 56.9 without (three of these from loading the first
  // tile's values with its keys).  Not with eight wavefronts: their steps are long, and what the second source costs the
  // main loop in scalar registers is as much as the launch (512 tokens on 16K keys, 28 heads on 4: 645 us with the append
  // kernel, 647 without).  Nor for long pieces of four (attention_appends()): the instance without the second source is 1 to 2 % faster
  // per tile, 3.5 % 64 wide (64 tokens on 14K keys, 8 heads on 2, 40 tiles a piece: 269 us with it, 265 without; 64 wide 158 and 153;
  // one instance for both, before: 270 and 161 where the rows need the append kernel anyway, for the rotary embedding).
  const bool fused = FUSED && p.k_new != nullptr;
  const int chunk0 = fused ? (int)p.len_prev : 0x7fffffff;
  const unsigned new_stride = (unsigned)(p.n_kv_heads * ROWB);  // bytes from one token's row to the next
  const unsigned char* knew = reinterpret_cast<const unsigned char*>(p.k_new) + (int64_t)g * ROWB;
  const unsigned char* vnew = reinterpret_cast<const unsigned char*>(p.v_new) + (int64_t)g * ROWB;
  auto row_at = [&](bool is_v, int row) __attribute__((always_inline)) -> const unsigned char* {
    const bool nw = FUSED && row >= chunk0;
    const unsigned char* base = nw ? (is_v ? vnew : knew) : (is_v ? vbase : kbase);
    return base + (unsigned)(row - (nw ? chunk0 : 0)) * (nw ? new_stride : (unsigned)ROWB);
  };
  // ... of a tile whose rows are all in the cache (old), or not
  auto row_of = [&](bool is_v, int row, auto old_tag) __attribute__((always_inline)) -> const unsigned char* {
    if constexpr (decltype(old_tag)::value || !FUSED) return (is_v ? vbase : kbase) + (unsigned)row * (unsigned)ROWB;
    return row_at(is_v, row);
  };
  auto is_old = [&](int h) __attribute__((always_inline)) -> bool { return first_key(h) + BN <= chunk0; };
  // This workgroup's share of the copy: rows [copy_r0, copy_r1) of K and of V, 16 bytes per thread, loaded before the
  // results are stored and stored behind them.
  constexpr int CPR = ROWB / 16, kCopyRows = NT / CPR;
  const int copy_r0 = fused ? rem * p.copy_rows : 0;
  const int copy_r1 = fused ? (copy_r0 + p.copy_rows < C ? copy_r0 + p.copy_rows : C) : 0;
  uintx4 copy_k = {}, copy_v = {};
  auto copy_load = [&](int r0) __attribute__((always_inline)) {
    const int r = r0 + tid / CPR;
    if (r < copy_r1) {
      const unsigned off = (unsigned)r * new_stride + (unsigned)(tid % CPR) * 16u;
      copy_k = *reinterpret_cast<const uintx4*>(knew + off);
      copy_v = *reinterpret_cast<const uintx4*>(vnew + off);
    }
  };
  auto copy_store = [&](int r0) __attribute__((always_inline)) {
    const int r = r0 + tid / CPR;
    if (r < copy_r1) {
      const unsigned off = (unsigned)(chunk0 + r) * (unsigned)ROWB + (unsigned)(tid % CPR) * 16u;
      __builtin_nontemporal_store(copy_k, reinterpret_cast<uintx4*>(const_cast<unsigned char*>(kbase) + off));
      __builtin_nontemporal_store(copy_v, reinterpret_cast<uintx4*>(const_cast<unsigned char*>(vbase) + off));
    }
  };

  // ---- split of a tile on its way into LDS.  K: thread = (row, 8 columns), read as it lies; the fragment of contraction
  // step ks, lane (m, hi), goes to slot m ^ (2 ks + hi) % 8 of its 32, so that neighbouring threads, which hold neighbouring
  // columns of one row, write different banks.  V: thread = (column, the 8 keys that registers 8 tt .. 8 tt + 7 of S^T stand
  // for in its half-wave).  Rows past the last one are read as the last one (and masked).  With fewer vectors than
  // threads (D = 64, eight wavefronts) the first half of the wavefronts splits K, the second V.
  const bool k_mine = ITEMS >= NT || tid < ITEMS, v_mine = ITEMS >= NT || tid >= NT - ITEMS;
  float stage_k[PER][8], stage_v[PER][8];
  auto load_k = [&](int h, auto old_tag) __attribute__((always_inline)) {
    const int key0 = first_key(h);
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int ci = it * NT + tid;
      int row = key0 + ci / (D / 8);
      if (row > L - 1) row = L - 1;
      const float4* src = reinterpret_cast<const float4*>(row_of(false, row, old_tag) + (ci % (D / 8)) * 32);
      if (k_mine) {
        const float4 a = src[0], b = src[1];
        stage_k[it][0] = a.x; stage_k[it][1] = a.y; stage_k[it][2] = a.z; stage_k[it][3] = a.w;
        stage_k[it][4] = b.x; stage_k[it][5] = b.y; stage_k[it][6] = b.z; stage_k[it][7] = b.w;
      }
    }
  };
  auto load_v = [&](int h, auto old_tag) __attribute__((always_inline)) {
    const int key0 = first_key(h);
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int vi = it * NT + tid - (ITEMS >= NT ? 0 : NT - ITEMS);
      const int grp = __builtin_amdgcn_readfirstlane(vi / D);  // 2 tt + half-wave; 64 consecutive threads share it
      const int key = key0 + 16 * (grp >> 1) + 4 * (grp & 1);
      if (v_mine) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          int row = key + 8 * (j >> 2) + (j & 3);
          if (row > L - 1) row = L - 1;
          stage_v[it][j] = *reinterpret_cast<const float*>(row_of(true, row, old_tag) + (vi % D) * 4);
        }
      }
    }
  };
  auto put = [&](int h, bool is_v, float (&stage)[PER][8]) __attribute__((always_inline)) {
    unsigned char* buf = smem + (h & 1) * BUFB + (is_v ? kTerms * TERMB : 0);
    if (is_v ? v_mine : k_mine) {
      float probe = 0.f;
#pragma unroll
      for (int it = 0; it < PER; ++it)
#pragma unroll
        for (int j = 0; j < 8; ++j) probe = __builtin_fmaf(stage[it][j], kProbe, probe);
      if (__builtin_expect(!(fabsf(probe) < INFINITY), 0)) {
        unsigned keys = 0;
        int tid_here = tid;
        asm volatile("" : "+v"(tid_here));
#pragma unroll
        for (int it = 0; it < PER; ++it) {
          const int grp = (it * NT + tid_here - (ITEMS >= NT ? 0 : NT - ITEMS)) / D;
          const int first = is_v ? 16 * (grp >> 1) + 4 * (grp & 1) : (it * NT + tid_here) / (D / 8);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const bool odd = !(fabsf(stage[it][j]) < kLargest);
            keys |= odd ? 1u << (first + (is_v ? 8 * (j >> 2) + (j & 3) : 0)) : 0u;
            if (is_v) stage[it][j] = odd ? 0.f : stage[it][j];  // (its weight will be 0)
          }
        }
        if (keys) atomicOr(&odd_keys[(unsigned)h % 3u], keys);
      }
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        if (is_v) {
#pragma unroll
          for (int j = 0; j < 8; ++j) stage[it][j] *= kValueScale;
        }
        uintx4 t[kTerms];
        split8(stage[it], t);
        int at;
        if (is_v) {
          const int vi = it * NT + tid - (ITEMS >= NT ? 0 : NT - ITEMS);
          const int col = vi % D, grp = vi / D;
          at = (((grp >> 1) * DB + col / 32) * 64 + (grp & 1) * 32 + col % 32) * 16;
        } else {
          const int ci = it * NT + tid, row = ci / (D / 8), c = ci % (D / 8);
          at = (c * 32 + (row ^ (c & 7))) * 16;
        }
#pragma unroll
        for (int i = 0; i < kTerms; ++i) *reinterpret_cast<uintx4*>(buf + i * TERMB + at) = t[i];
      }
    }
  };

  // ---- Q: lane (m, hi) keeps q[m][16 ks + 8 hi + j], j = 0..7, as terms
  uintx4 qt[KS][kTerms];
  bool odd_q = false, odd_row = false;  // some row of the unit, this lane's row
  if (tid < 3) odd_keys[tid] = 0;
  if (tid == 3) odd_tiles = 0;
  if (h_begin < h_end) {
    load_k(h_begin, std::false_type{});
    if (FUSED || kBothAhead) load_v(h_begin, std::false_type{});
  }
  {
    float raw[KS][8];
    const float* qrow = reinterpret_cast<const float*>(p.q) + ((int64_t)tok * Hq + head) * D + hi * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const float4 a = *reinterpret_cast<const float4*>(qrow + ks * 16), b = *reinterpret_cast<const float4*>(qrow + ks * 16 + 4);
      raw[ks][0] = a.x; raw[ks][1] = a.y; raw[ks][2] = a.z; raw[ks][3] = a.w;
      raw[ks][4] = b.x; raw[ks][5] = b.y; raw[ks][6] = b.z; raw[ks][7] = b.w;
    }
    if (p.rope_cos) {
      // Rotary embedding at the row's absolute position (Sec. 2), half-split pairs (j, j + D/2): the sine
      // product rounded first, then one fused multiply-add
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks) {
        const float* cs = p.rope_cos + (int64_t)tok * (D / 2) + ks * 16 + hi * 8;
        const float* sn = p.rope_sin + (int64_t)tok * (D / 2) + ks * 16 + hi * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float lo = raw[ks][e], up = raw[ks + KS / 2][e];
          const float tl = up * sn[e], tu = lo * sn[e];
          raw[ks][e] = __builtin_fmaf(lo, cs[e], -tl);
          raw[ks + KS / 2][e] = __builtin_fmaf(up, cs[e], tu);
        }
      }
    }
    float probe = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      split8(raw[ks], qt[ks]);
#pragma unroll
      for (int e = 0; e < 8; ++e) probe = __builtin_fmaf(raw[ks][e], kProbe, probe);
    }
    odd_row = pair_max(fabsf(probe) < INFINITY && p.scale_log2e < kMaxScale ? 0.f : 1.f) != 0.f;
    odd_q = !idle && __any(odd_row);
  }

  floatx16 o[DB];
  float m_run, l_run;
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };
  clear();
  const float sc = p.scale_log2e;

  // lane part of the LDS addresses
  unsigned k_at[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) k_at[i] = (unsigned)((2 * i + hi) * 32 + (m ^ ((2 * i + hi) & 7))) * 16u;

  if (h_begin < h_end) {
    __syncthreads();  // the words above are clear
    put(h_begin, false, stage_k);
    if (!FUSED && !kBothAhead) load_v(h_begin, std::false_type{});
    put(h_begin, true, stage_v);
  }
  floatx16 s;
  auto logits = [&](int h, auto split_tag) __attribute__((always_inline)) {
    const int key0 = first_key(h);
    if constexpr (decltype(split_tag)::value) {
      // the leading products in one sum, the small ones in another
      const unsigned char* buf = smem + (h & 1) * BUFB;
      floatx16 sm;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = sm[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        uintx4 a[kTerms];
#pragma unroll
        for (int i = 0; i < kTerms; ++i)
          a[i] = *reinterpret_cast<const uintx4*>(buf + k_at[ks & 3] + (ks >> 2) * 4096 + i * TERMB);
        sm = mfma16(a[2], qt[ks][1], sm);
        sm = mfma16(a[1], qt[ks][2], sm);
        sm = mfma16(a[2], qt[ks][0], sm);
        sm = mfma16(a[1], qt[ks][1], sm);
        sm = mfma16(a[0], qt[ks][2], sm);
        sm = mfma16(a[1], qt[ks][0], sm);
        sm = mfma16(a[0], qt[ks][1], sm);
        s = mfma16(a[0], qt[ks][0], s);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] += sm[r];
    } else {
      // fp32 instructions, operands from memory: contraction slot hi of step (ks, j) is column 16 ks + 8 hi + j
      // (formed from an opaque lane id, so that nothing is held for this through the loop over the tiles)
      int l2 = l;
      asm volatile("" : "+v"(l2));
      const int hi2 = l2 >> 5, m2 = l2 & 31;
      int row = key0 + m2, t2 = ur.tok(m2), h2 = ur.head(m2);
      if (row > L - 1) row = L - 1;
      if (t2 > C - 1) t2 = C - 1, h2 = G - 1;
      const float* krow = reinterpret_cast<const float*>(row_at(false, row)) + hi2 * 8;
      const float* qrow = reinterpret_cast<const float*>(p.q) + ((int64_t)t2 * Hq + g * G + h2) * D;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll 1
      for (int ks = 0; ks < KS; ++ks) {
        float kv[8], qv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) kv[e] = krow[16 * ks + e], qv[e] = qrow[16 * ks + 8 * hi2 + e];
        if (p.rope_cos) {
          const bool lower = ks < KS / 2;
          const int j0 = 16 * (lower ? ks : ks - KS / 2) + 8 * hi2;
          const float* cs = p.rope_cos + (int64_t)t2 * (D / 2) + j0;
          const float* sn = p.rope_sin + (int64_t)t2 * (D / 2) + j0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float t = qrow[(lower ? D / 2 : 0) + j0 + e] * sn[e];
            qv[e] = __builtin_fmaf(qv[e], cs[e], lower ? -t : t);
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[e], qv[e], s, 0, 0, 0);
      }
    }
  };
  auto softmax = [&](int h, unsigned hide) __attribute__((always_inline)) {  // hide: keys of the tile to leave out
    const int key0 = first_key(h);
    if (__builtin_expect(hide != 0, 0)) {
      int hi_here = hi;  // (opaque copies here and below: what rare code derives from a lane's place is not held through the loop)
      asm volatile("" : "+v"(hi_here));
      const unsigned mine = hide >> (4 * hi_here);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (mine & (1u << (8 * (r >> 2) + (r & 3)))) s[r] = -INFINITY;
    }
    const bool left = WIN && key0 < lb_last && key0 + BN > p.n_sink;  // keys between the sinks and the window
    if (key0 + BN > vis_first || left) {
      // visible inside the tile: keys below rel, and of those (window step) the ones below rel_sink or from rel_lb
      // on; all three are counted from the lane's own first key, 4 * hi
      // (opaque copy of the lane's half: the key offsets below are formed here, not once ahead of the tile loop
      // and then held in registers through it)
      int hi_here = hi;
      asm volatile("" : "+v"(hi_here));
      const int rel = my_vis - key0 - 4 * hi_here;
      const int rel_lb = WIN ? rel - p.window : -1, rel_sink = WIN ? p.n_sink - key0 - 4 * hi_here : 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int kk = 8 * (r >> 2) + (r & 3);  // key offset in the tile, less the lane's 4 * hi
        if (kk >= rel || (WIN && kk < rel_lb && kk >= rel_sink)) s[r] = -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = pair_max(mx) * sc;
    if (__any(mx > m_run + kThresh)) {
      // only rows that asked for it move, so a row's arithmetic never depends on its wave neighbours
      const float m2 = (mx > m_run + kThresh) ? mx : m_run;
      const float alpha = (m2 == -INFINITY) ? 1.f : exp2f(m_run - m2);
      m_run = m2;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], sc, -m_use));
      l_run += s[r];
    }
  };
  // registers 8 tt .. 8 tt + 7 of P^T contract keys 16 tt + 4 hi + {0..3, 8..11}
  auto add_values = [&](int h, auto split_tag) __attribute__((always_inline)) {
    if constexpr (decltype(split_tag)::value) {
      const unsigned char* buf = smem + (h & 1) * BUFB + kTerms * TERMB + l * 16;
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        float px[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) px[j] = s[8 * tt + j];
        uintx4 pt[kTerms];
        split8(px, pt);
#pragma unroll
        for (int db = 0; db < DB; db += 2) {
          uintx4 a[2][kTerms];
#pragma unroll
          for (int i = kTerms - 1; i >= 0; --i)
#pragma unroll
            for (int e = 0; e < 2; ++e) a[e][i] = *reinterpret_cast<const uintx4*>(buf + (tt * DB + db + e) * 1024 + i * TERMB);
#pragma unroll
          for (int i = kTerms - 1; i >= 0; --i)
#pragma unroll
            for (int j = kTerms - 1 - i; j >= 0; --j)
#pragma unroll
              for (int e = 0; e < 2; ++e) o[db + e] = mfma16(a[e][i], pt[j], o[db + e]);
        }
      }
    } else {
      const int key0 = first_key(h);
      int l2 = l;
      asm volatile("" : "+v"(l2));
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += 4) {
        float v[4][DB];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int row = key0 + 2 * r0 + j + 4 * (l2 >> 5);
          if (row > L - 1) row = L - 1;
          const float* vrow = reinterpret_cast<const float*>(row_at(true, row)) + (l2 & 31);
#pragma unroll
          for (int db = 0; db < DB; ++db) v[j][db] = vrow[db * 32];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[j][db], s[r0 + j], o[db], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  constexpr std::true_type by_terms{};
  constexpr std::false_type in_fp32{};
  // (A second wavefront per SIMD that does its O^T one step later, so that the two are never in the softmax together, was
  // 4 % slower; a priority for one of the two changed nothing.)
  unsigned hide = 0;
  auto step = [&](int h, auto old_tag) __attribute__((always_inline)) {
    __syncthreads();  // tile h is in LDS, and nobody reads tile h - 1 any more
    // Short pieces: nothing is fetched or split past the last tile (a piece of two halves spends a tenth of its time on
    // that).  Else the last tile once more, for nobody, which long loops do not notice.
    const bool more = !FUSED || h + 1 < h_end;
    const int hn = h + 1 < h_end ? h + 1 : h;
    const bool work = !idle && first_key(h) < vis_last;  // (else every row is masked)
    const unsigned hide_before = hide;
    hide = __builtin_amdgcn_readfirstlane(odd_keys[(unsigned)h % 3u]);
    if (more) {
      load_k(hn, old_tag);
      if (kBothAhead) load_v(hn, old_tag);
    }
    if (work) logits(h, by_terms);
    if (more) {
      put(h + 1, false, stage_k);
      if (!kBothAhead) load_v(hn, old_tag);
    }
    if (__builtin_expect((hide | hide_before) != 0, 0)) {
      if (tid == 0) {
        if (hide_before) odd_keys[(unsigned)(h + 2) % 3u] = 0;  // tile h - 1's, next used for tile h + 2
        if (hide) {
          const int n = odd_tiles;
          if (n < kOddList) odd_list[n].h = h, odd_list[n].keys = hide;
          odd_tiles = n + 1;
        }
      }
    }
    if (work) {
      softmax(h, hide);
      add_values(h, by_terms);
    }
    if (more) put(h + 1, true, stage_v);
  };
  // (two loops: with the choice between the two sources inside one, every tile of the prefix pays for it, 2.5 %)
  int h = h_begin;
  for (; h < h_end && (!FUSED || is_old(h + 1 < h_end ? h + 1 : h)); ++h) step(h, std::true_type{});
  if (FUSED)
    for (; h < h_end; ++h) step(h, std::false_type{});
  __syncthreads();

  copy_load(copy_r0);  // (in flight while the results leave)

  // ---- keys and rows for the fp32 instructions, and the epilogue: first the rows whose query the terms can hold
  const int n_odd = __builtin_amdgcn_readfirstlane(odd_tiles);
  float unscale = kValueUnscale;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    if (__builtin_expect((n_odd > 0 || pass > 0) && !idle, 0)) {
      const bool whole = pass > 0 || n_odd > kOddList;
      if (whole)
        clear();
      else
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= unscale;
      unscale = 1.f;
      const int n = whole ? h_end - h_begin : n_odd;
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        const int h = whole ? h_begin + i : __builtin_amdgcn_readfirstlane(odd_list[i].h);
        if (first_key(h) >= vis_last) break;  // (tiles ascend)
        logits(h, in_fp32);
        softmax(h, whole ? 0u : ~(unsigned)__builtin_amdgcn_readfirstlane(odd_list[i].keys));
        add_values(h, in_fp32);
      }
    }

    const float l_tot = pair_sum(l_run);
    if (store_ok && odd_row == (pass > 0)) {
      const int64_t n_rows = (int64_t)C * Hq;
      const int64_t row = (int64_t)tok * Hq + head;
      if (p.n_splits == 1) {
        const float inv = unscale / l_tot;
        float* orow = reinterpret_cast<float*>(p.out) + row * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg)
            *reinterpret_cast<float4*>(orow + db * 32 + 8 * rg + 4 * hi) =
                make_float4(o[db][rg * 4 + 0] * inv, o[db][rg * 4 + 1] * inv, o[db][rg * 4 + 2] * inv, o[db][rg * 4 + 3] * inv);
        if (p.lse && hi == 0) p.lse[(int64_t)head * C + tok] = (m_run + log2f(l_tot)) * 0.6931471805599453f;
      } else {
        float* prow = p.part_o + ((int64_t)split * n_rows + row) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg)
            *reinterpret_cast<float4*>(prow + db * 32 + 8 * rg + 4 * hi) =
                make_float4(o[db][rg * 4 + 0] * unscale, o[db][rg * 4 + 1] * unscale, o[db][rg * 4 + 2] * unscale, o[db][rg * 4 + 3] * unscale);
        if (hi == 0) *reinterpret_cast<float2*>(p.part_ml + ((int64_t)split * n_rows + row) * 2) = make_float2(m_run, l_tot);
      }
    }
    if (!odd_q) break;
  }

  copy_store(copy_r0);
  for (int r0 = copy_r0 + kCopyRows; r0 < copy_r1; r0 += kCopyRows) {
    copy_load(r0);
    copy_store(r0);
  }
}

// Rows that the append kernel has appended (rotary embedding) take the instance of short pieces for the shortest only: its first values
// come with the first keys, its loop is slower.  Measured, that / the other instance, rotary embedding, 4 tokens, 32 heads on 8: 1 tile 15.2 /
// 15.6 us, 2 21.9 / 22.2, 3 31.5 / 31.7, 6 51.8 / 51.7, 9 73.1 / 72.4; 64 wide, 64 tokens, 8 heads on 2: 1 tile 11.7 / 11.8, 2 15.8 / 15.7.
template <int D, bool WIN>
static void launch_f32(const AttnParams& p, int waves_per_wg, hipStream_t s) {
  const dim3 grid(padded_grid(p.n_wgs));
  if (waves_per_wg == 8)
    hipLaunchKernelGGL((attn_f32_kernel<D, WIN, 8, false>), grid, dim3(512), 0, s, p);
  else if (p.k_new || p.tiles_per_split <= (D == 64 ? 1 : 3))
    hipLaunchKernelGGL((attn_f32_kernel<D, WIN, 4, true>), grid, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((attn_f32_kernel<D, WIN, 4, false>), grid, dim3(256), 0, s, p);
}

hipError_t launch_attn_f32(const AttnParams& p, int head_dim, int waves_per_wg, hipStream_t s) {
  if (head_dim == 128)
    p.window > 0 ? launch_f32<128, true>(p, waves_per_wg, s) : launch_f32<128, false>(p, waves_per_wg, s);
  else if (head_dim == 64)
    p.window > 0 ? launch_f32<64, true>(p, waves_per_wg, s) : launch_f32<64, false>(p, waves_per_wg, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace kvfold
