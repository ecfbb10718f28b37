// Chunk-prefix attention of small steps, fp32: a workgroup owns one unit (32 packed rows of a KV head) and deals the keys of its
// piece to its wavefronts, as attn_few.hip does in bf16.  The arithmetic is the general fp32 kernel's (attn_f32.hip): operands as
// three bf16 terms, eight products for the logits, six for P V, sums in fp32; keys and queries that the terms cannot hold go
// through the fp32 instructions after the piece's end.
//
// It is for steps in which the general kernel leaves most of its wavefronts without rows (decoding: one of four or eight) and walks a
// piece with one wavefront's chain: split, products, softmax and split again, 8 us per 64 keys.  Here every wavefront has keys of its own
// and nothing to wait for until the results meet in LDS:
//  * K blocks of 32 keys come into LDS of the wavefront's own by direct copies; V comes into registers, whole rows per half-wave (the
//    columns of a matrix instruction's 32 are every fourth or every second one of the head); both a block ahead;
//  * the queries' terms are formed once per workgroup, a share in each wavefront, and read from LDS as they are used;
//  * the split of the next operands stands behind the matrix instructions of these, in an order that the compiler keeps: one
//    wavefront alone issues a vector instruction every 5.2 cycles and hides six of them under a matrix instruction's 32.
// What bounds it: 32 keys of 128-wide rows for each of four wavefronts take a CU 3.6 us, some 37 GB/s from beyond its XCD's L2, so that
// a step wants its keys on many CUs; 30K keys and more are bound by memory.  (That is this loop's rate, not the chip's: 128 wide, the wait for
// a block's values waits for the copies of the next keys as well, which were asked for behind them, and nothing is on its way through
// softmax and P V.  attn_few.hip's blocks come at 46 GB/s a CU.)  Four wavefronts where rows are 128 wide (eight have 256
// registers each and spill: one token on 30K keys 76 us, four 58), eight where they are 64 wide, one workgroup per CU.
// Captured steps, the better form of the general kernel -> this one: 32 heads on 8, one token on 300 / 4187 / 30K keys 15.5 -> 12.5,
// 28.1 -> 19.9, 91.8 -> 58.2 us (4.2 TB/s); 37 tokens on 300 20.0 -> 14.9; 8 heads on 2, one token on 30K 54.4 -> 27.9; 64 wide, 4 on
// 1, 128 tokens on 0 / 384 12.0 -> 7.5, 13.0 -> 10.2.  A fold of 4 x 128 tokens of that shape 50.9 -> 36.1 us.
// Error against 64 bits, relative to the general kernel's at its own split of the keys, 320 steps (1 to 128 tokens on 0 to 20K keys, five
// distributions), geometric means: outputs 0.94 (2-norm and largest), log-sum-exp 0.99.
#include "f32_terms.h"
#include "kvfold_internal.h"
#include "wave_ops.h"

namespace kvfold {

typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(2))) float floatx2;

template <int D, bool WIN, int NW>
__global__ void __launch_bounds__(NW * 64, NW / 4) attn_few_f32_kernel(AttnParams p) {
  constexpr int NT = NW * 64;
  constexpr int ROWB = D * 4, KS = D / 16, DB = D / 32;
  constexpr int BN = 32;  // keys of a block
  constexpr float kThresh = 8.0f;
  typedef __attribute__((ext_vector_type(DB))) float vecv;  // a lane's columns of a V row: DB m .. DB m + DB - 1
  constexpr int OROW = D * 4 + 16;
  constexpr int CH = D / 4;         // 16-byte chunks of a row
  constexpr int RPS = 64 / CH;      // rows of a 1 KiB copy
  constexpr int SLABS = BN / RPS;   // copies per block
  constexpr int BLOCKB = BN * ROWB;
  constexpr int KSW = 8;            // swizzle: pair of chunks ^= row % KSW
  constexpr int kOddList = 32;
  // a K block of each wavefront and the terms of the unit's queries, [ks][term][lane]; then the results, [wavefront][row][D]
  constexpr int SLOTS = NW == 4 ? 2 : 1;
  constexpr int kQueries = NW * SLOTS * BLOCKB, kRings = kQueries + KS * kTerms * 1024, kResults = NW * kRowsPerUnit * OROW;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kRings > kResults ? kRings : kResults];
  __shared__ unsigned odd_rows[KS];  // rows whose queries the terms cannot hold
  __shared__ floatx2 results_ml[NW * kRowsPerUnit];
  __shared__ struct { int b; unsigned keys; } odd_list[NW][kOddList];  // blocks with keys that the terms cannot hold
  const unsigned lds0 = (unsigned)(uintptr_t)((unsigned char __attribute__((address_space(3)))*)smem);
  unsigned char* const results = smem;

  // every line of the arguments is fetched now, in one round trip (they are not in the scalar cache yet)
  asm volatile("" ::"s"(p.q), "s"(p.n_tokens), "s"(p.len_prev), "s"(p.k_new), "s"(p.work_k), "s"(p.by_group.mul), "s"(p.copy_rows));

  const int lid = logical_workgroup(blockIdx.x, gridDim.x, p);
  if (lid >= p.n_wgs) return;
  const int g = (int)quot((unsigned)lid, p.by_wgs_per_kvh);
  const int rem = lid - g * (p.wgs_per_head * p.n_splits);
  const int split = (int)quot((unsigned)rem, p.by_wgs_per_head);
  const int u = p.wgs_per_head - 1 - (rem - split * p.wgs_per_head);  // late units, which see more keys, first

  const int tid = threadIdx.x, l = tid & 63, hi = l >> 5, m = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = p.n_tokens, Hq = p.n_q_heads, G = p.group;
  const int L = (int)p.len_prev + C;
  const int row0 = u * kRowsPerUnit, n_left = C * G - row0, rows = n_left < kRowsPerUnit ? n_left : kRowsPerUnit;
  const int row = row0 + (m < rows ? m : rows - 1);
  const int tok = (int)quot((unsigned)row, p.by_group), head = g * G + row - tok * G;
  const int my_vis = (int)p.len_prev + tok + 1;
  const RowRange rr = workgroup_rows(u, 1, p.units_per_head, p.by_group, C);
  const int vis_first = (int)p.len_prev + rr.row_lo + 1, vis_last = (int)p.len_prev + rr.row_hi + 1;
  const int lb_last = WIN ? vis_last - p.window : 0;  // the largest of the rows' first keys inside the window

  const TileMap tm = tile_map(p.len_prev, rr.row_lo, rr.row_hi, WIN ? p.n_sink : 0, WIN ? p.window : 0);
  const bool fused = p.k_new != nullptr;
  const int chunk0 = fused ? (int)p.len_prev : 0x7fffffff;  // rows from here on are read as handed in
  const int t_begin = split * p.tiles_per_split, t_end = t_begin + p.tiles_per_split < tm.ntiles ? t_begin + p.tiles_per_split : tm.ntiles;
  // Blocks of 32 keys of the logical tiles, and the first key of one; the last block of the last tile may lie beyond every row.
  auto first_key = [&](int b) __attribute__((always_inline)) -> int { return b * BN + (WIN && (b >> 1) >= tm.ns_t ? tm.skip * kTileKeys : 0); };
  const int b_all = 2 * tm.ntiles - (first_key(2 * tm.ntiles - 1) >= vis_last ? 1 : 0), b_end = 2 * t_end < b_all ? 2 * t_end : b_all;

  // The wavefront's blocks: every NW-th of the piece's, in cyclic order from a place that differs from piece to piece and head to
  // head (attn_few.hip).
  const int b_first = 2 * t_begin + w, n_blocks = b_first < b_end ? (int)((unsigned)(b_end - b_first + NW - 1) / (unsigned)NW) : 0;
  int b = b_first + NW * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_blocks) >> 16);

  const unsigned head_bytes = (unsigned)p.capacity * (unsigned)ROWB;  // (below 2^32, as the host checks)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(p.k_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(p.v_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned new_stride = (unsigned)(p.n_kv_heads * ROWB);
  const unsigned char* knew = reinterpret_cast<const unsigned char*>(p.k_new) + (unsigned)g * (unsigned)ROWB;
  const unsigned char* vnew = reinterpret_cast<const unsigned char*>(p.v_new) + (unsigned)g * (unsigned)ROWB;
  // any row; past the last one: the last one (and masked)
  auto row_at = [&](bool is_v, int r) __attribute__((always_inline)) -> const unsigned char* {
    r = r < L ? r : L - 1;
    const bool nw = r >= chunk0;
    return (nw ? (is_v ? vnew : knew) : (is_v ? vbase : kbase)) + (unsigned)(r - (nw ? chunk0 : 0)) * (nw ? new_stride : (unsigned)ROWB);
  };
  // Blocks whose rows all exist and lie on one side of the old cache's end: one base, one stride.
  auto plain = [&](int b) __attribute__((always_inline)) -> bool {
    const int first = first_key(b), last = first + BN - 1;
    return last < L && (last < chunk0 || first >= chunk0);
  };

  // K blocks come into LDS of the wavefront's own, the next one as soon as S^T is formed, in an order of chunks that leaves the reads of a fragment free of bank
  // conflicts: lane (m, hi) of the fragment ks holds row m, columns 16 ks + 8 hi + j.
  const unsigned my_lds = lds0 + (unsigned)(w * SLOTS * BLOCKB);
  const int lrow = l / CH;  // + i * RPS for copy i
  auto fetch_k = [&](int b, int slot) __attribute__((always_inline)) {
    const unsigned lds = my_lds + (unsigned)(slot * BLOCKB), chunk = (unsigned)((l % CH) ^ 2 * lrow);
    const int key0 = first_key(b);
    if (__builtin_expect(plain(b), 1)) {
      const bool nw = key0 >= chunk0;
      const unsigned stride = nw ? new_stride : (unsigned)ROWB;
      const unsigned char* base = (nw ? knew : kbase) + (uint64_t)(unsigned)(key0 - (nw ? chunk0 : 0)) * stride;
      unsigned off = (unsigned)lrow * stride;
#pragma unroll
      for (int i = 0; i < SLABS; ++i) {
        dma16(base, off + (chunk ^ (unsigned)(2 * ((i * RPS) % KSW))) * 16, lds + (unsigned)(i * 1024));
        off += (unsigned)RPS * stride;
      }
    } else {
#pragma unroll 1
      for (int i = 0; i < SLABS; ++i) {
        int r = key0 + lrow + i * RPS;
        r = r < L ? r : L - 1;
        const unsigned c16 = (chunk ^ (unsigned)(2 * ((i * RPS) % KSW))) * 16;
        if (r >= chunk0)
          dma16(knew, (unsigned)(r - chunk0) * new_stride + c16, lds + (unsigned)(i * 1024));
        else
          dma16(kbase, (unsigned)r * (unsigned)ROWB + c16, lds + (unsigned)(i * 1024));
      }
    }
  };
  unsigned k_at[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) k_at[i] = my_lds + (unsigned)(m * ROWB + (((2 * i + hi) ^ (m % KSW)) * 32));
  auto read_k = [&](int slot, int ks, int e) __attribute__((always_inline)) -> floatx4 { return *LDS_PTR(const floatx4, k_at[ks & 3] + (unsigned)(slot * BLOCKB + (ks >> 2) * 256 + e * 16)); };

  // V values come into registers as they lie: lane (m, hi) holds columns DB m + db of the keys that registers 8 tt + j of S^T stand for in
  // its half, 16 tt + 4 hi + {0..3, 8..11}: whole rows per half-wave, and what is column m of the matrix instruction's block db is
  // column DB m + db of the head.
  vecv vr[16];
  auto load_v = [&](int b, int tt) __attribute__((always_inline)) {
    const int key0 = first_key(b);
    const unsigned lane = (unsigned)(m * DB * 4);
    if (__builtin_expect(plain(b), 1)) {
      const bool nw = key0 >= chunk0;
      const unsigned stride = nw ? new_stride : (unsigned)ROWB;
      const unsigned char* base = (nw ? vnew : vbase) + (uint64_t)(unsigned)(key0 + 16 * tt - (nw ? chunk0 : 0)) * stride;
      const unsigned off = lane + (unsigned)(4 * hi) * stride;
#pragma unroll
      for (int j = 0; j < 8; ++j) vr[8 * tt + j] = *reinterpret_cast<const vecv*>(base + (off + (unsigned)(8 * (j >> 2) + (j & 3)) * stride));
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) vr[8 * tt + j] = *reinterpret_cast<const vecv*>(row_at(true, key0 + 16 * tt + 4 * hi + 8 * (j >> 2) + (j & 3)) + lane);
    }
  };
  if (n_blocks > 0) {
    fetch_k(b, 0);
    load_v(b, 0);
    load_v(b, 1);
  }

  // ---- Q as terms, dealt to the wavefronts by contraction steps: lane (m, hi) splits q[m][16 ks + 8 hi + j], j = 0..7
  const unsigned q_lds = lds0 + (unsigned)(kQueries + l * 16);
  for (int ks = w; ks < KS; ks += NW) {
    const int at = 16 * ks + 8 * hi;
    const float* qrow = reinterpret_cast<const float*>(p.q) + ((int64_t)tok * Hq + head) * D;
    float x[8];
    *reinterpret_cast<floatx4*>(x) = *reinterpret_cast<const floatx4*>(qrow + at);
    *reinterpret_cast<floatx4*>(x + 4) = *reinterpret_cast<const floatx4*>(qrow + at + 4);
    if (p.rope_cos) {
      // rotary embedding at the row's absolute position, as in attn_f32.hip
      const bool lower = ks < KS / 2;
      const int j0 = lower ? at : at - D / 2;
      const float* cs = p.rope_cos + (int64_t)tok * (D / 2) + j0;
      const float* sn = p.rope_sin + (int64_t)tok * (D / 2) + j0;
      const float* other = qrow + (lower ? D / 2 : 0) + j0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float t = other[e] * sn[e];
        x[e] = __builtin_fmaf(x[e], cs[e], lower ? -t : t);
      }
    }
    float probe = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) probe = __builtin_fmaf(x[e], kProbe, probe);
    uintx4 t[kTerms];
    split8(x, t);
#pragma unroll
    for (int i = 0; i < kTerms; ++i) *LDS_PTR(uintx4, q_lds + (unsigned)((ks * kTerms + i) * 1024)) = t[i];
    const uint64_t odd = __ballot(!(fabsf(probe) < INFINITY && p.scale_log2e < kMaxScale));
    if (l == 0) odd_rows[ks] = (unsigned)odd | (unsigned)(odd >> 32);
  }
  __syncthreads();
  bool odd_row;
  {
    unsigned odd = 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) odd |= odd_rows[ks];
    odd_row = (odd >> m) & 1;
  }
  const bool odd_q = __any(odd_row);

  floatx16 o[DB], s;
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

  auto softmax = [&](int b, unsigned hide) __attribute__((always_inline)) {  // hide: keys of the block to leave out
    const int key0 = first_key(b);
    if (__builtin_expect(hide != 0, 0)) {
      const unsigned mine = hide >> (4 * hi);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (mine & (1u << (8 * (r >> 2) + (r & 3)))) s[r] = -INFINITY;
    }
    const bool left = WIN && key0 < lb_last && key0 + BN > p.n_sink;  // keys between the sinks and the window
    if (key0 + BN > vis_first || left) {
      const int rel = my_vis - key0 - 4 * hi;
      const int rel_lb = WIN ? rel - p.window : -1, rel_sink = WIN ? p.n_sink - key0 - 4 * hi : 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int kk = 8 * (r >> 2) + (r & 3);
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

  int n_odd = 0;
#pragma unroll 1
  for (int i = 0; i < n_blocks; ++i) {
    const int nb = i + 1 < n_blocks ? (b + NW < b_end ? b + NW : b_first) : b;  // (after the last one: it once more, for nobody)
    // The block's keys have arrived: vector memory loads return in order, and the first of its values, whose register is asked for here, was
    // loaded behind them.  (How many loads the compiler makes of the values is its own affair: nothing counts them.)
    asm volatile("" : "+v"(vr[0])::"memory");
    const int slot = SLOTS == 2 ? i & 1 : 0;
    if (SLOTS == 2 && i + 1 < n_blocks) fetch_k(nb, slot ^ 1);
    floatx4 kr[2];
    uintx4 qt[kTerms];
    auto read_q = [&](int ks, int i) __attribute__((always_inline)) { qt[i] = *LDS_PTR(const uintx4, q_lds + (unsigned)((ks * kTerms + i) * 1024)); };
#pragma unroll
    for (int e = 0; e < 2; ++e) kr[e] = read_k(slot, 0, e);
#pragma unroll
    for (int i = kTerms - 1; i >= 0; --i) read_q(0, i);
    // The split of the next 16 columns goes behind the matrix instructions of these, a pair of values behind every second one, in an
    // order that the compiler keeps.
    floatx16 sm;
    float probe_k = 0.f, probe_v = 0.f;
    uintx4 a[2][kTerms];
    auto split_k = [&](int ks, int j) __attribute__((always_inline)) {
      const float x = kr[j >> 1][2 * (j & 1)], y = kr[j >> 1][2 * (j & 1) + 1];
      probe_k = __builtin_fmaf(x, kProbe, probe_k);
      probe_k = __builtin_fmaf(y, kProbe, probe_k);
      split2(x, y, a[ks & 1], j);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) split_k(0, j);
#pragma unroll
    for (int e = 0; e < 2; ++e) kr[e] = read_k(slot, 1, e);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      constexpr int kOfK[8] = {1, 0, 2, 1, 0, 2, 1, 0}, kOfQ[8] = {2, 2, 1, 1, 1, 0, 0, 0};
      constexpr floatx16 zero = {};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uintx4 &ka = a[ks & 1][kOfK[i]], &qa = qt[kOfQ[i]];
        if (i < 7)
          sm = mfma16(ka, qa, ks + i == 0 ? zero : sm);
        else
          s = mfma16(ka, qa, ks == 0 ? zero : s);
        if (ks + 1 < KS) {
          if (i % 2 == 0) split_k(ks + 1, i / 2);
          if (i == 1) read_q(ks + 1, 2);
          if (i == 4) read_q(ks + 1, 1);
          if (i == 7) read_q(ks + 1, 0);
          if (ks + 2 < KS && (i == 3 || i == 7)) kr[i >> 2] = read_k(slot, ks + 2, i >> 2);
        } else {
#pragma unroll
          for (int j = 2 * i; j < 2 * i + 2; ++j)
#pragma unroll
            for (int db = 0; db < DB; ++db) probe_v = __builtin_fmaf(vr[j][db], kProbe, probe_v);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (SLOTS == 1 && i + 1 < n_blocks) fetch_k(nb, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] += sm[r];

    unsigned hide = 0;
    if (__builtin_expect(__any(!(fabsf(probe_k) < INFINITY && fabsf(probe_v) < INFINITY)), 0)) {
      const uint64_t odd_k = __ballot(!(fabsf(probe_k) < INFINITY));  // (a lane's values are of one key)
      hide = (unsigned)odd_k | (unsigned)(odd_k >> 32);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        bool odd = false;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const bool one = !(fabsf(vr[j][db]) < kLargest);
          odd = odd || one;
          vr[j][db] = one ? 0.f : vr[j][db];  // (its weight will be 0)
        }
        const uint64_t lanes = __ballot(odd);
        const int first = 16 * (j >> 3) + 8 * ((j >> 2) & 1) + (j & 3);
        hide |= ((unsigned)lanes ? 1u << first : 0u) | ((unsigned)(lanes >> 32) ? 16u << first : 0u);
      }
      if (hide) {
        if (l == 0 && n_odd < kOddList) odd_list[w][n_odd].b = b, odd_list[w][n_odd].keys = hide;
        ++n_odd;
      }
    }
    softmax(b, hide);

    // registers 8 tt .. 8 tt + 7 of P^T contract keys 16 tt + 4 hi + {0..3, 8..11}
    uintx4 pt[2][kTerms];
#pragma unroll
    for (int j = 0; j < 8; ++j) split2(s[2 * j], s[2 * j + 1], pt[j >> 2], j & 3);
    auto split_v = [&](int t, int j) __attribute__((always_inline)) {  // t: 16-key half, 32-column block
      const int key = 8 * (t / DB) + 2 * j;
      split2(vr[key][t % DB] * kValueScale, vr[key + 1][t % DB] * kValueScale, a[t & 1], j);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) split_v(0, j);
#pragma unroll
    for (int t = 0; t < 2 * DB; ++t) {
      constexpr int kOfV[6] = {2, 1, 1, 0, 0, 0}, kOfP[6] = {0, 1, 0, 2, 1, 0};
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        o[t % DB] = mfma16(a[t & 1][kOfV[i]], pt[t / DB][kOfP[i]], o[t % DB]);
        if (t + 1 < 2 * DB && i < 4) split_v(t + 1, i);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    load_v(nb, 0);
    load_v(nb, 1);
    b = nb;
  }

  // ---- keys and rows for the fp32 instructions; the wavefronts' results meet in LDS: first the rows whose query the terms can hold
  wait_vm<0>();
  __syncthreads();  // the K blocks are used up
  float unscale = kValueUnscale;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    if (__builtin_expect(n_odd > 0 || pass > 0, 0)) {
      const bool whole = pass > 0 || n_odd > kOddList;
      if (whole)
        clear();
      else
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= unscale;
      unscale = 1.f;
      __threadfence_block();  // the list is lane 0's
      const int n = whole ? n_blocks : n_odd;
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        const int bb = whole ? b_first + NW * i : __builtin_amdgcn_readfirstlane(odd_list[w][i].b);
        const unsigned hide = whole ? 0u : ~(unsigned)__builtin_amdgcn_readfirstlane(odd_list[w][i].keys);
        // contraction slot hi of step (ks, j) is column 16 ks + 8 hi + j
        const float* krow = reinterpret_cast<const float*>(row_at(false, first_key(bb) + m)) + hi * 8;
        const float* qrow = reinterpret_cast<const float*>(p.q) + ((int64_t)tok * Hq + head) * D;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks) {
          float kv[8], qv[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) kv[e] = krow[16 * ks + e], qv[e] = qrow[16 * ks + 8 * hi + e];
          if (p.rope_cos) {
            const bool lower = ks < KS / 2;
            const int j0 = 16 * (lower ? ks : ks - KS / 2) + 8 * hi;
            const float* cs = p.rope_cos + (int64_t)tok * (D / 2) + j0;
            const float* sn = p.rope_sin + (int64_t)tok * (D / 2) + j0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float t = qrow[(lower ? D / 2 : 0) + j0 + e] * sn[e];
              qv[e] = __builtin_fmaf(qv[e], cs[e], lower ? -t : t);
            }
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[e], qv[e], s, 0, 0, 0);
        }
        softmax(bb, hide);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const vecv v = *reinterpret_cast<const vecv*>(row_at(true, first_key(bb) + 8 * (r >> 2) + (r & 3) + 4 * hi) + m * DB * 4);
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[db], s[r], o[db], 0, 0, 0);
        }
      }
    }
    const float l_tot = pair_sum(l_run);
    if (odd_row == (pass > 0)) {
      // rows r of the matrix instruction's blocks are columns DB r .. DB r + DB - 1
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        vecv x;
#pragma unroll
        for (int db = 0; db < DB; ++db) x[db] = o[db][r] * unscale;
        *reinterpret_cast<vecv*>(results + (w * kRowsPerUnit + m) * OROW + (8 * (r >> 2) + 4 * hi + (r & 3)) * DB * 4) = x;
      }
      if (hi == 0) results_ml[w * kRowsPerUnit + m] = floatx2{m_run, l_tot};
    }
    if (!odd_q) break;
  }

  // ---- fused append: this workgroup's share of the chunk's rows, 16 bytes of a K row and of the V row per thread and turn, loaded here
  // and stored behind the results
  constexpr int CPR = ROWB / 16, kCopyRows = NT / CPR;
  const int copy_r0 = fused ? rem * p.copy_rows : 0;
  const int copy_r1 = fused ? (copy_r0 + p.copy_rows < C ? copy_r0 + p.copy_rows : C) : 0;
  floatx4 copy_k = {}, copy_v = {};
  auto copy_load = [&](int r0) __attribute__((always_inline)) {
    const int r = r0 + tid / CPR;
    if (r < copy_r1) {
      const unsigned off = (unsigned)r * new_stride + (unsigned)(tid % CPR) * 16u;
      copy_k = *reinterpret_cast<const floatx4*>(knew + off);
      copy_v = *reinterpret_cast<const floatx4*>(vnew + off);
    }
  };
  auto copy_store = [&](int r0) __attribute__((always_inline)) {
    const int r = r0 + tid / CPR;
    if (r < copy_r1) {
      const unsigned off = (unsigned)(chunk0 + r) * (unsigned)ROWB + (unsigned)(tid % CPR) * 16u;
      __builtin_nontemporal_store(copy_k, reinterpret_cast<floatx4*>(const_cast<unsigned char*>(kbase) + off));
      __builtin_nontemporal_store(copy_v, reinterpret_cast<floatx4*>(const_cast<unsigned char*>(vbase) + off));
    }
  };
  copy_load(copy_r0);
  __syncthreads();

  constexpr int V = D / 4;  // 16-byte column vectors of a row
  const int c = tid % V;
  const int64_t n_rows = (int64_t)C * Hq;
#pragma unroll 1
  for (int r = tid / V; r < rows; r += NT / V) {
    floatx2 ml[NW];
    float M = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      ml[ww] = results_ml[ww * kRowsPerUnit + r];
      M = fmaxf(M, ml[ww].x);
    }
    float sum = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(results + (ww * kRowsPerUnit + r) * OROW + c * 16);
      const bool none = ml[ww].y == 0.f;  // it saw no visible key, and its O may be NaN: 0 times a value that is not finite
      const float f = none ? 0.f : __builtin_amdgcn_exp2f(ml[ww].x - M);
      sum += f * ml[ww].y;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(f, none ? 0.f : x[e], acc[e]);
    }
    const int t = (int)quot((unsigned)(row0 + r), p.by_group), h = g * G + row0 + r - t * G;
    const int64_t at = (int64_t)t * Hq + h;
    if (p.n_splits == 1) {
      const float inv = 1.f / sum;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] *= inv;
      *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + at * D + c * 4) = acc;
      if (p.lse && c == 0) p.lse[(int64_t)h * C + t] = (M + log2f(sum)) * 0.6931471805599453f;
    } else {
      *reinterpret_cast<floatx4*>(p.part_o + ((int64_t)split * n_rows + at) * D + c * 4) = acc;
      if (c == 0) *reinterpret_cast<floatx2*>(p.part_ml + ((int64_t)split * n_rows + at) * 2) = floatx2{M, sum};
    }
  }

  copy_store(copy_r0);
  for (int r0 = copy_r0 + kCopyRows; r0 < copy_r1; r0 += kCopyRows) {
    copy_load(r0);
    copy_store(r0);
  }
}

template <int D, int NW>
static void launch_few_f32(const AttnParams& p, hipStream_t s) {
  const dim3 grid(padded_grid(p.n_wgs));
  if (p.window > 0)
    hipLaunchKernelGGL((attn_few_f32_kernel<D, true, NW>), grid, dim3(NW * 64), 0, s, p);
  else
    hipLaunchKernelGGL((attn_few_f32_kernel<D, false, NW>), grid, dim3(NW * 64), 0, s, p);
}

hipError_t launch_attn_few_f32(const AttnParams& p, int head_dim, hipStream_t s) {
  if (head_dim == 128)
    launch_few_f32<128, 4>(p, s);
  else if (head_dim == 64)
    launch_few_f32<64, 8>(p, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace kvfold
