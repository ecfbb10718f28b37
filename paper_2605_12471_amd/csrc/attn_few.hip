// Chunk-prefix attention of small steps, bf16: a workgroup owns one unit (32 packed rows of a KV head) and deals the keys of its
// piece to its wavefronts.  The arithmetic and its rounding points are the general bf16 kernel's (attn_bf16.hip): queries scaled by
// scale * log2(e) and rounded once more, P = 2^(S - m) rounded to bf16 for P V, row sums in fp32 from the unrounded P, the reference
// m stale by at most 2^16.
//
// Two kinds of step are for it.  Few rows (C G <= 32, a few tokens at a time, every key visible up to the row's own position; at most 16 rows but for
// long ranges of one or two KV heads, and all of them 64 wide, have a kernel of their own by now, attn_decode.hip; the figures of one token below are from before) read every key once and compute next to nothing: they are bound by memory when the cache is long and by what a launch does
// once when it is short.  A few units per KV head on not too many keys, or under a window, are bound by the chain of a wavefront: the
// general kernel walks a piece tile by tile with its four wavefronts side by side on four units, behind a software pipeline whose start
// and code cost more than a short step's work, and needs a split and its merge to fill the chip.  Here
//  * the keys of a workgroup's piece are dealt to its four or eight wavefronts in blocks of 32, and each runs alone: its K and V block
//    come into LDS of its own (16 KB at D = 128; 128 KB a CU with two workgroups of four or one of eight), so there is no barrier
//    until the results are merged through LDS;
//  * the next K block is fetched as soon as S^T is formed, the next V block after O^T: eight wavefronts per CU, each with up
//    to 16 KB in flight, are more than memory can deliver;
//  * the loop is not unrolled or pipelined: code that runs once is fetched at about 3 bytes per ns.
// The price: every unit brings its own copy of each K and V block into LDS, 16 KB where a general workgroup shares them among
// four or eight units.  Eight blocks of 128-wide rows take a full CU 1.45 us (1.15 in the fit to whole steps, plan_key_waves()), so grids of
// more than two workgroups per CU stay with the general kernel (choose_plan()), and the units of a piece belong on one XCD, whose L2 has the
// rows for all of them (xcd_share_log2()).
// One token, 32 heads on 8, D = 128, whole step, general kernel -> this one: 1K keys 12.5 -> 11.8 us (unsplit, one launch
// instead of two), 4K 15.6 -> 13.5, 16K 23.0 -> 18.8, 32K 33.5 -> 29.8, 128K 102.5 -> 95 us (5.9 TB/s; a plain streaming
// read gets 5.8 to 6.2).  With the start in 32-bit arithmetic, the faster merge and pieces of even numbers of tiles: 1K 9.4 us, 4K
// 10.5, 8K 13.0, 128K 93.5.  At 4K keys that is two dependent launches, 7.6 and 3.0 us, of which the rows themselves would
// take 3.  Several units, general kernel -> eight wavefronts: 128 tokens on 1000 keys 18.9 -> 12.4 us, 256 on 300 15.9 -> 11.0, 256 on
// 2000 26.9 -> 19.4; window 4 + 1020, 256 tokens 18.9 -> 12.5; four wavefronts, 16 tokens on 4187 keys 15.9 -> 14.1.  Inside the
// kernel, the window step, 12.6 us: 1.6 to the first block, 7.8 for the five or six blocks of a wavefront, 1 until the last is
// through, 2 for the results through LDS.
// (The last workgroup of a unit to merge its pieces, as in meet.h, gains nothing with 32 rows: 89 shapes, both precisions, 0.999 of the time, 64 wide in
// fp32 0.94 to 0.98, 128 wide up to 1.12.)
#include "append_rows.h"
#include "kvfold_internal.h"
#include "wave_ops.h"

namespace kvfold {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short short4_;
typedef __attribute__((ext_vector_type(8))) short short8_;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) unsigned uintx4;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(2))) float floatx2;

template <int D, int NW>
constexpr int few_lds_bytes() {
  const int rings = NW * 2 * 32 * D * 2, results = NW * kRowsPerUnit * (D * 4 + 16) + NW * kRowsPerUnit * 8;
  return rings > results ? rings : results;
}

// ROT (several units per KV head, rotary embedding, rows read as handed in): the workgroups that read a row are many, and each rotates its
// own copy, in LDS, as it comes to the block, and the rows of the chunk that it appends; the arithmetic is the append kernel's, and so are
// the bits.  That kernel's launch against 0.3 to 1 us in each block with rows of the chunk: 32 heads on 8, 99 tokens on 189 keys
// 12.2 -> 11.3 us, 64 wide, 128 on 128 8.85 -> 7.42 (attention_appends() has the limits).  An instance of its own, for the registers that it takes.
// 64 wide: at most 128 registers, so that a CU has room for two workgroups of eight wavefronts, on which the plan counts; a row's chunks are
// rotated one after the other for that.  With 142 registers steps of more than 256 workgroups took two rounds: 430 shapes, those 78 of
// them 1.11 of the general kernel's time, now 0.96 (89 tokens on 7K keys, 32 heads on 8: 24.4 -> 20.4 us), the others 0.74 as before.
template <int D, int NW, bool WIN, bool MULTI, bool ROT>
__global__ void __launch_bounds__(NW * 64, D == 64 ? 4 : 2) attn_few_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned lds0 = (unsigned)(uintptr_t)((unsigned char __attribute__((address_space(3)))*)smem);
  constexpr int NT = NW * 64;
  constexpr int CH = D / 8, ROWB = D * 2, KS = D / 16, DB = D / 32;
  constexpr int BLOCKB = 32 * ROWB;         // a K or V block
  constexpr int RPS = 64 / CH;              // rows of a 1 KiB copy
  constexpr int SLABS = 32 / RPS;           // copies per block
  constexpr int KSW = CH < 16 ? CH : 16;    // K swizzle: chunk ^= row % KSW
  constexpr int VSW = CH / 4;               // V swizzle: chunk ^= (row & 3) * VSW
  constexpr float kStale = 16.0f;           // log2 units

  // every line of the arguments is fetched now, in one round trip (they are not in the scalar cache yet)
  asm volatile("" ::"s"(p.q), "s"(p.n_tokens), "s"(p.len_prev), "s"(p.k_new), "s"(p.work_k), "s"(p.by_group.mul), "s"(p.copy_rows));

  const int lid = logical_workgroup(blockIdx.x, gridDim.x, p);
  if (lid >= p.n_wgs) return;
  const int g = (int)quot((unsigned)lid, p.by_wgs_per_kvh);
  const int rem = lid - g * (MULTI ? p.wgs_per_head * p.n_splits : p.n_splits);  // one workgroup per KV head, piece and unit
  const int split = MULTI ? (int)quot((unsigned)rem, p.by_wgs_per_head) : rem;
  const int u = MULTI ? p.wgs_per_head - 1 - (rem - split * p.wgs_per_head) : 0;  // late units, which see more keys, first

  const int tid = threadIdx.x, l = tid & 63, hi = l >> 5, m = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = p.n_tokens, Hq = p.n_q_heads, G = p.group;
  const int n_packed = C * G, row0 = u * kRowsPerUnit;  // the KV head's packed rows: row j is token j / G, head j % G of the group
  const int rows = !MULTI || n_packed - row0 < kRowsPerUnit ? n_packed - row0 : kRowsPerUnit;
  const int row = row0 + (m < rows ? m : rows - 1);
  const int tok = (int)quot((unsigned)row, p.by_group), head = g * G + row - tok * G;
  const int my_vis = (int)p.len_prev + tok + 1;
  RowRange rr = {0, C - 1};
  if (MULTI) rr = workgroup_rows(u, 1, p.units_per_head, p.by_group, C);
  const int vis_first = (int)p.len_prev + rr.row_lo + 1, vis_last = (int)p.len_prev + rr.row_hi + 1;
  const int lb_last = WIN ? vis_last - p.window : 0;  // the largest of the rows' first keys inside the window

  TileMap tm = {0, 0, (int)(((unsigned)vis_last + kTileKeys - 1) / kTileKeys)};
  if (MULTI) tm = tile_map(p.len_prev, rr.row_lo, rr.row_hi, WIN ? p.n_sink : 0, WIN ? p.window : 0);
  const bool fused = p.k_new != nullptr;
  const KeyRange kr = key_range(tm, split, p.tiles_per_split, p.len_prev, C, fused);
  // Blocks of 32 keys of the logical tiles, and the first key of one; the last block of the last tile may lie beyond every row.
  auto first_key = [&](int b) __attribute__((always_inline)) -> int { return b * 32 + (WIN && (b >> 1) >= tm.ns_t ? tm.skip * kTileKeys : 0); };
  const int b_all = MULTI ? 2 * tm.ntiles - (first_key(2 * tm.ntiles - 1) >= vis_last ? 1 : 0) : (int)(((unsigned)vis_last + 31) / 32);
  const int b_end = 2 * kr.t_end < b_all ? 2 * kr.t_end : b_all;

  const unsigned head_bytes = (unsigned)p.capacity * (unsigned)ROWB;  // (below 2^32, as the host checks)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(p.k_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(p.v_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned new_stride = (unsigned)(p.n_kv_heads * ROWB);
  const unsigned char* knew = reinterpret_cast<const unsigned char*>(p.k_new) + (unsigned)g * (unsigned)ROWB;
  const unsigned char* vnew = reinterpret_cast<const unsigned char*>(p.v_new) + (unsigned)g * (unsigned)ROWB;

  // Blocks whose rows all exist and lie on one side of the old cache's end (one unit: before it) are plain; else each row comes from the cache or the
  // chunk, or is redirected to the piece's last row (and masked).
  auto plain = [&](int b) __attribute__((always_inline)) -> bool {
    const unsigned first = (unsigned)first_key(b), last = first + 31;
    return last <= kr.row_lim && (last < kr.chunk_row0 || (MULTI && first >= kr.chunk_row0));
  };
  const unsigned my_lds = lds0 + (unsigned)(w * 2 * BLOCKB);
  const int lrow = l / CH;  // + i * RPS for copy i
  auto fetch = [&](bool is_v, int b) __attribute__((always_inline)) {
    const unsigned lds = my_lds + (is_v ? BLOCKB : 0);
    const unsigned chunk = is_v ? (unsigned)((l % CH) ^ ((lrow & 3) * VSW)) : (unsigned)((l % CH) ^ (lrow % KSW));
    const int key0 = first_key(b);
    if (!MULTI && __builtin_expect(plain(b), 1)) {  // (one base for all blocks, constant distances: fewer instructions ahead of the first fetch)
      const unsigned char* base = is_v ? vbase : kbase;
      const unsigned off = (unsigned)(b * 32 + lrow) * ROWB;
#pragma unroll
      for (int i = 0; i < SLABS; ++i)
        dma16(base, off + (unsigned)(i * RPS * ROWB) + ((is_v ? chunk : chunk ^ (unsigned)((i * RPS) % KSW)) * 16), lds + (unsigned)(i * 1024));
    } else if (MULTI && __builtin_expect(plain(b), 1)) {
      const bool nw = (unsigned)key0 >= kr.chunk_row0;  // rows of the chunk as handed in (fused append)
      const unsigned stride = nw ? new_stride : (unsigned)ROWB;
      const unsigned char* base = (nw ? (is_v ? vnew : knew) : (is_v ? vbase : kbase)) + (uint64_t)((unsigned)key0 - (nw ? kr.chunk_row0 : 0u)) * stride;
      unsigned off = (unsigned)lrow * stride;
#pragma unroll
      for (int i = 0; i < SLABS; ++i) {
        dma16(base, off + ((is_v ? chunk : chunk ^ (unsigned)((i * RPS) % KSW)) * 16), lds + (unsigned)(i * 1024));
        off += (unsigned)RPS * stride;
      }
    } else {
#pragma unroll 1
      for (int i = 0; i < SLABS; ++i) {
        const DmaRow src = dma_row(kr, (int)((unsigned)key0 / kTileKeys), (int)((unsigned)key0 % kTileKeys) + lrow + i * RPS);
        const unsigned c16 = (is_v ? chunk : chunk ^ (unsigned)((i * RPS) % KSW)) * 16;
        if (src.from_chunk)
          dma16(is_v ? vnew : knew, src.row * new_stride + c16, lds + (unsigned)(i * 1024));
        else
          dma16(is_v ? vbase : kbase, src.row * (unsigned)ROWB + c16, lds + (unsigned)(i * 1024));
      }
    }
  };

  // The wavefront's blocks, every NW-th of the piece's, in cyclic order from a place that differs from piece to piece and
  // head to head: pieces and heads lie powers of two apart, and workgroups in step would ask the same few memory channels
  // for their rows.
  const int b_first = 2 * kr.t_begin + w, n_blocks = b_first < b_end ? (int)((unsigned)(b_end - b_first + NW - 1) / (unsigned)NW) : 0;
  int b = b_first + NW * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_blocks) >> 16);
  // A chunk whose rows need work on their way (append_rows.h): this workgroup, the only one of its piece, appends those it is going
  // to read, ahead of any block that holds some.
  int work_r0 = 0, work_r1 = 0;
  if (!MULTI && __builtin_expect(p.work_k && kr.t_begin < kr.t_end, 0)) {
    work_r0 = kr.t_begin * kTileKeys - (int)p.len_prev;
    if (work_r0 < 0) work_r0 = 0;
    work_r1 = (int)kr.row_lim + 1 - (int)p.len_prev;
  }
  const bool block_first = work_r1 <= work_r0 || b * 32 + 32 <= (int)p.len_prev;
  if (block_first && n_blocks > 0) {
    fetch(false, b);
    fetch(true, b);
  }

  // ---- Q, scaled; lane (m, hi) holds q[m][16 ks + 8 hi + j]
  bf16x8 qf[KS];
  {
    const __bf16* qrow = reinterpret_cast<const __bf16*>(p.q) + ((int64_t)tok * Hq + head) * D + hi * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 16);
    if (p.rope_cos) {
      // rotary embedding, bit for bit that of a caller who rotates and stores bf16 (see attn_bf16.hip)
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks) {
        const float* cs = p.rope_cos + (int64_t)tok * (D / 2) + ks * 16 + hi * 8;
        const float* sn = p.rope_sin + (int64_t)tok * (D / 2) + ks * 16 + hi * 8;
        const bf16x8 lo = qf[ks], up = qf[ks + KS / 2];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float tl = (float)up[e] * sn[e], tu = (float)lo[e] * sn[e];
          qf[ks][e] = (__bf16)__builtin_fmaf((float)lo[e], cs[e], -tl);
          qf[ks + KS / 2][e] = (__bf16)__builtin_fmaf((float)up[e], cs[e], tu);
        }
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[ks][e] = (__bf16)((float)qf[ks][e] * p.scale_log2e);
  }

  if (!MULTI && __builtin_expect(work_r1 > work_r0, 0)) {
    append_work_rows<D>(reinterpret_cast<const unsigned char*>(p.work_k) + g * ROWB, reinterpret_cast<const unsigned char*>(p.work_v) + g * ROWB, new_stride,
                        const_cast<unsigned char*>(kbase) + (uint64_t)p.len_prev * ROWB, const_cast<unsigned char*>(vbase) + (uint64_t)p.len_prev * ROWB,
                        p.rope_cos, p.rope_sin, p.work_qmax, work_r0, work_r1, tid);
    __syncthreads();
    if (!block_first && n_blocks > 0) {
      fetch(false, b);
      fetch(true, b);
    }
  }

  // ---- fused append: this workgroup's share of the chunk's rows, 16 bytes per thread and turn.  One unit per KV head: here, ahead of the
  // output, which may lie on them.  Several: loaded here, a K and a V row at a time, and stored behind the results.  (The one unit's
  // behind its results as well: one token on 17 to 12K keys 1.005 of the time, with the rotary embedding 1.011.)
  if (!MULTI && fused) {
    const int r0 = split * p.copy_rows, r1 = r0 + p.copy_rows < C ? r0 + p.copy_rows : C;
    const int nvec = (r1 > r0 ? r1 - r0 : 0) * CH;
    for (int i = tid; i < 2 * nvec; i += NT) {
      const bool is_v = i >= nvec;
      const int e = is_v ? i - nvec : i, r = r0 + e / CH, c = e % CH;
      const uintx4 x = *reinterpret_cast<const uintx4*>((is_v ? vnew : knew) + (int64_t)r * new_stride + c * 16);
      __builtin_nontemporal_store(x, reinterpret_cast<uintx4*>(const_cast<unsigned char*>(is_v ? vbase : kbase) + (p.len_prev + r) * ROWB + c * 16));
    }
  }
  constexpr int kCopyRows = NT / CH, kCopyTurns = kCopyRows >= kRowsPerUnit ? 1 : kRowsPerUnit / kCopyRows;
  const int copy_r0 = MULTI && fused ? rem * p.copy_rows : 0;
  const int copy_r1 = MULTI && fused ? (copy_r0 + p.copy_rows < C ? copy_r0 + p.copy_rows : C) : 0;
  uintx4 copy_k[kCopyTurns] = {}, copy_v[kCopyTurns] = {};
  auto copy_load = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kCopyTurns; ++i) {
      const int r = r0 + i * kCopyRows + tid / CH;
      if (r < copy_r1) {
        const unsigned off = (unsigned)r * new_stride + (unsigned)(tid % CH) * 16u;
        copy_k[i] = *reinterpret_cast<const uintx4*>(knew + off);
        copy_v[i] = *reinterpret_cast<const uintx4*>(vnew + off);
        if (ROT) {
          const int c = tid % CH;
          const bool lower = c < CH / 2;
          const uintx4 other = *reinterpret_cast<const uintx4*>(knew + (lower ? off + ROWB / 2 : off - ROWB / 2));
          const int64_t at = (int64_t)r * (D / 2) + (lower ? c : c - CH / 2) * 8;
          bf16x8 v = __builtin_bit_cast(bf16x8, copy_k[i]);
          rotate_vec<__bf16, 8>(v, __builtin_bit_cast(bf16x8, other), p.rope_cos + at, p.rope_sin + at, lower);
          copy_k[i] = __builtin_bit_cast(uintx4, v);
        }
      }
    }
  };
  auto copy_store = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kCopyTurns; ++i) {
      const int r = r0 + i * kCopyRows + tid / CH;
      if (r < copy_r1) {
        const unsigned off = (unsigned)((int)p.len_prev + r) * (unsigned)ROWB + (unsigned)(tid % CH) * 16u;
        __builtin_nontemporal_store(copy_k[i], reinterpret_cast<uintx4*>(const_cast<unsigned char*>(kbase) + off));
        __builtin_nontemporal_store(copy_v[i], reinterpret_cast<uintx4*>(const_cast<unsigned char*>(vbase) + off));
      }
    }
  };

  if (MULTI) copy_load(copy_r0);

  // ---- LDS read offsets (general kernel's layouts): K fragment ks, row m, chunk 2 ks + hi; V^T by the transpose read, lane i
  // of a 16-lane group supplies row i / 4 of a 4-row group and 4 columns
  unsigned kaddr[KS], vaddr[DB];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kaddr[ks] = my_lds + (unsigned)(m * ROWB + (((ks * 2 + hi) ^ (m % KSW)) * 16));
  {
    const int i16 = l & 15, b2 = (l >> 4) & 1, v_row = 4 * hi + (i16 >> 2);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      vaddr[db] = my_lds + (unsigned)(BLOCKB + v_row * ROWB + (((4 * db + 2 * b2 + ((i16 & 3) >> 1)) ^ ((v_row & 3) * VSW)) * 16) + 8 * (i16 & 1));
  }

  floatx16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

#pragma unroll 1
  for (int i = 0; i < n_blocks; ++i) {
    const int nb = b + NW < b_end ? b + NW : b_first;
    const bool more = i + 1 < n_blocks;
    // copies complete in order; a block that is not plain may have taken more of them than SLABS
    if (plain(b))
      wait_vm<SLABS>();
    else
      wait_vm<0>();
    const int key0 = first_key(b);
    if (ROT && __builtin_expect(key0 + 32 > (int)p.len_prev, 0)) {
      // two lanes a row, each a half of its pairs of 16-byte chunks (c, c + CH / 2)
      const int r = l >> 1, row = key0 + r < (int)kr.row_lim ? key0 + r : (int)kr.row_lim, t = row - (int)p.len_prev;
      if (t >= 0) {
        const unsigned at_row = my_lds + (unsigned)(r * ROWB);
#pragma unroll D == 64 ? 1 : CH / 4
        for (int i = 0; i < CH / 4; ++i) {
          const int c = (l & 1) * (CH / 4) + i;
          const unsigned lo_at = at_row + (unsigned)((c ^ (r % KSW)) * 16), up_at = at_row + (unsigned)(((c + CH / 2) ^ (r % KSW)) * 16);
          const int64_t at = (int64_t)t * (D / 2) + c * 8;
          const bf16x8 lo = *LDS_PTR(const bf16x8, lo_at), up = *LDS_PTR(const bf16x8, up_at);
          bf16x8 lo2 = lo, up2 = up;
          rotate_vec<__bf16, 8>(lo2, up, p.rope_cos + at, p.rope_sin + at, true);
          rotate_vec<__bf16, 8>(up2, lo, p.rope_cos + at, p.rope_sin + at, false);
          *LDS_PTR(bf16x8, lo_at) = lo2;
          *LDS_PTR(bf16x8, up_at) = up2;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    floatx16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 a = *LDS_PTR(const bf16x8, kaddr[ks]);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], s, 0, 0, 0);
    }
    asm volatile("" : "+v"(s)::"memory");  // every read of the K block has returned
    if (more) fetch(false, nb);

    const bool left = WIN && key0 < lb_last && key0 + 32 > p.n_sink;  // keys between the sinks and the window
    if (key0 + 32 > vis_first || left) {  // wave-uniform: some row does not see the whole block
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
    mx = pair_max(mx);
    // only rows that ask for it move, so a row's arithmetic never depends on its wave neighbours
    const bool mine = mx > m_run + kStale || (m_run == -INFINITY && mx > -INFINITY);
    if (__any(mine)) {
      const float m2 = mine ? mx : m_run;
      const float alpha = m_run == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m2);  // (without history: l = 0, O = 0)
      m_run = m2;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    const float ref = m_run == -INFINITY ? 0.f : m_run;
    uintx4 pb[2];  // P^T fragments: 8 bf16 per 16-key slab
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float a = __builtin_amdgcn_exp2f(s[2 * k] - ref), c = __builtin_amdgcn_exp2f(s[2 * k + 1] - ref);
      l_run += a;
      l_run += c;
      bf16x2 pk;
      pk[0] = (__bf16)a;
      pk[1] = (__bf16)c;
      pb[k >> 2][k & 3] = __builtin_bit_cast(unsigned, pk);
    }

    if (more && plain(nb))
      wait_vm<SLABS>();
    else
      wait_vm<0>();
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const unsigned at = vaddr[db] + (unsigned)(16 * tt * ROWB);
        const short4_ lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4_, at));
        const short4_ up = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4_, at + 8 * ROWB));
        const short8_ a8 = __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a8), __builtin_bit_cast(bf16x8, pb[tt]), o[db], 0, 0, 0);
      }
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(o[db])::"memory");  // every read of the V block has returned
    if (more) fetch(true, nb);
    b = nb;
  }

  // ---- the wavefronts' results meet in LDS: [wavefront][row][D] and [wavefront][row] (m, l)
  wait_vm<0>();  // (the chunk's rows are used up before the output may take their place)
  const float l_tot = pair_sum(l_run);
  if ((WIN || __builtin_expect(first_key(b_first) >= vis_first, 0)) && n_blocks > 0 && __any(l_tot == 0.f)) {
    // rows that saw none of the wavefront's keys: O may be NaN, 0 times a value that is not finite
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = l_tot == 0.f ? 0.f : o[db][r];
  }
  __syncthreads();
  constexpr int OROW = D * 4 + 16;
  const unsigned obase = lds0 + (unsigned)(w * kRowsPerUnit * OROW), mlbase = lds0 + (unsigned)(NW * kRowsPerUnit * OROW);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      floatx4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[db][rg * 4 + e];
      *LDS_PTR(floatx4, obase + (unsigned)(m * OROW + (db * 32 + 8 * rg + 4 * hi) * 4)) = v;
    }
  if (hi == 0) *LDS_PTR(floatx2, mlbase + (unsigned)((w * kRowsPerUnit + m) * 8)) = floatx2{m_run, l_tot};
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
      ml[ww] = *LDS_PTR(const floatx2, mlbase + (unsigned)((ww * kRowsPerUnit + r) * 8));
      M = fmaxf(M, ml[ww].x);
    }
    float L = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const floatx4 x = *LDS_PTR(const floatx4, lds0 + (unsigned)((ww * kRowsPerUnit + r) * OROW + c * 16));
      const float f = ml[ww].y == 0.f ? 0.f : __builtin_amdgcn_exp2f(ml[ww].x - M);  // (0: it saw no visible key)
      L += f * ml[ww].y;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += f * x[e];
    }
    const int t = (int)quot((unsigned)(row0 + r), p.by_group), h = g * G + row0 + r - t * G;
    const int64_t at = (int64_t)t * Hq + h;
    if (p.n_splits == 1) {
      const float inv = 1.f / L;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[e] * inv);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + at * D + c * 4) = v;
      if (p.lse && c == 0) p.lse[(int64_t)h * C + t] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
    } else {
      *reinterpret_cast<floatx4*>(p.part_o + ((int64_t)split * n_rows + at) * D + c * 4) = acc;
      if (c == 0) *reinterpret_cast<float2*>(p.part_ml + ((int64_t)split * n_rows + at) * 2) = make_float2(M, L);
    }
  }

  if (MULTI) {
    copy_store(copy_r0);
    for (int r0 = copy_r0 + kCopyTurns * kCopyRows; r0 < copy_r1; r0 += kCopyTurns * kCopyRows) {
      copy_load(r0);
      copy_store(r0);
    }
  }
}

template <int D, int NW, bool WIN, bool MULTI, bool ROT>
static hipError_t prepare_few_one() {
  // once per device (idempotent; a benign race at worst sets it twice)
  static bool attr_done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (attr_done[dev]) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_few_kernel<D, NW, WIN, MULTI, ROT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, few_lds_bytes<D, NW>());
  if (e == hipSuccess) attr_done[dev] = true;
  return e;
}
template <int D>
static hipError_t prepare_few() {
  hipError_t e = prepare_few_one<D, 4, false, true, false>();
  if (D == 128 && e == hipSuccess) e = prepare_few_one<128, 4, false, false, false>();
  if (e == hipSuccess) e = prepare_few_one<D, 4, false, true, true>();
  if (e == hipSuccess) e = prepare_few_one<D, 8, false, true, false>();
  if (e == hipSuccess) e = prepare_few_one<D, 8, false, true, true>();
  if (e == hipSuccess) e = prepare_few_one<D, 8, true, true, false>();
  return e;
}
hipError_t prepare_attn_few(int head_dim) { return head_dim == 128 ? prepare_few<128>() : prepare_few<64>(); }

template <int D, int NW, bool WIN, bool MULTI, bool ROT>
static void launch_few_one(const AttnParams& p, hipStream_t s) {
  hipLaunchKernelGGL((attn_few_kernel<D, NW, WIN, MULTI, ROT>), dim3(padded_grid(p.n_wgs)), dim3(NW * 64), (few_lds_bytes<D, NW>()), s, p);
}
template <int D>
static void launch_few(const AttnParams& p, int key_waves, hipStream_t s) {
  const bool rotate = p.k_new && p.rope_cos;
  if (D == 128 && key_waves == 4 && p.units_per_head == 1)  // (64 wide: attn_decode.hip)
    launch_few_one<128, 4, false, false, false>(p, s);
  else if (key_waves == 4)
    rotate ? launch_few_one<D, 4, false, true, true>(p, s) : launch_few_one<D, 4, false, true, false>(p, s);
  else if (p.window > 0)
    launch_few_one<D, 8, true, true, false>(p, s);
  else
    rotate ? launch_few_one<D, 8, false, true, true>(p, s) : launch_few_one<D, 8, false, true, false>(p, s);
}

hipError_t launch_attn_few(const AttnParams& p, int head_dim, int key_waves, hipStream_t s) {
  if (head_dim == 128)
    launch_few<128>(p, key_waves, s);
  else if (head_dim == 64)
    launch_few<64>(p, key_waves, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace kvfold
