// Chunk-prefix attention of the fold step, bf16 operands on the gfx950 matrix cores.
//
// What it computes (paper Sec. 2, "KV-Fold"): row i of the chunk, query head h, attends to cache
// rows j <= len_prev + i of KV head h / G -- the whole prefix plus the causal part of the chunk
// itself:
//     out[i][h] = sum_j softmax_j(scale * q[i][h] . K[j]) V[j].
// The chunk's rows are either in the cache already (the append kernel ran first) or are read from
// k_new / v_new as handed in while this kernel also copies them into the cache (fused append; a key
// tile with rows on both sides of the old cache's end is filled from both).  Under the sink +
// sliding-window mask (Sec. 6, the streaming baseline) a row sees of those keys only the first
// n_sink and the last `window`, and the key tiles in between are never touched.
//
// Mapping to the machine
//  * Work unit = 32 consecutive packed rows of a KV head: its (token, head of the group) pairs,
//    token-major.  A wavefront owns QB units, a workgroup 4 wavefronts; all units of a workgroup
//    share one KV head, so a K/V tile staged in LDS is reused across the grouped-query heads, and
//    with QB = 2 every K/V fragment read from LDS feeds two MFMAs.  Units ascend with the tokens,
//    so the wavefronts of a workgroup see (almost) the same key range and only the last tiles need
//    the causal mask; a chunk of C tokens fills ceil(C G / 32) units, whatever C is.
//  * 64-key K/V tiles travel HBM/L2 -> LDS with global_load_lds_dwordx4 (no registers), several
//    tiles ahead, into rings of NV+1 (K) and NV (V) slots; the XOR swizzle that makes the later
//    LDS reads conflict-free is applied by choosing which 16-byte chunk each lane fetches.
//  * Per tile a wavefront forms S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (keys are the M rows),
//    so each lane ends up with 32 logits of ONE query: row max / row sum are in-lane plus one
//    exchange between lanes l and l^32.  The accumulator layout of S^T is, up to a fixed
//    permutation of the keys inside a 16-key slab, the B-operand layout of the next product
//    O^T = V^T P^T; V^T fragments are read from the row-major V tile with the LDS transpose read
//    (ds_read_b64_tr_b16) using the same permutation, so P never leaves registers.
//  * Software pipeline inside the wavefront, in half tiles of 32 keys: while the matrix pipe forms
//    S^T of half h+1 and then accumulates O^T of half h, the vector ALU turns S^T of half h into P
//    (exp2, bf16 pack, row sums) -- one exp2 behind every MFMA, the first quarter of a half already
//    in the tail of the step before, because a single wavefront hides only about 16-20 cycles of
//    other instructions under each 32-cycle MFMA.
//  * Online softmax in base 2 with ONE vector instruction per logit: the queries are multiplied by
//    scale*log2(e) once (and rounded to bf16 again), and the S^T accumulators start from -m (the
//    running row max) instead of 0, so the matrix pipe delivers S*scale*log2e - m and P is a bare
//    exp2.  m only has to be a reference close enough to the true row max for P to stay inside the
//    float range, so on tiles below the causal horizon no row max is taken at all: the row sum of a
//    half, which is needed anyway, bounds its largest P, and when it passes 2^20 the reference moves
//    up by a whole power of two (O, l and the in-flight logits are corrected exactly).  A row sum
//    beyond 2^60, infinite or NaN means the logits jumped by more than that inside one half; the
//    workgroup then starts over in a mode that takes the exact row max of every half before its
//    exp2 (the mode the masked tiles at the causal horizon always use, stale by at most 2^16).
//    P is rounded to bf16 by the hardware pack convert; row sums add the unrounded fp32 values.
//  * Optional split of the key range over workgroups: partial (max, sum, O) go to a workspace
//    and are merged by the combine kernel.
//  * Start and end of a workgroup are kept short (they are 4 % of a short-prefix launch and half of a
//    small one): every line of the kernel arguments is fetched in one round trip, the first two tiles are
//    on their way before the Q rows and the rest of the ring after them (a wait for Q is a wait for all
//    that was issued before), the first reference is set without touching the still-zero O, and the
//    finished O^T is turned in the dead ring space so that every store instruction writes whole rows.
//    Code a launch runs once costs what it is long, about 3 bytes per ns: what is outside the main loop
//    is kept small rather than unrolled, row addresses take a few 32-bit instructions (a row's place is
//    formed once per lane and handed round), the copy of the chunk's rows runs behind the results'
//    stores, and a piece of the prefix stays in the main loop to its last tile.  Measured inside the
//    kernel (100 tokens on 2000 keys, 7 pieces), from entry to the first tile and from the last tile to
//    the end: one-unit kernel 3.9 -> 3.1 us and 3.5 -> 2.0 us, two-unit kernel 6.1 -> 5.2 and 6.9 -> 3.5,
//    against 64-bit row arithmetic written out for every store and the ring filled ahead of Q.
#include <type_traits>

#include "kvfold_internal.h"
#include "wave_ops.h"

namespace kvfold {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4_;
typedef __attribute__((ext_vector_type(8))) short short8_;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) unsigned uintx4;
typedef __attribute__((ext_vector_type(2))) unsigned uintx2;
typedef __attribute__((ext_vector_type(4))) float floatx4;

// Wait until at most N LDS reads are outstanding (compiler-visible, so that it adds none of its own
// for fragments covered by this wait).  gfx9 encoding: vmcnt and expcnt left at their maxima.
template <int N>
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// MFMA issued by hand so that the register files are under control: S^T accumulates in VGPRs
// (the vector ALU reads it next), O^T in AGPRs, and the Q fragments (B operands) and the K
// fragments (A operands, loaded from LDS straight into AGPRs) sit in AGPRs too.
// The compiler does not see these as matrix instructions, so the read-after-MFMA-write distances
// the hardware needs are kept by construction (see mfma_settle_*()).
__device__ __forceinline__ void mfma_qk_first(floatx16& s, const bf16x8& a, const bf16x8& q, const floatx16& c0) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(s) : "a"(a), "a"(q), "v"(c0));
}
__device__ __forceinline__ void mfma_qk(floatx16& s, const bf16x8& a, const bf16x8& q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(a), "a"(q));
}
__device__ __forceinline__ void mfma_pv(floatx16& o, const bf16x8& a, const bf16x8& pfrag) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(pfrag));
}
// 48 idle issue cycles tied to a register tuple: everything that reads or writes `x` afterwards
// is ordered behind a finished matrix pipe (an 8-pass MFMA result is readable 19 cycles after issue).
__device__ __forceinline__ void mfma_settle_v(floatx16& x) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" : "+v"(x));
}
__device__ __forceinline__ void mfma_settle_a(floatx16& x) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" : "+a"(x));
}

constexpr int vote_bytes(int qb) { return qb == 2 ? 16 : 0; }  // (the one-unit kernel has no vote, and two workgroups fill the LDS to its last byte)
constexpr float kRescaleThreshold = 16.0f;  // log2 units: stale running max tolerated up to 2^16
constexpr float kSumThreshold = 1048576.0f;             // 2^20: row sum of a half that moves the reference up
constexpr float kRedoThreshold = 1152921504606846976.0f;  // 2^60: beyond this the workgroup starts over

// Slot schedule of one pipeline step of a wavefront with QA active units (QA = QB in the ordinary
// step; QA = 1 in a two-unit wavefront whose first unit has passed its causal horizon).  A step
// handles one 32-key half hh and consists of M MFMA slots: M1 slots forming S^T of half hh+1 (phase
// 1), then M2 slots accumulating O^T += V^T P^T of half hh (phase 2).  A single wavefront hides only
// about 16-20 cycles of other instructions under one 32-cycle MFMA (an exp2 costs 8, plain vector
// instructions 4), so everything else is dealt out evenly, a fixed share behind every MFMA:
//   * exp2 / pack / row-sum "events" of half hh (one event = one exp2; the second event of a logit
//     pair also packs the pair, and each event adds the exp2 before it to the row sum): events
//     [NEAR, NE) in slots [0, EW) of the half's own step, so that slab 0 of P is packed before phase
//     2 and slab 1 before its second half; with SUM_MODE the first NEAR events (all in slab 0) are
//     taken EARLY, in the tail slots [EW, M) of the step before, as soon as that S^T is complete;
//   * LDS fragment reads one batch ahead, in slots [0, RW), RW half way into the tail, one wait per batch;
//   * SUM_MODE: the test of the row sums against 2^20 right after the last event; else the row
//     maxima of half hh+1 and the rescale decision in the exp-free tail [RM0, M);
//   * in odd steps the workgroup barrier and the ring refill (DMA) in the tail [EW, M).
template <int D, int QA, bool SUM_MODE, int LPG>
struct Sched {
  static constexpr int KS = D / 16, DB = D / 32;
  static constexpr int M1 = KS * QA;       // MFMAs of phase 1 (K fragment ks feeds QA of them)
  static constexpr int M2 = 2 * DB * QA;   // MFMAs of phase 2 (V^T fragment (tt, db) feeds QA of them)
  static constexpr int M = M1 + M2;
  static constexpr int NP = QA * 8;        // logit pairs per step; pair k: slab k / (4 QA), unit (k / 4) % QA
  static constexpr int NE = 2 * NP;        // exp events
  static constexpr int EW = M1 + M2 / 2;
  static constexpr int NEAR = SUM_MODE ? (NE * (M - EW) / M) & ~1 : 0;
  static constexpr int NMAIN = NE - NEAR;
  static_assert(NEAR <= NE / 2, "early events must stay inside slab 0");
  static_assert(NEAR + (M1 * NMAIN + EW - 1) / EW >= NE / 2, "slab 0 would not be complete at the start of phase 2");
  static constexpr int GK = KS / 2;        // K fragments per batch (two batches per step)
  static constexpr int GV = DB;            // V^T fragments per batch (two batches per step, 2 reads each)
  static constexpr int R = 2 * GK + 4 * GV;  // LDS read instructions per step, in issue order:
                                             //   kg[1] (GK) | vg[0] (2 GV) | vg[1] (2 GV) | kg[0] of the next step (GK)
  static constexpr int RW = EW + (M - EW) / 2;  // (measured: spreading the reads a little into the tail beats stopping at EW)
  static_assert(EW + 1 < M, "no slot for the row-sum test");
  static constexpr int RM1 = M - 1 - QA;   // row-max slots [RM0, RM1), then QA + 1 decision slots
  static constexpr int RM0 = (EW - (M >= 32 ? 2 : 0)) < RM1 ? (EW - (M >= 32 ? 2 : 0)) : RM1 - 1;
  static_assert(SUM_MODE || RM0 >= M1 + 1, "row maxima would read S^T before its MFMAs retire");
  static_assert(SUM_MODE || (RM1 > RM0 && RM1 + QA < M), "no room for the row maxima");
  static_assert(LPG <= (M - EW) * 4, "ring refill does not fit the tail");
  // read r is issued in slot r * RW / R; reads issued before slot sl:
  static constexpr int rd_before(int sl) {
    int n = 0;
    for (int r = 0; r < R; ++r) n += (r * RW / R) < sl;
    return n;
  }
};

// 64 wide, a CU's LDS and registers have room for three workgroups of the one-unit kernel, and have to keep it: with the code that merges two pieces
// the compiler takes 180 registers where it is asked for two, and 3570 tokens on 30 keys, 32 heads on 8, took 80 us for 71, 2525 on 67 under a
// window of 267, 32 on 2, 24.8 for 20.2.  Asked for three it takes 156, without a spill, as before that code.
template <int D, int QB, int NV>
__global__ void __launch_bounds__(256, (QB == 2 ? 1 : D == 64 && NV == kRingShared ? 3 : 2)) attn_bf16_kernel(AttnParams p) {
  // Sum-driven reference updates (no row max below the causal horizon) for the two-unit kernel, whose
  // single wavefront per SIMD cannot hide the row-max work; the one-unit kernel has a second
  // wavefront to hide it and fewer registers, and takes the exact row max of every half.
  constexpr bool SUM_MODE = QB == 2;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned lds0 = (unsigned)(uintptr_t)((unsigned char __attribute__((address_space(3)))*)smem);
  constexpr int NK = NV + 1;         // K ring slots (K runs half a tile ahead of V in the pipeline)
  constexpr int CH = D / 8;          // 16-byte chunks per row
  constexpr int ROWB = D * 2;        // bytes per row
  constexpr int BN = kTileKeys;      // 64
  constexpr int KS = D / 16;         // contraction steps of S^T = K Q^T
  constexpr int DB = D / 32;         // 32-wide blocks of the head dim in O^T
  constexpr int TILEB = BN * ROWB;   // bytes of one K (or V) tile
  constexpr int HALFB = 32 * ROWB;   // bytes of a 32-key half tile
  constexpr int RPS = 64 / CH;       // rows covered by one 1 KiB DMA slab
  constexpr int SLABS = CH / 4;      // slabs per wavefront per tensor per tile
  constexpr int LPG = 2 * SLABS;     // DMA instructions per wavefront per tile (K + V)
  constexpr int KSW = CH < 16 ? CH : 16;  // K swizzle: chunk ^= row % KSW
  constexpr int VSW = CH / 4;             // V swizzle: chunk ^= (row & 3) * VSW

  // rings: K slots [0, NK), V slots [NK, NK + NV)

  // every line of the arguments is fetched now, in one round trip (they are not in the scalar cache yet)
  asm volatile("" ::"s"(p.q), "s"(p.n_tokens), "s"(p.units_per_head), "s"(p.k_new), "s"(p.by_group.mul), "s"(p.copy_rows));

  // ---- which workgroup am I (XCD-aware: a KV head stays on its XCDs, see logical_id())
  const int wgs_per_kvh = p.wgs_per_head * p.n_splits;
  const int lid = logical_workgroup(blockIdx.x, gridDim.x, p);
  if (lid >= p.n_wgs) return;
  const int g = (int)quot((unsigned)lid, p.by_wgs_per_kvh);
  const int rem = lid - g * wgs_per_kvh;
  const int split = (int)quot((unsigned)rem, p.by_wgs_per_head);
  // Later token blocks see more keys.  Default order: heaviest first (longest-processing-time
  // first over several rounds of workgroups).  With pair_order the grid is resident at once, two
  // workgroups per CU, dispatched in id order: the first half descends from the heaviest, the second
  // half ascends from the lightest, so the two workgroups that share a CU add up to the same work.
  int ug;
  {
    const int idx = rem - split * p.wgs_per_head, W = p.wgs_per_head, half = (W + 1) / 2;
    ug = (!p.pair_order || idx < half) ? W - 1 - idx : idx - half;
  }

  const int tid = threadIdx.x, l = tid & 63, hi = l >> 5, m = l & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = p.n_tokens, Hq = p.n_q_heads, G = p.group;
  const int Lm1 = (int)(p.len_prev + C - 1);  // last valid cache row
  constexpr int UPW = kUnitsPerWg * QB;        // units per workgroup
  const float sc = p.scale_log2e;

  // ---- my units
  const unsigned n_packed = (unsigned)(C * G);
  int tok[QB];            // of this lane's row (the chunk's last row where the unit runs past it)
  unsigned q_row[QB];     // its place among the [token][query head] rows
  int unit_of[QB];        // the units themselves, wave-uniform
  bool unit_valid[QB];
  int my_vis[QB];     // keys visible to this lane's query row
  int vis_first[QB];  // keys visible to the unit's first row (key blocks entirely below need no mask)
  int vis_last0 = 0;  // keys visible to the last row of unit 0: tiles entirely beyond are dead for it
  // Sink + sliding-window step (Sec. 6 of the paper, the streaming baseline's mask): the row that sees keys
  // [0, vis) sees of them only j < n_sink and j >= vis - window.  lb_last: the largest such lower bound among
  // the rows of the wavefront's units; key blocks that begin below it need the left mask.
  const bool win = p.window > 0;
  const int n_sink = p.n_sink;
  int lb_last = 0;
  // pair_units (two-unit kernel): wavefront number n = 4 ug + w of the KV head owns unit n, counted from
  // the first token block, and unit U-1-n, counted from the last, so that every wavefront has the
  // same number of (row, key) pairs to do whatever the causal horizon; else units 2n and 2n+1.
  const bool pair_units = QB == 2 && p.pair_units;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int n = ug * kUnitsPerWg + w;
    const int u = !pair_units ? n * QB + qb : (qb == 0 ? n : p.units_per_head - 1 - n);
    const bool valid = !pair_units ? u < p.units_per_head : (qb == 0 ? 2 * n <= p.units_per_head - 1 : 2 * n < p.units_per_head - 1);
    const int uc = u < 0 ? 0 : (u < p.units_per_head ? u : p.units_per_head - 1);
    unsigned row = (unsigned)(uc * kRowsPerUnit + m);  // packed row of the KV head
    row = row < n_packed ? row : n_packed - 1;
    tok[qb] = (int)quot(row, p.by_group);
    q_row[qb] = row + (unsigned)tok[qb] * (unsigned)(Hq - G) + (unsigned)(g * G);
    unit_of[qb] = uc;
    unit_valid[qb] = valid;
    {
      const int vis_last = (int)p.len_prev + unit_last_token(uc, p.by_group, C) + 1;
      if (qb == 0) vis_last0 = vis_last;
      if (win && vis_last - p.window > lb_last) lb_last = vis_last - p.window;
    }
    my_vis[qb] = (int)p.len_prev + tok[qb] + 1;
    vis_first[qb] = (int)p.len_prev + unit_first_token(uc, p.by_group) + 1;
  }
  const bool idle = !unit_valid[0];  // (then the second unit does not exist either)
  const int vis_min = vis_first[0];  // units ascend with the tokens, so unit 0 has the nearest horizon

  // ---- tile range of this workgroup / split
  int nkeys_wg;
  {
    // the unit of the workgroup with the farthest horizon: its last one, or with pair_units the partner of its first
    int ulast = pair_units ? p.units_per_head - 1 - ug * kUnitsPerWg : ug * UPW + UPW - 1;
    if (ulast > p.units_per_head - 1) ulast = p.units_per_head - 1;
    if (ulast < 0) ulast = 0;
    nkeys_wg = (int)p.len_prev + unit_last_token(ulast, p.by_group, C) + 1;
  }
  // logical tiles 0 .. ntiles-1 of this workgroup; under a window the tiles between the sinks and the window
  // are left out: logical tile t is physical tile t + (t >= ns_t ? skip : 0)
  TileMap tm;
  if (win) {
    const RowRange rr = workgroup_rows(ug, UPW, p.units_per_head, p.by_group, C);
    tm = tile_map(p.len_prev, rr.row_lo, rr.row_hi, n_sink, p.window);
  } else {
    tm.ns_t = 0;
    tm.skip = 0;
    tm.ntiles = (nkeys_wg + BN - 1) / BN;
  }
  const int ns_t = tm.ns_t, t_skip = tm.skip;
  auto tphys = [&](int t) __attribute__((always_inline)) -> int { return t + (t >= ns_t ? t_skip : 0); };
  // first logical tile whose physical tile is not below tp
  auto tlogical = [&](int tp) __attribute__((always_inline)) -> int {
    if (tp < ns_t) return tp;
    return tp - t_skip > ns_t ? tp - t_skip : ns_t;
  };
  // this workgroup's piece of them, and what its DMA may touch (shared with the host-side model of this walk)
  const KeyRange kr = key_range(tm, split, p.tiles_per_split, p.len_prev, C, p.k_new != nullptr);
  const int t_begin = kr.t_begin, t_end = kr.t_end;
  const int t_new = kr.t_straddle >= 0 ? kr.t_straddle : kr.t_new;  // first physical tile with rows of the chunk

  const unsigned head_bytes = (unsigned)p.capacity * (unsigned)ROWB;  // (below 2^32, as the host checks)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(p.k_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(p.v_cache) + (uint64_t)(unsigned)g * head_bytes;

  // ---- fused append (paper Sec. 2: the chunk's K/V rows join the cache): tiles from t_new on lie in the
  // chunk and are streamed from the rows as handed in, [C][Hkv][d], so no workgroup waits for another's
  // copy; the copy into the cache, for the steps to come, is shared out over the workgroups of the KV head.
  const bool fused = p.k_new != nullptr;
  const unsigned new_stride = (unsigned)(p.n_kv_heads * ROWB);  // bytes from one token's row to the next
  const unsigned char* knew = reinterpret_cast<const unsigned char*>(p.k_new) + (unsigned)g * (unsigned)ROWB;
  const unsigned char* vnew = reinterpret_cast<const unsigned char*>(p.v_new) + (unsigned)g * (unsigned)ROWB;
  // This workgroup's share of the copy: rows [r0, r1) of K and of V, 16 bytes per lane and access, loaded before the
  // results are stored and stored behind them, so that its latency is not paid on its own.
  constexpr int kCopyRows = 256 / CH;  // rows of a turn: a thread moves 16 bytes of a K row and of the V row
  constexpr int kCopyTurns = 2;        // turns whose loads are in flight together
  int copy_r0 = 0, copy_r1 = 0;
  if (fused) {
    copy_r0 = rem * p.copy_rows;
    copy_r1 = copy_r0 + p.copy_rows < C ? copy_r0 + p.copy_rows : C;
  }
  uintx4 copy_k[kCopyTurns] = {}, copy_v[kCopyTurns] = {};
  auto copy_load = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kCopyTurns; ++u) {
      const int r = r0 + u * kCopyRows + tid / CH;
      if (r0 + u * kCopyRows < copy_r1 && r < copy_r1) {
        const unsigned off = (unsigned)r * new_stride + (unsigned)(tid % CH) * 16u;
        copy_k[u] = *reinterpret_cast<const uintx4*>(knew + off);
        copy_v[u] = *reinterpret_cast<const uintx4*>(vnew + off);
      }
    }
  };
  auto copy_store = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kCopyTurns; ++u) {
      const int r = r0 + u * kCopyRows + tid / CH;
      if (r0 + u * kCopyRows < copy_r1 && r < copy_r1) {
        const unsigned off = (unsigned)((int)p.len_prev + r) * (unsigned)ROWB + (unsigned)(tid % CH) * 16u;
        __builtin_nontemporal_store(copy_k[u], reinterpret_cast<uintx4*>(const_cast<unsigned char*>(kbase) + off));
        __builtin_nontemporal_store(copy_v[u], reinterpret_cast<uintx4*>(const_cast<unsigned char*>(vbase) + off));
      }
    }
  };

  // ---- DMA addressing: wavefront w moves slabs w, w+4, ...; lane l lands at chunk (l % CH) of row
  // slab*RPS + l / CH and therefore fetches the chunk that the swizzle maps there.  Lane offsets are 32-bit (the host
  // checks capacity * row bytes < 2^32, and the fused append's chunk the same).
  const int dma_row0 = w * RPS + l / CH;  // + i * 4 * RPS for slab i
  const unsigned dma_kc = (unsigned)(((l % CH) ^ (dma_row0 % KSW)) * 16);
  const unsigned dma_vc = (unsigned)(((l % CH) ^ ((dma_row0 & 3) * VSW)) * 16);
  const unsigned dma_koff = (unsigned)dma_row0 * ROWB + dma_kc;  // lane part of an offset into the cache
  const unsigned dma_voff = (unsigned)dma_row0 * ROWB + dma_vc;
  const int t_last = t_end - 1;
  // Slab i of a tile, in the main loop over plain cache tiles (64 rows that are all there).  The ring runs NV + 1 tiles
  // ahead and knows no end: past the piece its last tile is fetched again (an L2 hit), so that pieces of the prefix
  // never leave the main loop.
  auto issue_slab = [&](bool is_v, int t_log, int slot, int i) __attribute__((always_inline)) {
    const int t = tphys(t_log < t_last ? t_log : t_last);
    const unsigned lds = lds0 + (unsigned)(((is_v ? NK : 0) + slot) * TILEB + (w + 4 * i) * 1024);
    const unsigned off = (is_v ? dma_voff : dma_koff) + (unsigned)(t * BN + i * 4 * RPS) * ROWB;
    dma16(is_v ? vbase : kbase, off, lds);
  };
  // A whole tile, plain or not, outside the slot schedule; nothing past the piece.  A plain tile -- 64 rows that all
  // exist and lie on one side of the old cache's end -- has a uniform base that moves from slab to slab.  Else rows
  // past the piece's last row are redirected to that row (never used, and so never fetched from HBM either).  The one
  // tile with rows on both sides of the cache's end (cache length not a multiple of the tile): each lane fetches from
  // its own side, two DMA instructions with complementary lanes fill a slab.
  auto issue_tile = [&](bool is_v, int t_log, int slot) __attribute__((always_inline)) {
    if (t_log >= t_end) return;
    const int t = tphys(t_log);
    unsigned lds = lds0 + (unsigned)(((is_v ? NK : 0) + slot) * TILEB + w * 1024);
    if (__builtin_expect(t != kr.t_straddle && (unsigned)(t * BN + BN - 1) <= kr.row_lim, 1)) {
      const bool nw = t >= kr.t_new;  // rows of the chunk as handed in (fused append)
      const unsigned stride = nw ? new_stride : (unsigned)ROWB;
      const unsigned row = (unsigned)(t * BN) - (nw ? (unsigned)p.len_prev : 0u);
      const unsigned char* base = (nw ? (is_v ? vnew : knew) : (is_v ? vbase : kbase)) + (uint64_t)(row * stride);
      unsigned off = (unsigned)dma_row0 * stride + (is_v ? dma_vc : dma_kc);
#pragma unroll
      for (int i = 0; i < SLABS; ++i) {
        dma16(base, off, lds);
        off += stride * (unsigned)(4 * RPS);
        lds += 4096u;
      }
    } else {
#pragma unroll 1
      for (int i = 0; i < SLABS; ++i) {
        const DmaRow src = dma_row(kr, t, dma_row0 + i * 4 * RPS);
        if (src.from_chunk)
          dma16(is_v ? vnew : knew, src.row * new_stride + (is_v ? dma_vc : dma_kc), lds);
        else
          dma16(is_v ? vbase : kbase, src.row * (unsigned)ROWB + (is_v ? dma_vc : dma_kc), lds);
        lds += 4096u;
      }
    }
  };

  // ---- the Q rows, the first two tiles, then the rest of the ring.  The Q rows come through LDS as well, into the part of the ring that the
  // first two tiles leave free: copies complete in order, so that Q is waited for alone and while the tiles are on their way; loads into
  // registers would be waited for by the compiler, which counts no copies, together with all that was issued around them (then Q was
  // there 4.5 us after a workgroup's start, two tiles of every workgroup later, and the rest of the ring was asked for only then).  Q,
  // pre-multiplied by scale*log2(e), stays in registers for the whole kernel.  Code that a launch runs once is fetched at about 3 bytes
  // per ns (measured: an unrolled fill of 6 KB took 2.3 us of a workgroup's start), so the fill is a loop.
  auto prefill = [&](int j0, int j1) __attribute__((always_inline)) {
    // Steady state at the top of the even step of tile t: K[t], K[t+1], V[t] are in LDS and visible, the
    // groups {K[t+1+j], V[t+j]}, j = 1 .. NV-1, are in flight.  Tile t_begin + j takes ring slot j.
#pragma unroll 1
    for (int j = j0; j <= j1; ++j) {
      issue_tile(false, t_begin + j, j);
      if (j > 0) issue_tile(true, t_begin + j - 1, j - 1);
    }
  };
  // This wavefront's 32 QB rows: the K slots from the third on, then the V slots from the second on.  A row's chunks lie as a K row's do.
  constexpr int QAREA = QB * HALFB;
  static_assert(4 * QAREA <= (NK - 2 + NV - 1) * TILEB && (NK - 2) * TILEB % QAREA == 0, "Q does not fit the free slots");
  const unsigned q_lds = lds0 + (unsigned)(2 * TILEB + w * QAREA) + (w * QAREA >= (NK - 2) * TILEB ? (unsigned)TILEB : 0u);
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    unsigned place[32 / RPS];  // of the rows that the lane fetches from: held by the lanes whose rows they are
#pragma unroll
    for (int i = 0; i < 32 / RPS; ++i) place[i] = (unsigned)__builtin_amdgcn_ds_bpermute(4 * (i * RPS + l / CH), (int)q_row[qb]);
#pragma unroll
    for (int i = 0; i < 32 / RPS; ++i) {
      const unsigned char* qrow = reinterpret_cast<const unsigned char*>(p.q) + (uint64_t)place[i] * ROWB + (unsigned)(((l % CH) ^ ((i * RPS + l / CH) % KSW)) * 16);
      dma16_at(qrow, q_lds + (unsigned)(qb * HALFB + i * 1024));
    }
  }
  prefill(0, 1);
  bf16x8 qf[QB][KS];
  {
    bf16x8 raw[QB][KS];
    if (t_begin + 1 < t_end)
      wait_vm<3 * SLABS>();  // (K, K and V; more where a tile is filled from both sides)
    else
      wait_vm<0>();
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) raw[qb][ks] = *LDS_PTR(const bf16x8, q_lds + (unsigned)(qb * HALFB + m * ROWB + (((ks * 2 + hi) ^ (m % KSW)) * 16)));
    if (p.rope_cos) {
      // Rotary embedding at the row's absolute position (Sec. 2), half-split pairs (j, j + D/2), fp32 with
      // the sine product rounded first, result rounded to bf16: bit for bit what a caller that rotates q
      // itself and stores it as bf16 would hand in.  Fragments ks and ks + KS/2 hold the two halves of 8 pairs.
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
        for (int ks = 0; ks < KS / 2; ++ks) {
          const float* cs = p.rope_cos + (int64_t)tok[qb] * (D / 2) + ks * 16 + hi * 8;
          const float* sn = p.rope_sin + (int64_t)tok[qb] * (D / 2) + ks * 16 + hi * 8;
          const bf16x8 lo = raw[qb][ks], up = raw[qb][ks + KS / 2];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float tl = (float)up[e] * sn[e], tu = (float)lo[e] * sn[e];
            raw[qb][ks][e] = (__bf16)__builtin_fmaf((float)lo[e], cs[e], -tl);
            raw[qb][ks + KS / 2][e] = (__bf16)__builtin_fmaf((float)up[e], cs[e], tu);
          }
        }
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[qb][ks][e] = (__bf16)((float)raw[qb][ks][e] * sc);
        asm volatile("" : "+a"(qf[qb][ks]));  // park the fragment in the AGPR file, where the MFMAs read it
      }
  }

  __builtin_amdgcn_s_barrier();  // every wavefront has its Q out of the slots that are filled now
  prefill(2, NV);

  // ---- LDS read offsets (per lane) of the tile currently being read, ring slot included; moved
  // from slot to slot once per tile
  // K fragment (A operand of S^T): row kb*32+m, chunk ks*2+hi, swizzled by row % KSW = m % KSW
  int kslot, vslot;  // ring slots of tile t (wave-uniform)
  unsigned kaddr[KS];
  unsigned vaddr[DB];

  // ---- running state
  floatx16 o[QB][DB];   // O^T accumulators (AGPRs)
  floatx16 negm[QB];    // -m (0 while no key has been seen) in every element: start value of S^T
  float m_run[QB], l_run[QB];
  int overflowed = 0;   // wave-uniform: a row sum left the range the sum-driven rescale can repair
  auto reset_state = [&]() __attribute__((always_inline)) {
    kslot = 0;
    vslot = 0;
    // derived from an opaque copy of the lane id, so that nothing computed here is kept in registers
    // across the main loop for the sake of a restart that almost never happens
    int l2 = l;
    asm volatile("" : "+v"(l2));
    const int hi2 = l2 >> 5, m2 = l2 & 31;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      kaddr[ks] = lds0 + (unsigned)(m2 * ROWB + (((ks * 2 + hi2) ^ (m2 % KSW)) * 16)) + (unsigned)(kslot * TILEB);
    // V^T fragment via transpose read: lane i of a 16-lane block supplies row (i/4) of a 4-row group and 4 columns
    const int i16 = l2 & 15, b2 = (l2 >> 4) & 1;
    const int v_row = 4 * hi2 + (i16 >> 2);  // + 16*tt (+8)
#pragma unroll
    for (int db = 0; db < DB; ++db)
      vaddr[db] = lds0 + (unsigned)(v_row * ROWB + (((4 * db + 2 * b2 + ((i16 & 3) >> 1)) ^ ((v_row & 3) * VSW)) * 16) + 8 * (i16 & 1)) +
                  (unsigned)((NK + vslot) * TILEB);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      m_run[qb] = -INFINITY;
      l_run[qb] = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) negm[qb][r] = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qb][db][r] = 0.f;
    }
  };

  // ---- building blocks of the software pipeline --------------------------------------------
  // K fragment ks of the current K tile (imm = 0) or of its second half (imm = HALFB), read from LDS
  // straight into AGPRs.  The compiler does not see an LDS access here: every use is covered by one
  // of the wait_lds<>() calls of the pipeline.
  auto k_frag = [&](int ks, int imm) __attribute__((always_inline)) -> bf16x8 {
    bf16x8 f;
    if (imm == 0)
      asm volatile("ds_read_b128 %0, %1" : "=a"(f) : "v"(kaddr[ks]));
    else
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=a"(f) : "v"(kaddr[ks]), "n"(HALFB));
    return f;
  };
  // causal mask (and, under a window, the mask of the keys between the sinks and the window) of the 32-key
  // half hh (logical numbering)
  auto mask_half = [&](floatx16 (&s)[QB], int hh, int q0 = 0) __attribute__((always_inline)) {
    // (opaque copies: whatever is derived from them is computed here, not once ahead of all loops and
    // then held in registers through the unmasked main loop)
    int hi_here = hi;
    asm volatile("" : "+v"(hi_here));
    const int key0 = (2 * tphys(hh >> 1) + (hh & 1)) * 32;  // first key of the half
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (qb < q0) continue;
      if (key0 + 32 > vis_first[qb]) {  // wave-uniform
        int vis_here = my_vis[qb];
        asm volatile("" : "+v"(vis_here));
        const int rel = vis_here - key0;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + 4 * hi_here + (r & 3) >= rel) s[qb][r] = -INFINITY;
      }
      if (win && key0 < lb_last && key0 + 32 > n_sink) {  // wave-uniform
        int vis_here = my_vis[qb];
        asm volatile("" : "+v"(vis_here));
        const int rel_lb = vis_here - p.window - key0, rel_sink = n_sink - key0;  // visible: below rel_sink or from rel_lb on
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int kk = 8 * (r >> 2) + 4 * hi_here + (r & 3);
          if (kk < rel_lb && kk >= rel_sink) s[qb][r] = -INFINITY;
        }
      }
    }
  };
  // mx[] holds the row maxima of a half whose logits are already relative to the running max, i.e.
  // by how much the max would grow.  The running max is raised only when it lags by more than
  // 2^16 (or has never been set).  The decision (cross-lane max, compare) is taken early, under
  // the matrix pipe; the branch comes later.
  auto rescale_need = [&](const float (&dm)[QB], int q0 = 0) __attribute__((always_inline)) -> bool {
    int need = 0;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)  // no short-circuit: plain lane-wise compares, one wave-wide reduction at the end
      if (qb >= q0) need |= (int)(dm[qb] > kRescaleThreshold) | ((int)(m_run[qb] == -INFINITY) & (int)(dm[qb] > -INFINITY));
    return __any(need);
  };
  auto rescale_decide = [&](const float (&mx)[QB], float (&dm)[QB], int q0 = 0) __attribute__((always_inline)) -> bool {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (qb >= q0) dm[qb] = pair_max(mx[qb]);
    return rescale_need(dm, q0);
  };
  // s holds the logits of the half the maxima came from: they were formed against the old max
  auto rescale_apply = [&](const float (&dm)[QB], floatx16 (&s)[QB], int q0 = 0) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (qb < q0) continue;
      const float cur = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
      // only rows that asked for it move, so a row's arithmetic never depends on its wave neighbours
      const bool mine = (dm[qb] > kRescaleThreshold) || (m_run[qb] == -INFINITY && dm[qb] > -INFINITY);
      const float m2 = mine ? fmaxf(m_run[qb], cur + dm[qb]) : m_run[qb];
      const float use = (m2 == -INFINITY) ? 0.f : m2;
      const float delta = use - cur;
      // a row without history (l = 0, O = 0) has nothing to scale, and its first reference may lie far enough
      // below zero for 2^-delta to overflow
      const float alpha = (m_run[qb] == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(-delta);
      m_run[qb] = m2;
      l_run[qb] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        negm[qb][r] = -use;
        s[qb][r] -= delta;
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        mfma_settle_a(o[qb][db]);
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qb][db][r] *= alpha;
      }
    }
  };
  // The first half of a pass: no history, so the row max of the half is the reference (0 for a row that sees
  // none of its keys) and neither l nor O needs touching.
  auto reference_first = [&](const float (&mx)[QB], floatx16 (&s)[QB]) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float dm = pair_max(mx[qb]);
      const float use = (dm > -INFINITY) ? dm : 0.f;
      m_run[qb] = dm;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        negm[qb][r] = -use;
        s[qb][r] -= use;
      }
      asm volatile("" : "+v"(negm[qb]));  // 16 registers from here on, not one value splatted anew ahead of every MFMA chain
    }
  };
  // ls[] holds the row sums of the half just exponentiated (per lane: the 16 keys it owns).  A sum
  // above 2^20 moves the reference up by the power of two just above it, which is exact; s holds
  // the in-flight logits of the next half, formed against the old reference.  Both lanes of a row
  // decide on the larger of their two sums, so a row never depends on its wave neighbours.
  auto rescale_from_sum = [&](const float (&ls)[QB], floatx16 (&s)[QB], int q0 = 0) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (qb < q0) continue;
      const float tot = pair_max(ls[qb]);
      const bool bad = !(tot <= kRedoThreshold);  // also infinite or NaN
      overflowed |= __any((int)bad);
      const bool mine = !(tot <= kSumThreshold) && !bad;
      const int e = mine ? __builtin_amdgcn_frexp_expf(tot) : 0;  // tot < 2^e
      const float delta = (float)e;
      const float alpha = __builtin_ldexpf(1.0f, -e);
      const float cur = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
      const float use = cur + delta;
      if (mine) m_run[qb] = use;
      l_run[qb] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        negm[qb][r] = -use;
        s[qb][r] -= delta;
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        mfma_settle_a(o[qb][db]);
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qb][db][r] *= alpha;
      }
    }
  };
  auto rowmax_all = [&](floatx16 (&s)[QB], float (&mx)[QB], int q0 = 0) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (qb < q0) continue;
      float a = fmaxf(s[qb][0], s[qb][1]);
#pragma unroll
      for (int r = 2; r < 16; r += 2) a = fmaxf(fmaxf(a, s[qb][r]), s[qb][r + 1]);
      mx[qb] = a;
    }
  };

  // ---- the software pipeline (slot schedule: struct Sched) -----------------------------------
  constexpr int GK = KS / 2, GV = DB;  // fragments per batch, whatever the number of active units

  floatx16 sA[QB], sB[QB];
  uintx4 pb[QB][2];      // P^T fragments: 8 bf16 per 16-key slab, as packed pairs
  float lsum_early[QB];  // row sums of the early events of the half that the next step finishes
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) lsum_early[qb] = 0.f;
  // One exp event of a half whose logits are in s: event j covers logit j of the half's 2 NP, in
  // pairs; the second event of a pair also packs the pair into its P^T slot and the first adds the
  // previous pair's second exp to the row sum (`first`: there is none pending).
  float ev_a = 0.f, ev_b = 0.f;  // first exp of the pair in flight; second exp not yet in its row sum
  // unit that event j of a step with units Q0 .. QB-1 belongs to
  auto ev_unit = [](int j, int Q0, int QA) constexpr { return Q0 + (((j >> 1) % (QA * 4)) >> 2); };
  auto exp_event = [&](const floatx16 (&s)[QB], float (&ls)[QB], int j, bool first, auto q0_tag) __attribute__((always_inline)) {
    constexpr int Q0 = decltype(q0_tag)::value, QA = QB - Q0;  // active units Q0 .. QB-1
    const int k = j >> 1, slab = k / (QA * 4), kk = k % (QA * 4);
    const int qb = Q0 + (kk >> 2), jj = kk & 3, r = 8 * slab + 2 * jj;
    if ((j & 1) == 0) {
      if (first)
        asm volatile("v_exp_f32_e32 %0, %1" : "=v"(ev_a) : "v"(s[qb][r]));
      else
        asm volatile(
            "v_exp_f32_e32 %0, %2\n\t"
            "v_add_f32_e32 %1, %3, %1"
            : "=&v"(ev_a), "+v"(ls[ev_unit(j - 1, Q0, QA)])
            : "v"(s[qb][r]), "v"(ev_b));
    } else {
      float eb;
      unsigned pku;
      asm volatile(
          "v_exp_f32_e32 %0, %3\n\t"
          "v_add_f32_e32 %2, %4, %2\n\t"
          "v_cvt_pk_bf16_f32 %1, %4, %0"
          : "=&v"(eb), "=v"(pku), "+v"(ls[qb])
          : "v"(s[qb][r + 1]), "v"(ev_a));
      pb[qb][slab][jj] = pku;
      ev_b = eb;
    }
  };
  // the early events of a half all at once (prologue, masked steps, and again after a sum-driven shift)
  auto early_events = [&](const floatx16 (&s)[QB], auto q0_tag) __attribute__((always_inline)) {
    constexpr int Q0 = decltype(q0_tag)::value, QA = QB - Q0;
    constexpr int NEAR = Sched<D, QA, SUM_MODE, LPG>::NEAR;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) lsum_early[qb] = 0.f;
    if (NEAR > 0) {
#pragma unroll
      for (int j = 0; j < NEAR; ++j) exp_event(s, lsum_early, j, j == 0, q0_tag);
      lsum_early[ev_unit(NEAR - 1, Q0, QA)] += ev_b;
    }
  };
  bf16x8 kg[2][GK];          // K fragment batches
  short4_ vh[2][GV][2];      // V^T fragment batches, as the two transpose-read halves of each fragment
  auto v_half = [&](int tt, int db, int half, int imm) __attribute__((always_inline)) -> short4_ {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4_, vaddr[db] + (unsigned)(imm + 16 * tt * ROWB + half * 8 * ROWB)));
  };

  // One pipeline step for half hh.  On entry s_cur holds S^T of half hh (masked, relative to the
  // running max), kg[0] the first batch of K fragments of half hh+1, and kaddr/vaddr point at the
  // tiles of halves hh+1 / hh.  ODD steps (second half of a tile) end with the workgroup barrier
  // and the ring refill for the tiles after next; MASKED selects the variant for halves hh+1 that
  // reach past the causal horizon, and for every half once a row sum has overflowed (mask, then the
  // exact row max, after the matrix work); PLAIN the variant whose refill consists of cache tiles only, slab by slab in
  // the slot schedule, where the others refill whole tiles after the matrix work.  q0_tag = 1 (two-unit kernel only):
  // unit 0 has passed its causal horizon for good and only unit 1 is worked on, with the schedule of a one-unit step; a
  // masked step of both units that is followed by such a step (next_unit1_only) leaves the early events in that step's
  // numbering.  Past the piece's last tile the ring need not hold keys: the last step forms an S^T of stale LDS
  // contents, on which nothing may be decided.
  auto step = [&](floatx16 (&s_cur)[QB], floatx16 (&s_next)[QB], int hh, auto odd_tag, auto masked_tag, auto plain_tag,
                  auto q0_tag, bool next_unit1_only = false) __attribute__((always_inline)) {
    constexpr bool PLAIN = decltype(plain_tag)::value;
    constexpr bool ODD = decltype(odd_tag)::value;
    constexpr bool MASKED = decltype(masked_tag)::value;
    constexpr int Q0 = decltype(q0_tag)::value, QA = QB - Q0;
    using S = Sched<D, QA, SUM_MODE, LPG>;
    constexpr int M1 = S::M1, M = S::M, EW = S::EW, NE = S::NE, NEAR = S::NEAR, NMAIN = S::NMAIN, NP = S::NP;
    constexpr int R = S::R, RW = S::RW, RM0 = S::RM0, RM1 = S::RM1;
    const int t = hh >> 1;
    constexpr int KIMM = ODD ? 0 : HALFB;  // even hh: half hh+1 is the second half of tile t
    constexpr int VIMM = ODD ? HALFB : 0;  // even hh: half hh is the first half of tile t
    float lsum[QB], lsum_next[QB];  // row sums of half hh (early part included) and of the early part of hh+1
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      lsum[qb] = lsum_early[qb];
      lsum_next[qb] = 0.f;
    }  // (entries of units before Q0 are carried along untouched and never added anywhere)
    float mx[QB], dm[QB];
    bool need_rescale = false;
    int sum_flag = 0;      // per lane: a row sum of this half passed 2^20 (or is not a number)
    int kslot_prev = 0, vslot_prev = 0;
    const bool more = (SUM_MODE ? PLAIN : !ODD) || hh + 1 < 2 * t_end;  // half hh + 1 is there (or nothing is decided on it)

    wait_lds<0>();  // kg[0] (fetched at the end of the previous step) has landed
#pragma unroll
    for (int i = 0; i < M; ++i) {
      // ---- waits and the barrier come before the MFMA of the slot
      if (i == GK * QA) wait_lds<(S::rd_before(GK * QA) - GK)>();                 // kg[1]
      if (i == M1) wait_lds<(S::rd_before(M1) - GK - 2 * GV)>();                  // vg[0]
      if (i == EW) wait_lds<(S::rd_before(EW) - GK - 4 * GV)>();                  // vg[1]
      if (ODD && i == EW) {
        // Every read of K[t] and V[t] by this wave has returned.  K[t+2] and V[t+1] were issued
        // NV-1 tiles ago: they are the oldest group in flight.
        if (PLAIN || (NV > 2 && t + NV < t_end))
          wait_vm<(NV - 2) * LPG>();
        else
          wait_vm<0>();  // the group issued last is not whole
        __builtin_amdgcn_s_barrier();  // ... and this holds for every wave of the workgroup
        kslot_prev = kslot == 0 ? NK - 1 : kslot - 1;  // K[t]'s slot (kslot already names K[t+1]) takes K[t+1+NV]
        vslot_prev = vslot;                            // V[t]'s slot takes V[t+NV]
      }
      // ---- the MFMA
      if (i < M1) {
        const int ks = i / QA, qb = Q0 + i % QA;
        if (ks == 0)
          mfma_qk_first(s_next[qb], kg[0][0], qf[qb][0], negm[qb]);
        else
          mfma_qk(s_next[qb], kg[ks / GK][ks % GK], qf[qb][ks]);
      } else {
        const int sl = (i - M1) / QA, qb = Q0 + (i - M1) % QA, tt = sl / DB, db = sl % DB;
        const short8_ a8 = __builtin_shufflevector(vh[sl / GV][sl % GV][0], vh[sl / GV][sl % GV][1], 0, 1, 2, 3, 4, 5, 6, 7);
        mfma_pv(o[qb][db], __builtin_bit_cast(bf16x8, a8), __builtin_bit_cast(bf16x8, pb[qb][tt]));
      }
      __builtin_amdgcn_sched_barrier(0);
      // ---- its share of everything else
      // LDS reads
#pragma unroll
      for (int r = (i * R + RW - 1) / RW; r < ((i + 1) * R + RW - 1) / RW && r < R; ++r) {  // rd_slot(r) == i
        if (r < GK) {
          kg[1][r] = k_frag(GK + r, KIMM);
        } else if (r < GK + 4 * GV) {
          const int q = r - GK, f = q / 2, half = q % 2;  // fragment f = (tt, db) of the half, in use order
          vh[f / GV][f % GV][half] = v_half(f / DB, f % DB, half, VIMM);
        } else {
          const int j = r - GK - 4 * GV;
          kg[0][j] = k_frag(j, ODD ? HALFB : 0);  // kg[0] of the NEXT step (half hh+2)
        }
      }
      // after an even step the next K half starts a new tile: move the K read offsets to its ring
      // slot, a few per slot, between the last read of this tile's K and the first of the next
      if (!ODD && i >= GK * QA && i < GK * QA + (KS + 1) / 2) {
        const int kn = kslot + 1 == NK ? 0 : kslot + 1;
        const unsigned dk = (unsigned)((kn - kslot) * TILEB);
        const int a = (i - GK * QA) * 2;
        kaddr[a] += dk;
        if (a + 1 < KS) kaddr[a + 1] += dk;
        if (i == GK * QA + (KS + 1) / 2 - 1) kslot = kn;
      }
      // exp events of half hh ...
      if (i == EW) lsum[ev_unit(NE - 1, Q0, QA)] += ev_b;
#pragma unroll
      for (int j = NEAR + (i * NMAIN + EW - 1) / EW; j < NEAR + ((i + 1) * NMAIN + EW - 1) / EW && j < NE; ++j)
        exp_event(s_cur, lsum, j, j == NEAR, q0_tag);
      // ... and, below the causal horizon, the early ones of half hh+1, whose S^T is complete by now
      if (!MASKED && NEAR > 0 && i >= EW) {
#pragma unroll
        for (int j = ((i - EW) * NEAR + (M - EW) - 1) / (M - EW); j < ((i - EW + 1) * NEAR + (M - EW) - 1) / (M - EW) && j < NEAR; ++j)
          exp_event(s_next, lsum_next, j, j == 0, q0_tag);
        if (i == M - 1) lsum_next[ev_unit(NEAR - 1, Q0, QA)] += ev_b;
      }
      if (SUM_MODE && i == EW + 1) {
#pragma unroll
        for (int qb = Q0; qb < QB; ++qb) sum_flag |= (int)!(lsum[qb] <= kSumThreshold);
      }
      // row maxima of half hh+1 (its last MFMA is at least RM0 - M1 slots old), then the decision
      if (!SUM_MODE && !MASKED && i >= RM0 && i < RM1) {
#pragma unroll
        for (int k = ((i - RM0) * NP) / (RM1 - RM0); k < ((i - RM0 + 1) * NP) / (RM1 - RM0); ++k) {
          const int q2 = Q0 + (k >> 3), r = 2 * (k & 7);
          if (r == 0)
            mx[q2] = fmaxf(s_next[q2][0], s_next[q2][1]);
          else
            mx[q2] = fmaxf(fmaxf(mx[q2], s_next[q2][r]), s_next[q2][r + 1]);
        }
      }
      if (!SUM_MODE && !MASKED && i >= RM1 && i < RM1 + QA) dm[Q0 + i - RM1] = pair_max(mx[Q0 + i - RM1]);
      if (!SUM_MODE && !MASKED && i == RM1 + QA) need_rescale = rescale_need(dm, Q0);
      // ring refill and the V address of the next tile (odd steps, after the barrier)
      if (ODD && i >= EW) {
        if (PLAIN) {
#pragma unroll
          for (int d = ((i - EW) * LPG) / (M - EW); d < ((i - EW + 1) * LPG) / (M - EW); ++d) {
            if (d < SLABS) issue_slab(false, t + 1 + NV, kslot_prev, d);
            else issue_slab(true, t + NV, vslot_prev, d - SLABS);
          }
        }
        if (i == M - 1) {
          const int vn = vslot + 1 == NV ? 0 : vslot + 1;
          const unsigned dv = (unsigned)((vn - vslot) * TILEB);
#pragma unroll
          for (int d2 = 0; d2 < DB; ++d2) vaddr[d2] += dv;
          vslot = vn;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int qb = Q0; qb < QB; ++qb) {
      l_run[qb] += lsum[qb];
      lsum_early[qb] = lsum_next[qb];
    }
    if constexpr (SUM_MODE) {
      if (__builtin_expect(__any(sum_flag), 0)) {
#pragma unroll
        for (int qb = Q0; qb < QB; ++qb) mfma_settle_v(s_next[qb]);
        rescale_from_sum(lsum, s_next, Q0);  // (past the last half s_next is stale, and merely moved)
        if (!MASKED) early_events(s_next, q0_tag);  // they were formed against the old reference: once more
      }
    }
    if (!PLAIN && ODD) {
      issue_tile(false, t + 1 + NV, kslot_prev);
      issue_tile(true, t + NV, vslot_prev);
    }
    if (MASKED && more) {
#pragma unroll
      for (int qb = Q0; qb < QB; ++qb) mfma_settle_v(s_next[qb]);
      mask_half(s_next, hh + 1, Q0);
      rowmax_all(s_next, mx, Q0);
      need_rescale = rescale_decide(mx, dm, Q0);
    }
    if (__builtin_expect(need_rescale, 0)) {
      // One-unit kernel: `more` is looked at in here; as part of the branch its scalar instructions ended every step
      // (C = 128 on 32K keys, 28 heads on 4: 145 us with them, 141 without).
      if (!SUM_MODE && !MASKED) asm volatile("");
      if (SUM_MODE || MASKED || more) {
#pragma unroll
        for (int qb = Q0; qb < QB; ++qb) mfma_settle_v(s_next[qb]);
        rescale_apply(dm, s_next, Q0);
      }
    }
    if (MASKED) {
      if (QB == 2 && Q0 == 0 && next_unit1_only)
        early_events(s_next, std::integral_constant<int, QB - 1>{});
      else
        early_events(s_next, q0_tag);
    }
  };

  if (t_begin < t_end) {
    // A second pass (exact = true) follows only if a row sum overflowed in the first.
    for (bool exact = false;; exact = true) {
      reset_state();
      // Tiles whose two steps only produce halves entirely below the nearest causal horizon take the
      // fast variant: step 2t+1 produces half 2t+2 = keys [64t+64, 64t+96), so it needs 64t+96 <= vis_min.
      // (tile bounds are worked out on physical tiles, i.e. on keys, and then turned into logical tile numbers)
      int t_fast = tlogical((vis_min - 96) / BN + 1);  // first tile that is not fast (vis_min >= 1)
      if (vis_min < 96 || exact) t_fast = 0;
      if (!exact && tphys(t_end - 1) * BN + BN <= vis_min) t_fast = t_end;  // the piece ends below every horizon
      if (t_fast > t_end) t_fast = t_end;
      // Under a window the first tiles (the sinks, and the tiles that begin below the window of the wavefront's
      // last row) are masked on the left: tiles [t_begin, t_lead) take the masked variant
      int t_lead = win ? tlogical((lb_last + BN - 1) / BN) : 0;
      if (win && t_lead < ns_t) t_lead = ns_t;
      if (t_lead > t_end) t_lead = t_end;
      // Two-unit kernel: from tile t_dead on every key is beyond the last row of unit 0 and only unit 1
      // is worked on, fast up to its own horizon (t_fast1), masked from there.
      int t_dead = tlogical((vis_last0 + BN - 1) / BN);
      if (t_dead < t_lead) t_dead = t_lead;
      if (QB == 1 || exact || t_dead > t_end) t_dead = t_end;
      int t_fast1 = tlogical((vis_first[QB - 1] - 96) / BN + 1);
      if (vis_first[QB - 1] < 96 || exact) t_fast1 = 0;
      if (t_fast1 > t_end) t_fast1 = t_end;
      // ... and tiles whose refill (tile t + 1 + NV) is a plain tile of the cache take the main loop (every tile of a
      // piece that holds nothing else).
      int t_plain = tlogical((Lm1 + 1) / BN < t_new ? (Lm1 + 1) / BN : t_new);
      t_plain = t_plain >= t_end ? t_end : t_plain - NV - 1;
      if (t_plain > t_fast) t_plain = t_fast;
      // Prologue.  The first pass finds the ring's fill under way; a second pass fills it again.
      if (exact) prefill(0, NV);
      if (t_begin + NV < t_end)  // every group of the fill is whole
        wait_vm<(NV - 1) * LPG>();
      else
        wait_vm<0>();
      __builtin_amdgcn_s_barrier();
      if (idle) {
        // no rows of its own: this wavefront only moves its share of the tiles (the LDS bandwidth and the power of
        // computing on rows that do not exist would be taken from the wavefronts that have some)
        for (int t = t_begin, ks = 0, vs = 0; t < t_end; ++t) {
          if (NV > 2 && t + NV < t_end)
            wait_vm<(NV - 2) * LPG>();
          else
            wait_vm<0>();
          __builtin_amdgcn_s_barrier();
          issue_tile(false, t + 1 + NV, ks);
          issue_tile(true, t + NV, vs);
          ks = ks + 1 == NK ? 0 : ks + 1;
          vs = vs + 1 == NV ? 0 : vs + 1;
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kg[ks / GK][ks % GK] = k_frag(ks, 0);
        wait_lds<0>();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            if (ks == 0)
              mfma_qk_first(sA[qb], kg[0][0], qf[qb][ks], negm[qb]);
            else
              mfma_qk(sA[qb], kg[ks / GK][ks % GK], qf[qb][ks]);
          }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) mfma_settle_v(sA[qb]);
        if (win || t_begin * BN + 32 > vis_min) mask_half(sA, 2 * t_begin);
        float mx[QB];
        rowmax_all(sA, mx);
        reference_first(mx, sA);
        if (QB == 2 && t_begin >= t_dead && t_dead < t_end)
          early_events(sA, std::integral_constant<int, QB - 1>{});  // the first step already works on unit 1 alone
        else
          early_events(sA, std::integral_constant<int, 0>{});
        // first K batch of the first step: second half of tile t_begin
#pragma unroll
        for (int j = 0; j < GK; ++j) kg[0][j] = k_frag(j, HALFB);
        constexpr std::integral_constant<int, 0> both{};
        constexpr std::false_type even{}, unmasked{}, mixed{};
        constexpr std::true_type odd{}, masked{}, plain{};
        int t = t_begin;
        for (; t < t_lead; ++t) {
          step(sA, sB, 2 * t, even, masked, mixed, both);
          step(sB, sA, 2 * t + 1, odd, masked, mixed, both, t + 1 == t_dead && t_dead < t_end);
        }
        // The main loop's first instructions within the first half of a 32-byte piece of code: a loop whose head lies at the end of one costs
        // every tile a fetch.  4096 tokens on 127K keys, 32 heads on 8, head at byte 4, 8 and 16 of a piece 6392 to 6400 us, 20 6443, 28 6470.
        asm volatile(".p2align 5\n\ts_nop 0");
        for (; t < t_plain; ++t) {
          step(sA, sB, 2 * t, even, unmasked, plain, both);
          step(sB, sA, 2 * t + 1, odd, unmasked, plain, both);
        }
        for (; t < t_fast; ++t) {
          step(sA, sB, 2 * t, even, unmasked, mixed, both);
          step(sB, sA, 2 * t + 1, odd, unmasked, mixed, both);
        }
        for (; t < t_dead; ++t) {
          step(sA, sB, 2 * t, even, masked, mixed, both);
          step(sB, sA, 2 * t + 1, odd, masked, mixed, both, t + 1 == t_dead && t_dead < t_end);
        }
        if constexpr (QB == 2) {
          // unit 0 is done for good (every further key is beyond its last row): unit 1 alone
          constexpr std::integral_constant<int, 1> second{};
          for (; t < t_fast1; ++t) {
            step(sA, sB, 2 * t, even, unmasked, mixed, second);
            step(sB, sA, 2 * t + 1, odd, unmasked, mixed, second);
          }
          for (; t < t_end; ++t) {
            step(sA, sB, 2 * t, even, masked, mixed, second);
            step(sB, sA, 2 * t + 1, odd, masked, mixed, second);
          }
        }
      }
      wait_vm<0>();  // nothing of ours may still be writing LDS when the workgroup retires or starts over
      wait_lds<0>();
      if (!SUM_MODE || exact) {
        __syncthreads();  // every wavefront of the workgroup is through with the rings
        break;
      }
      {
        // Did a row sum of any wavefront overflow?  (The votes have words of their own behind the rings.)
        if (l == 0) *LDS_PTR(int, lds0 + (unsigned)((NK + NV) * TILEB) + 4u * (unsigned)w) = overflowed;
        __syncthreads();  // ... which also finds every wavefront through with the rings
        int any_overflow = 0;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) any_overflow |= *LDS_PTR(const int, lds0 + (unsigned)((NK + NV) * TILEB) + 4u * (unsigned)ww);
        any_overflow = __builtin_amdgcn_readfirstlane(any_overflow);
        if (__builtin_expect(any_overflow == 0, 1)) break;
      }
    }
    mfma_settle_a(o[0][0]);  // (one wait for all; the others are tied behind it)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int db = 0; db < DB; ++db) asm volatile("" : "+a"(o[qb][db]));
  } else {
    reset_state();
  }

  // ---- epilogue.  O^T leaves through LDS (the rings are dead by now): a lane holds four consecutive
  // columns of one row, which stored directly would be 8- or 16-byte pieces scattered over 32 rows per
  // instruction; turned in LDS, every store instruction writes whole rows, 16 bytes per lane.
  // (the lane's place and its row's token and head are formed anew: nothing is held for them through the main loop)
  const int le = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), hie = le >> 5, me = le & 31;
  copy_load(copy_r0);  // (in flight while the results leave)
  constexpr int OROWF = D * 4 + 16;  // padded LDS row: fp32 partials
  constexpr int OROWH = D * 2 + 16;  // padded LDS row: bf16 output
  const unsigned obase = lds0 + (unsigned)(w * kRowsPerUnit * OROWF);  // this wavefront's staging area, reused by its units
  float l_all[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) l_all[qb] = pair_sum(l_run[qb]);

  // ---- two pieces: the later of a row's two wavefronts has them both in the end.  Each leaves its partial results, lane by lane as they lie
  // in its registers, and then counts itself; who finds the count odd is the second, fetches the other's and goes on as if there were one
  // piece.  Nobody waits for anybody.  The counts are even between steps, whatever ran in between.  Partial results by accesses of device
  // scope (past the L2, which the other piece need not share).  The arithmetic is the combine kernel's, in the order of the pieces, so that
  // the bits do not depend on who came second.  Against that kernel: its launch, the turn through LDS, and the second's way through memory.
  bool whole = p.n_splits == 1;
  if (p.merge_count && !idle) {
    constexpr int kDeviceScope = 16, kRawBuffer = 0x00020000;  // sc1; word 3 of a descriptor: untyped
    const unsigned n_waves = (unsigned)(p.n_kv_heads * p.wgs_per_head * kUnitsPerWg), wave = (unsigned)((g * p.wgs_per_head + ug) * kUnitsPerWg + w);
    const unsigned mine = (unsigned)split * n_waves + wave, theirs = (unsigned)(1 - split) * n_waves + wave;
    const __amdgpu_buffer_rsrc_t po = __builtin_amdgcn_make_buffer_rsrc(p.part_o, 0, 2 * n_waves * (unsigned)(QB * DB * 4096), kRawBuffer);
    const __amdgpu_buffer_rsrc_t pml = __builtin_amdgcn_make_buffer_rsrc(p.part_ml, 0, 2 * n_waves * (unsigned)(QB * 512), kRawBuffer);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      uintx2 ml;
      ml[0] = __float_as_uint(m_run[qb]);
      ml[1] = __float_as_uint(l_all[qb]);
      __builtin_amdgcn_raw_buffer_store_b64(ml, pml, (unsigned)le * 8u, (mine * QB + (unsigned)qb) * 512u, kDeviceScope);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          uintx4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(o[qb][db][rg * 4 + e]);
          __builtin_amdgcn_raw_buffer_store_b128(v, po, (unsigned)le * 16u, (mine * QB * DB + (unsigned)(qb * DB + db)) * 4096u + (unsigned)rg * 1024u, kDeviceScope);
        }
    }
    wait_vm<0>();
    unsigned count = 0;
    if (le == 0) count = __hip_atomic_fetch_add(p.merge_count + wave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    whole = __builtin_amdgcn_readfirstlane((int)count) & 1;
    if (whole) {
      asm volatile("" ::: "memory");
      uintx2 ml[QB];
      uintx4 x[QB][DB][4];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        ml[qb] = __builtin_amdgcn_raw_buffer_load_b64(pml, (unsigned)le * 8u, (theirs * QB + (unsigned)qb) * 512u, kDeviceScope);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg)
            x[qb][db][rg] = __builtin_amdgcn_raw_buffer_load_b128(po, (unsigned)le * 16u, (theirs * QB * DB + (unsigned)(qb * DB + db)) * 4096u + (unsigned)rg * 1024u, kDeviceScope);
      }
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float m_b = __uint_as_float(ml[qb][0]), l_b = __uint_as_float(ml[qb][1]), m_a = m_run[qb], l_a = l_all[qb];
        // no visible key for the row in a piece, whose O may be NaN then: 0 times a value that is not finite
        const bool none_a = l_a == 0.f, none_b = l_b == 0.f;
        if (none_a) m_a = -INFINITY;
        if (none_b) m_b = -INFINITY;
        const float m2 = fmaxf(m_a, m_b), ref = m2 == -INFINITY ? 0.f : m2;
        const float f_a = __builtin_amdgcn_exp2f(m_a - ref), f_b = __builtin_amdgcn_exp2f(m_b - ref);
        m_run[qb] = m2;
        l_all[qb] = split == 0 ? __builtin_fmaf(l_b, f_b, l_a * f_a) : __builtin_fmaf(l_a, f_a, l_b * f_b);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float a = none_a ? 0.f : o[qb][db][r], b = none_b ? 0.f : __uint_as_float(x[qb][db][r >> 2][r & 3]);
            o[qb][db][r] = split == 0 ? __builtin_fmaf(b, f_b, a * f_a) : __builtin_fmaf(a, f_a, b * f_b);
          }
      }
    }
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = l_all[qb];
    const unsigned row0 = (unsigned)(unit_of[qb] * kRowsPerUnit);
    // rows of the unit that exist
    const int n_live = !unit_valid[qb] ? 0 : (int)(n_packed - row0) < kRowsPerUnit ? (int)(n_packed - row0) : kRowsPerUnit;
    const bool store_row = hie == 0 && me < n_live;
    // place of the lane's row among the KV head's rows of [token][query head]
    const unsigned my_row = row0 + (unsigned)me, my_tok = quot(my_row, p.by_group), my_place = my_row + my_tok * (unsigned)(Hq - G);
    // `rows` whole rows of `chunks` 16-byte pieces, turned in LDS, to dst (the KV head's first row); few instructions per
    // store and a loop: written out with 64-bit row arithmetic for each store this took 3 us of a workgroup's end
    auto store_rows = [&](unsigned char* dst, auto bytes_tag, unsigned lds_row) __attribute__((always_inline)) {
      constexpr int BYTES = decltype(bytes_tag)::value, CPR = BYTES / 16, RPI = 64 / CPR;
      const unsigned r_lane = (unsigned)le / CPR, c = (unsigned)le % CPR * 16u;
      unsigned char* lane_dst = dst + c;
      unsigned at = obase + r_lane * lds_row + c;
#pragma unroll 1
      for (unsigned i = r_lane; i < (unsigned)kRowsPerUnit; i += 4 * RPI) {
        uintx4 x[4];
#pragma unroll
        for (unsigned j = 0; j < 4; ++j) x[j] = *LDS_PTR(const uintx4, at + j * RPI * lds_row);
#pragma unroll
        for (unsigned j = 0; j < 4; ++j) asm volatile("" : "+v"(x[j]));
#pragma unroll
        for (unsigned j = 0; j < 4; ++j) {
          const unsigned r = i + j * RPI;
          const unsigned at_row = (unsigned)__builtin_amdgcn_ds_bpermute((int)(4 * r), (int)my_place);
          if ((int)r < n_live) __builtin_nontemporal_store(x[j], reinterpret_cast<uintx4*>(lane_dst + (uint64_t)at_row * BYTES));
        }
        at += 4 * RPI * lds_row;
      }
    };
    if (whole) {
      const float inv = 1.f / l_tot;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[qb][db][rg * 4 + e] * inv);
          *LDS_PTR(bf16x4, obase + (unsigned)(me * OROWH + (db * 32 + 8 * rg + 4 * hie) * 2)) = v;
        }
      if (p.lse && store_row)
        p.lse[(int64_t)(g * G + (int)(my_row - my_tok * (unsigned)G)) * C + my_tok] = (m_run[qb] + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;
      store_rows(reinterpret_cast<unsigned char*>(p.out) + (uint64_t)(g * G) * (D * 2), std::integral_constant<int, D * 2>{}, OROWH);
    } else if (!p.merge_count) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          floatx4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = o[qb][db][rg * 4 + e];
          *LDS_PTR(floatx4, obase + (unsigned)(me * OROWF + (db * 32 + 8 * rg + 4 * hie) * 4)) = v;
        }
      const uint64_t first = (uint64_t)split * (uint64_t)(C * Hq) + (uint64_t)(g * G);  // the head's first row of this piece
      if (store_row)
        *reinterpret_cast<float2*>(p.part_ml + (first + my_place) * 2) = make_float2(m_run[qb], l_tot);
      store_rows(reinterpret_cast<unsigned char*>(p.part_o) + first * (D * 4), std::integral_constant<int, D * 4>{}, OROWF);
    }
  }

  copy_store(copy_r0);
  for (int r0 = copy_r0 + kCopyTurns * kCopyRows; r0 < copy_r1; r0 += kCopyTurns * kCopyRows) {
    copy_load(r0);
    copy_store(r0);
  }
}

template <int D, int QB, int NV>
static hipError_t prepare_one() {
  constexpr int lds_bytes = (2 * NV + 1) * kTileKeys * D * 2 + vote_bytes(QB);
  // per device: the attribute belongs to the device's copy of the kernel (idempotent; a benign race at worst
  // sets it twice)
  static bool attr_done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!attr_done[dev]) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_bf16_kernel<D, QB, NV>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    attr_done[dev] = true;
  }
  return hipSuccess;
}

template <int D, int QB, int NV>
static hipError_t launch_one(const AttnParams& p, hipStream_t s) {
  constexpr int lds_bytes = (2 * NV + 1) * kTileKeys * D * 2 + vote_bytes(QB);
  hipError_t e = prepare_one<D, QB, NV>();  // a no-op after kvfold_cache_create
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bf16_kernel<D, QB, NV>), dim3(padded_grid(p.n_wgs)), dim3(256), lds_bytes, s, p);
  return hipGetLastError();
}

template <int D>
static hipError_t prepare_all() {
  hipError_t e = prepare_one<D, 2, kRingAlone>();
  if (D == 128 && e == hipSuccess) e = prepare_one<128, 1, kRingAlone>();
  if (e == hipSuccess) e = prepare_one<D, 1, kRingShared>();
  return e;
}

hipError_t prepare_attn_bf16(int head_dim) {
  return head_dim == 128 ? prepare_all<128>() : head_dim == 64 ? prepare_all<64>() : hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_any(const AttnParams& p, int qb, int n_cu, hipStream_t s) {
  if (qb == 2) return launch_one<D, 2, kRingAlone>(p, s);
  return D == 128 && ring_slots(D, qb, p.n_wgs, n_cu) == kRingAlone ? launch_one<128, 1, kRingAlone>(p, s) : launch_one<D, 1, kRingShared>(p, s);
}

hipError_t launch_attn_bf16(const AttnParams& p, int head_dim, int qb, int n_cu, hipStream_t s) {
  return head_dim == 128 ? launch_any<128>(p, qb, n_cu, s) : head_dim == 64 ? launch_any<64>(p, qb, n_cu, s) : hipErrorInvalidValue;
}

}  // namespace kvfold
