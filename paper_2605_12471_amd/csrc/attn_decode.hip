// Chunk-prefix attention of at most 16 packed rows per KV head (32 where heads are 64 wide), bf16: decoding, one token or a few at a time, every
// key visible up to the row's own position.  A workgroup owns the KV head's one unit and a piece of its keys.  Rounding points as in the
// general bf16 kernel (attn_bf16.hip): queries scaled by scale * log2(e) and rounded once more, P = 2^(S - m) rounded to bf16 for P V, row
// sums in fp32 from the unrounded P, the reference m stale by at most 2^16.
//
// Such a step reads every key once and computes next to nothing: it is bound by memory when the cache is long and, when it is
// short, by the chain of what a launch does once.  So nothing stands between memory and the matrix instructions:
//  * The keys are dealt to four wavefronts in blocks of 32, and each runs alone until the results meet in LDS.
//  * K and V come straight into registers, whole lines at a time, and are waited for one by one by the compiler's own count.  The 16x16x32
//    shapes make that possible.  S^T = K Q^T takes 16 keys as its rows: a lane's share is 16 bytes of one K row, four lanes have a row's 64
//    bytes.  O^T = V^T P^T takes 16 columns of V as its rows, each lane with eight keys: a lane loads its 16 (64 wide: 8) bytes of eight V
//    rows, sixteen lanes a whole row, and one byte permutation per register pairs up the keys of each column.  Instruction j's
//    rows are every eighth (64 wide: fourth) column of the head, from the j-th on, which is only a matter of where O is written to.
//    The keys of a lane's eight P values are those whose S^T it holds, four of each 16.
//  * Two blocks are in flight per wavefront, 32 KB, a block's successor but one as soon as its K (V) is used up.
//  * At most 16 rows (one token of up to 16 heads a group) take half the matrix instructions and exponentials of 32.
// Against the few-rows kernel (attn_few.hip), which takes its blocks through LDS, the steps' own times (captured graphs, caches from memory): one
// token, 32 heads on 8, 128 wide, 93 keys 5.08 -> 3.79 us, 1000 8.34 -> 7.05, 4187 10.75 -> 9.30, 16K 17.8 -> 16.8, 128K 95.1 -> 91.8
// (5.84 TB/s); 64 wide 4187 keys 9.00 -> 8.13.  Over 116 shapes (1 to 64 heads, 1 to 16 tokens on 64 to 127K keys) 0.92 of the time, each at
// its plan.  17 to 32 rows of 128 columns stay there: here they take 392 registers, one wavefront per SIMD, and gained nothing (14 shapes 0.99,
// 8 tokens on 4187 keys, 32 heads on 8, 13.0 / 12.9; 2 on 115K, 32 on 2, 29.9 / 32.4).  Nor do long ranges of one or two KV heads come
// here, whose pieces leave half the CUs without a workgroup (plan_with(); one token on 88K keys, 32 heads on 2, 128 workgroups, 24.7 / 25.7).
#include <type_traits>

#include "append_rows.h"
#include "kvfold_internal.h"
#include "meet.h"
#include "wave_ops.h"

namespace kvfold {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) unsigned uintx4;
typedef __attribute__((ext_vector_type(2))) unsigned uintx2;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(2))) float floatx2;

#define GLOBAL_PTR(T, p) ((T __attribute__((address_space(1)))*)(p))

constexpr int kDecodeWaves = 4;

// NC: groups of 16 rows (1: at most 16 packed rows).
template <int D, int NC>
__global__ void __launch_bounds__(kDecodeWaves * 64, 2) attn_decode_kernel(AttnParams p) {
  constexpr int NW = kDecodeWaves, NT = NW * 64;
  constexpr int CH = D / 8, ROWB = D * 2, KS = D / 32;  // 16-byte chunks and bytes of a row, contraction steps of S^T
  constexpr int J = D / 16;                             // matrix instructions of P V, and columns of a lane's share of a V row
  constexpr int VW = D / 32;                            // registers of that share
  constexpr float kStale = 16.0f;                       // log2 units
  constexpr int ROWS = NC * 16, OROW = D * 4 + 16;
  __shared__ __attribute__((aligned(16))) unsigned char red_o[NW * ROWS * OROW];
  __shared__ floatx2 red_ml[NW * ROWS];
  __shared__ int last;

  // every line of the arguments is fetched now, in one round trip (they are not in the scalar cache yet)
  asm volatile("" ::"s"(p.q), "s"(p.n_tokens), "s"(p.len_prev), "s"(p.k_new), "s"(p.work_k), "s"(p.by_group.mul), "s"(p.copy_rows));

  const int lid = logical_workgroup(blockIdx.x, gridDim.x, p);
  if (lid >= p.n_wgs) return;
  const int g = (int)quot((unsigned)lid, p.by_wgs_per_kvh);
  const int split = lid - g * p.n_splits;  // one workgroup per KV head and piece

  const int tid = threadIdx.x, l = tid & 63, kg = l >> 4, c16 = l & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C = p.n_tokens, Hq = p.n_q_heads, G = p.group;
  const int rows = C * G;  // the KV head's packed rows: row j is token j / G, head j % G of the group

  // ---- Q, ahead of everything else that comes from memory; lane (c16, kg) holds q[16 nc + c16][32 ks + 8 kg + j]
  int tok[NC], my_vis[NC];
  bf16x8 qf[NC][KS];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    const int r = nc * 16 + c16, row = r < rows ? r : rows - 1;
    tok[nc] = (int)quot((unsigned)row, p.by_group);
    my_vis[nc] = (int)p.len_prev + tok[nc] + 1;
    const unsigned place = (unsigned)(row + tok[nc] * (Hq - G) + g * G);
    const __bf16* qrow = reinterpret_cast<const __bf16*>(p.q) + (uint64_t)place * D + kg * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[nc][ks] = *reinterpret_cast<const bf16x8*>(qrow + ks * 32);
  }

  const int vis_first = (int)p.len_prev + 1, vis_last = (int)p.len_prev + C;
  const TileMap tm = {0, 0, (int)(((unsigned)vis_last + kTileKeys - 1) / kTileKeys)};
  const bool fused = p.k_new != nullptr;
  const KeyRange kr = key_range(tm, split, p.tiles_per_split, p.len_prev, C, fused);
  const int b_all = (int)(((unsigned)vis_last + 31) / 32), b_end = 2 * kr.t_end < b_all ? 2 * kr.t_end : b_all;

  const unsigned head_bytes = (unsigned)p.capacity * (unsigned)ROWB;  // (below 2^32, as the host checks)
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(p.k_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(p.v_cache) + (uint64_t)(unsigned)g * head_bytes;
  const unsigned new_stride = (unsigned)(p.n_kv_heads * ROWB);
  const unsigned char* knew = reinterpret_cast<const unsigned char*>(p.k_new) + (unsigned)g * (unsigned)ROWB;
  const unsigned char* vnew = reinterpret_cast<const unsigned char*>(p.v_new) + (unsigned)g * (unsigned)ROWB;

  // ---- the angles of the rows and this workgroup's share of the append, ahead of the long loads as well
  constexpr int RS = KS / 2;
  floatx4 cs[NC][RS][2], sn[NC][RS][2];
  if (p.rope_cos) {
#pragma unroll
    for (int nc = 0; nc < NC; ++nc)
#pragma unroll
      for (int ks = 0; ks < RS; ++ks)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          cs[nc][ks][h] = *reinterpret_cast<const floatx4*>(p.rope_cos + tok[nc] * (D / 2) + ks * 32 + kg * 8 + h * 4);
          sn[nc][ks][h] = *reinterpret_cast<const floatx4*>(p.rope_sin + tok[nc] * (D / 2) + ks * 32 + kg * 8 + h * 4);
        }
  }
  // Rows [copy_r0, copy_r1) of K and V, 16 bytes per thread and turn; the first turn is loaded here.
  const int copy_r0 = fused ? split * p.copy_rows : 0, copy_r1 = fused ? (copy_r0 + p.copy_rows < C ? copy_r0 + p.copy_rows : C) : 0;
  const int copy_n = copy_r1 > copy_r0 ? (copy_r1 - copy_r0) * CH : 0;
  auto copy_at = [&](int i, bool& is_v, int& r, int& c) __attribute__((always_inline)) {
    is_v = i >= copy_n;
    const int e = is_v ? i - copy_n : i;
    r = copy_r0 + e / CH;
    c = e % CH;
  };
  auto copy_load = [&](int i) __attribute__((always_inline)) -> uintx4 {
    bool is_v;
    int r, c;
    copy_at(i, is_v, r, c);
    return *GLOBAL_PTR(const uintx4, (uint64_t)(uintptr_t)(is_v ? vnew : knew) + (unsigned)r * new_stride + (unsigned)c * 16);
  };
  auto copy_store = [&](int i, const uintx4& x) __attribute__((always_inline)) {
    bool is_v;
    int r, c;
    copy_at(i, is_v, r, c);
    __builtin_nontemporal_store(x, reinterpret_cast<uintx4*>(const_cast<unsigned char*>(is_v ? vbase : kbase) + (p.len_prev + r) * ROWB + c * 16));
  };
  uintx4 copied;
  if (copy_n > 0) copied = copy_load(tid < 2 * copy_n ? tid : 2 * copy_n - 1);

  // The wavefront's blocks of 32 keys are every NW-th of the piece's.  All but its last are plain: their rows exist and lie before the old
  // cache's end.  The last may reach beyond (at most 32 rows do); each of its rows then comes from the cache or the chunk, or is redirected
  // to the piece's last row (and masked).  That block comes first; the plain ones follow in cyclic order from a place that differs from
  // piece to piece and head to head: pieces and heads lie powers of two apart, and workgroups in step would ask the same few memory
  // channels for their rows.
  const int b_first = 2 * kr.t_begin + w, n_blocks = b_first < b_end ? (int)((unsigned)(b_end - b_first + NW - 1) / (unsigned)NW) : 0;
  const int b_last = b_first + NW * (n_blocks - 1);
  const bool special = (unsigned)b_last * 32u + 31u > kr.row_lim || (unsigned)b_last * 32u + 31u >= kr.chunk_row0;
  const int n_plain = n_blocks - (special ? 1 : 0), b_plain = b_first + NW * n_plain;
  auto next = [&](int x) __attribute__((always_inline)) -> int { return x + NW < b_plain ? x + NW : b_first; };

  // A block's rows: K rows c16 and 16 + c16, V rows 4 kg + e and 16 + 4 kg + e (e < 4).  Plain blocks come by buffer loads: a lane's place in a
  // block is fixed, the block's is a scalar, and a block that does not exist (past the last) is asked for in an empty buffer, which costs
  // no traffic, so that the loads in flight are the same on every path and the compiler can count them.
  struct KBlock {
    uintx4 f[2][KS];
  };
  typedef __attribute__((ext_vector_type(VW))) unsigned vvec;
  struct VBlock {
    vvec d[8];
  };
  const unsigned k_lane = (unsigned)c16 * ROWB + (unsigned)kg * 16, v_lane = (unsigned)(4 * kg) * ROWB + (unsigned)c16 * (VW * 4);
  auto load_k = [&](KBlock& x, int blk, bool there) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(kbase), 0, there ? head_bytes : 0u, kRawBuffer);
    const unsigned at = (unsigned)blk * (32u * ROWB);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) x.f[t][ks] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rows, k_lane + ks * 64, at + t * 16 * ROWB, 0));
  };
  auto load_v = [&](VBlock& x, int blk, bool there) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(vbase), 0, there ? head_bytes : 0u, kRawBuffer);
    const unsigned at = (unsigned)blk * (32u * ROWB);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const unsigned voff = v_lane + (e & 3) * ROWB, soff = at + (e >> 2) * 16 * ROWB;
      if constexpr (VW == 4)
        x.d[e] = __builtin_bit_cast(vvec, __builtin_amdgcn_raw_buffer_load_b128(rows, voff, soff, 0));
      else
        x.d[e] = __builtin_bit_cast(vvec, __builtin_amdgcn_raw_buffer_load_b64(rows, voff, soff, 0));
    }
  };

  // A chunk whose rows need work on their way (append_rows.h): this workgroup, the only one of its piece, appends those it is going
  // to read, ahead of its first block.
  int work_r0 = 0, work_r1 = 0;
  if (__builtin_expect(p.work_k && kr.t_begin < kr.t_end, 0)) {
    work_r0 = kr.t_begin * kTileKeys - (int)p.len_prev;
    if (work_r0 < 0) work_r0 = 0;
    work_r1 = (int)kr.row_lim + 1 - (int)p.len_prev;
  }
  if (__builtin_expect(work_r1 > work_r0, 0)) {
    append_work_rows<D>(reinterpret_cast<const unsigned char*>(p.work_k) + g * ROWB, reinterpret_cast<const unsigned char*>(p.work_v) + g * ROWB, new_stride,
                        const_cast<unsigned char*>(kbase) + (uint64_t)p.len_prev * ROWB, const_cast<unsigned char*>(vbase) + (uint64_t)p.len_prev * ROWB,
                        p.rope_cos, p.rope_sin, p.work_qmax, work_r0, work_r1, tid);
    __syncthreads();
  }

  auto rotate_q = [&]() __attribute__((always_inline)) {
    if (p.rope_cos) {
      // rotary embedding, bit for bit that of a caller who rotates and stores bf16 (see attn_bf16.hip)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int ks = 0; ks < RS; ++ks) {
          const bf16x8 lo = qf[nc][ks], up = qf[nc][ks + RS];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float c = cs[nc][ks][e >> 2][e & 3], s = sn[nc][ks][e >> 2][e & 3], tl = (float)up[e] * s, tu = (float)lo[e] * s;
            qf[nc][ks][e] = (__bf16)__builtin_fmaf((float)lo[e], c, -tl);
            qf[nc][ks + RS][e] = (__bf16)__builtin_fmaf((float)up[e], c, tu);
          }
        }
    }
  };
  auto scale_q = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int nc = 0; nc < NC; ++nc)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[nc][ks][e] = (__bf16)((float)qf[nc][ks][e] * p.scale_log2e);
  };
  floatx4 o[NC][J];
  float m_run[NC], l_run[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    m_run[nc] = -INFINITY;
    l_run[nc] = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) o[nc][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // S^T of a block, masked; then P and the reference; then O
  floatx4 s[NC][2];
  auto logits = [&](const KBlock& x, int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int nc = 0; nc < NC; ++nc)
#pragma unroll
      for (int t = 0; t < 2; ++t) s[nc][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) s[nc][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x.f[t][ks]), qf[nc][ks], s[nc][t], 0, 0, 0);
    const int key0 = blk * 32;
    if (__builtin_expect(key0 + 32 > vis_first, 0)) {  // wave-uniform: some row does not see the whole block
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) {
        const int rel = my_vis[nc] - key0 - 4 * kg;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if ((e >> 2) * 16 + (e & 3) >= rel) s[nc][e >> 2][e & 3] = -INFINITY;
      }
    }
  };
  uintx4 pb[NC];  // P^T fragments: the lane's eight keys
  auto weights = [&]() __attribute__((always_inline)) {
    bool mine[NC];
    float mx[NC];
    bool any = false;
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
      mx[nc] = fmaxf(fmaxf(fmaxf(s[nc][0][0], s[nc][0][1]), fmaxf(s[nc][0][2], s[nc][0][3])), fmaxf(fmaxf(s[nc][1][0], s[nc][1][1]), fmaxf(s[nc][1][2], s[nc][1][3])));
      mx[nc] = pair_max(row16_max(mx[nc]));
      // only rows that ask for it move, so a row's arithmetic never depends on its wave neighbours
      mine[nc] = mx[nc] > m_run[nc] + kStale || (m_run[nc] == -INFINITY && mx[nc] > -INFINITY);
      any |= mine[nc];
    }
    if (__any(any)) {
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) {
        const float m2 = mine[nc] ? mx[nc] : m_run[nc];
        const float alpha = m_run[nc] == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run[nc] - m2);  // (without history: l = 0, O = 0)
        m_run[nc] = m2;
        l_run[nc] *= alpha;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[nc][j][r] *= alpha;
      }
    }
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
      const float ref = m_run[nc] == -INFINITY ? 0.f : m_run[nc];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float a = __builtin_amdgcn_exp2f(s[nc][k >> 1][2 * (k & 1)] - ref), c = __builtin_amdgcn_exp2f(s[nc][k >> 1][2 * (k & 1) + 1] - ref);
        l_run[nc] += a;
        l_run[nc] += c;
        bf16x2 pk;
        pk[0] = (__bf16)a;
        pk[1] = (__bf16)c;
        pb[nc][k] = __builtin_bit_cast(unsigned, pk);
      }
    }
  };
  auto outputs = [&](const VBlock& x) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      uintx4 a;
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = __builtin_amdgcn_perm(x.d[2 * k + 1][j >> 1], x.d[2 * k][j >> 1], j & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
        o[nc][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, pb[nc]), o[nc][j], 0, 0, 0);
    }
  };

  if (n_blocks > 0) {
    KBlock ka, kb;
    VBlock va, vb;
    int b = special ? b_last : 0, bp = b_first + NW * (int)(((((unsigned)(split * 8 + g) * 40503u) & 0xffffu) * (unsigned)n_plain) >> 16);
    if (!special) {
      b = bp;
      bp = next(bp);
    }
    {
      uint64_t k_at[2], v_at[8];
      if (special) {
        // (few lanes' worth of arithmetic and no branches: the row's source is chosen by its base)
        const uint64_t kc = (uint64_t)(uintptr_t)kbase, vc = (uint64_t)(uintptr_t)vbase, kn = (uint64_t)(uintptr_t)knew, vn = (uint64_t)(uintptr_t)vnew;
        auto row_at = [&](uint64_t cache, uint64_t chunk, int key) __attribute__((always_inline)) -> uint64_t {
          const DmaRow src = dma_row(kr, 0, key);
          return (src.from_chunk ? chunk : cache) + src.row * (src.from_chunk ? new_stride : (unsigned)ROWB);
        };
#pragma unroll
        for (int t = 0; t < 2; ++t) k_at[t] = row_at(kc, kn, b * 32 + t * 16 + c16) + (unsigned)kg * 16;
#pragma unroll
        for (int e = 0; e < 8; ++e) v_at[e] = row_at(vc, vn, b * 32 + (e >> 2) * 16 + 4 * kg + (e & 3)) + (unsigned)c16 * (VW * 4);
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) k_at[t] = (uint64_t)(uintptr_t)kbase + ((unsigned)(b * 32 + t * 16) * ROWB + k_lane);
#pragma unroll
        for (int e = 0; e < 8; ++e) v_at[e] = (uint64_t)(uintptr_t)vbase + ((unsigned)(b * 32 + (e >> 2) * 16 + (e & 3)) * ROWB + v_lane);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ka.f[t][ks] = *GLOBAL_PTR(const uintx4, k_at[t] + ks * 64);
#pragma unroll
      for (int e = 0; e < 8; ++e) va.d[e] = *GLOBAL_PTR(const vvec, v_at[e]);
    }
    int b2 = bp, left = n_blocks;
    asm volatile("" ::: "memory");
    rotate_q();
    load_k(kb, b2, left > 1);
    asm volatile("" ::: "memory");
    scale_q();
    logits(ka, b);
    load_v(vb, b2, left > 1);
    asm volatile("" ::: "memory");
#pragma unroll 1
    while (left > 2) {
      const int b3 = next(b2), b4 = next(b3);
      load_k(ka, b3, true);
      asm volatile("" ::: "memory");
      weights();
      outputs(va);
      load_v(va, b3, true);
      asm volatile("" ::: "memory");
      logits(kb, b2);
      load_k(kb, b4, left > 3);
      asm volatile("" ::: "memory");
      weights();
      outputs(vb);
      load_v(vb, b4, left > 3);
      asm volatile("" ::: "memory");
      b = b3;
      b2 = b4;
      left -= 2;
      logits(ka, b);
    }
    weights();
    outputs(va);
    if (left == 2) {
      logits(kb, b2);
      weights();
      outputs(vb);
    }
  }

  // ---- the append: stored ahead of the output, which may lie on the rows
  if (tid < 2 * copy_n) copy_store(tid, copied);
  for (int i = tid + NT; i < 2 * copy_n; i += NT) copy_store(i, copy_load(i));

  // ---- the wavefronts' results meet in LDS: [wavefront][row][D] and [wavefront][row] (m, l)
  float l_tot[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    l_tot[nc] = pair_sum(row16_sum(l_run[nc]));
    if (__builtin_expect(b_first * 32 >= vis_first, 0) && l_tot[nc] == 0.f) {
      // rows that saw none of the wavefront's keys: O may be NaN, 0 times a value that is not finite
#pragma unroll
      for (int j = 0; j < J; ++j) o[nc][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int r = nc * 16 + c16;
    if (r < rows) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < J; jj += 4) {
          const floatx4 v = {o[nc][jj][i], o[nc][jj + 1][i], o[nc][jj + 2][i], o[nc][jj + 3][i]};
          *reinterpret_cast<floatx4*>(red_o + (w * ROWS + r) * OROW + ((4 * kg + i) * J + jj) * 4) = v;
        }
      if (kg == 0) red_ml[w * ROWS + r] = floatx2{m_run[nc], l_tot[nc]};
    }
  }
  __syncthreads();

  constexpr int V = D / 4;  // 16-byte column vectors of a row
  const int c = tid % V;
  const int64_t n_rows = (int64_t)C * Hq;
  const Partials<D> parts(p);
#pragma unroll 1
  for (int r = tid / V; r < rows; r += NT / V) {
    floatx2 ml[NW];
    float M = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      ml[ww] = red_ml[ww * ROWS + r];
      M = fmaxf(M, ml[ww].x);
    }
    float L = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(red_o + (ww * ROWS + r) * OROW + c * 16);
      const float f = ml[ww].y == 0.f ? 0.f : __builtin_amdgcn_exp2f(ml[ww].x - M);  // (0: it saw no visible key)
      L += f * ml[ww].y;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += f * x[e];
    }
    const int t = (int)quot((unsigned)r, p.by_group), h = g * G + r - t * G;
    const int64_t at = (int64_t)t * Hq + h;
    if (p.n_splits == 1) {
      const float inv = 1.f / L;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[e] * inv);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + at * D + c * 4) = v;
      if (p.lse && c == 0) p.lse[(int64_t)h * C + t] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
    } else {
      if (p.meet_count) {
        parts.store(split, (unsigned)at, c, acc, M, L);
      } else {
        *reinterpret_cast<floatx4*>(p.part_o + ((int64_t)split * n_rows + at) * D + c * 4) = acc;
        if (c == 0) *reinterpret_cast<float2*>(p.part_ml + ((int64_t)split * n_rows + at) * 2) = make_float2(M, L);
      }
    }
  }
  if (!p.meet_count || !last_to_meet(p, g, &last)) return;
  // a row or two per wavefront
  const int cv = l % V, part = l / V;
  auto finish = [&](auto pieces, auto per_wave) __attribute__((always_inline)) {
    constexpr int B = decltype(per_wave)::value;
    unsigned at[B];
    int at_lse[B];
    floatx4 acc[B];
    float M[B], L[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int r = w + j * NW < rows ? w + j * NW : rows - 1, t = (int)quot((unsigned)r, p.by_group), h = g * G + r - t * G;
      at[j] = (unsigned)(t * Hq + h);
      at_lse[j] = h * C + t;
    }
    parts.template merge<decltype(pieces)::value, B>(at, part, cv, acc, M, L);
#pragma unroll
    for (int j = 0; j < B; ++j) {
      if (w + j * NW >= rows || part != 0) continue;
      const float inv = 1.f / L[j];
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[j][e] * inv);
      *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + (int64_t)at[j] * D + cv * 4) = v;
      if (p.lse && cv == 0) p.lse[at_lse[j]] = (M[j] + __builtin_amdgcn_logf(L[j])) * 0.6931471805599453f;
    }
  };
  constexpr std::integral_constant<int, kMeetSplitsFew * V / 64 * (D == 64 ? 2 : 1)> few{};
  constexpr std::integral_constant<int, kMeetSplits * V / 64> many{};
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};
  const bool little = p.n_splits <= decltype(few)::value * 64 / V;
  if (rows <= NW)
    little ? finish(few, one) : finish(many, one);
  else if (D == 128 || little)
    finish(few, two);
  else
    finish(many, two);
}

template <int D, int NC>
static void launch_decode_one(const AttnParams& p, hipStream_t s) {
  hipLaunchKernelGGL((attn_decode_kernel<D, NC>), dim3(padded_grid(p.n_wgs)), dim3(kDecodeWaves * 64), 0, s, p);
}

hipError_t launch_attn_decode(const AttnParams& p, int head_dim, hipStream_t s) {
  const bool few = p.n_tokens * p.group <= 16;
  if (head_dim == 128 && few)
    launch_decode_one<128, 1>(p, s);
  else if (head_dim == 64)
    few ? launch_decode_one<64, 1>(p, s) : launch_decode_one<64, 2>(p, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace kvfold
