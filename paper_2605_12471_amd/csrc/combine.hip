// Merge of split-prefix partial results.  When a chunk has too few rows to fill the chip, the key
// range of one fold step (paper Sec. 2: keys K_{0:t}) is cut into S contiguous pieces handled by
// different workgroups; each leaves, per (row, head), its running maximum m_s (log2 units), the
// sum l_s of 2^(logit - m_s) and the unnormalised O_s.  Softmax over the union is recovered exactly:
//   M = max_s m_s,  L = sum_s l_s 2^(m_s - M),  out = sum_s O_s 2^(m_s - M) / L.
// HBM-bound (reads S * (d + 2) floats per row once, writes d elements); launch-latency bound for few rows.
#include "kvfold_internal.h"

namespace kvfold {

// Thread layout of a 256-thread block: rows x SG split groups x V 16-byte column vectors (V = head_dim / 4), all powers of
// two, so that a thread finds its place by shifts.  All loads of a thread's pieces, up to eight, are in flight together, and
// their weights are taken against one maximum.  Against the form before (run-time divisions, four pieces at a time folded one
// by one), the kernel in a trace of steps: 32 rows x 17 pieces 3.9 -> 3.3 us, 1184 x 27 6.6 -> 5.9, 3584 x 18 9.5 -> 8.4, 8192 x 8 9.7 ->
// 8.7, 32768 x 2 10.6 -> 9.2 (4.6 TB/s), 1024 x 56 9.1 -> 7.9, 2048 x 40 10.3 -> 10.0.
// Split group sg of a row folds pieces sg, sg + SG, ..., at most eight, into one (m, l, O); the SG results meet in LDS.  With few
// rows (decode-shaped steps: 32 rows, 64 pieces) this keeps every load of a row in flight at once instead of walking the
// pieces one after another.
constexpr int kCombineThreads = 256;
constexpr int kBatch = 8;  // pieces of a thread, at most: their loads are in flight together

// (Four wavefronts per SIMD asked for: the compiler then takes 64 registers, else 92, and 32768 x 2 takes 10.8 us.)
template <int LV>  // log2 V
__global__ void __launch_bounds__(kCombineThreads, 4) combine_kernel(CombineParams p, int log2_sg, unsigned dealt) {
  constexpr unsigned V = 1u << LV, D = 4 * V;
  extern __shared__ __attribute__((aligned(16))) float red[];  // [rows][SG][V] partial O (16 bytes each), then [rows][SG] (m, l)
  typedef __attribute__((ext_vector_type(4))) float floatx4;
  typedef __attribute__((ext_vector_type(2))) float floatx2;
  const unsigned tid = threadIdx.x, SG = 1u << log2_sg;
  const unsigned dv = tid & (V - 1), grp = tid >> LV, sg = grp & (SG - 1), rl = grp >> log2_sg;
  // The hardware hands block b to XCD b % 8; the first `dealt` blocks are neighbours on one XCD instead (launch_combine()).
  const unsigned b = blockIdx.x, block = b < dealt ? b % kNumXcd * (dealt / kNumXcd) + b / kNumXcd : b;
  const unsigned row = block * (kCombineThreads >> (LV + log2_sg)) + rl, n_rows = (unsigned)p.n_rows;
  const bool live = row < n_rows;
  floatx4* red_o = reinterpret_cast<floatx4*>(red);
  floatx2* red_ml = reinterpret_cast<floatx2*>(red + kCombineThreads * 4);

  // (row, piece) pairs are at most 2^19 of at most 512 bytes: 32-bit offsets
  const unsigned char* po = reinterpret_cast<const unsigned char*>(p.part_o);
  const unsigned char* pml = reinterpret_cast<const unsigned char*>(p.part_ml);
  static_assert(kMaxSplits <= kBatch * (kCombineThreads >> 5), "a thread's pieces in one batch, whatever the width");
  // (Pieces and rows past the last are read as the last: a load under a lane's own condition is waited for on the way to the next.)
  floatx2 ml[kBatch];
  floatx4 o[kBatch];
  const unsigned n_splits = (unsigned)p.n_splits, from = row < n_rows ? row : n_rows - 1;
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    if (u * SG >= n_splits) break;
    const unsigned s = u * SG + sg, at = (s < n_splits ? s : n_splits - 1) * n_rows + from;
    ml[u] = *reinterpret_cast<const floatx2*>(pml + at * 8u);
    o[u] = *reinterpret_cast<const floatx4*>(po + at * (D * 4u) + dv * 16u);
  }
  float m = -INFINITY, l = 0.f;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    if (u * SG >= n_splits) break;
    if (u * SG + sg >= n_splits) ml[u].y = 0.f;
    if (ml[u].y == 0.f) {  // no visible key for the row in this piece, whose O may be NaN: 0 times a value that is not finite
      ml[u].x = -INFINITY;
      o[u] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    m = fmaxf(m, ml[u].x);
  }
  {
    const float ref = m == -INFINITY ? 0.f : m;  // (-inf: every logit of the row is, or it sees nothing of these pieces)
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (u * SG >= n_splits) break;
      const float b = __builtin_amdgcn_exp2f(ml[u].x - ref);
      l = __builtin_fmaf(ml[u].y, b, l);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(o[u][e], b, acc[e]);
    }
  }
  if (SG > 1) {
    red_o[tid] = acc;  // [row of the block][split group][column vector]
    if (dv == 0) red_ml[grp] = floatx2{m, l};
    __syncthreads();
    if (sg != 0) return;
    for (unsigned g = 1; g < SG; ++g) m = fmaxf(m, red_ml[grp + g].x);
    const float ref = m == -INFINITY ? 0.f : m;
    const float b0 = __builtin_amdgcn_exp2f(red_ml[grp].x - ref);
    l *= b0;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= b0;
    for (unsigned g = 1; g < SG; ++g) {
      const floatx2 x = red_ml[grp + g];
      const floatx4 o = red_o[tid + (g << LV)];
      const float b = __builtin_amdgcn_exp2f(x.x - ref);
      l = __builtin_fmaf(x.y, b, l);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(o[e], b, acc[e]);
    }
  }
  if (!live) return;

  const float inv = 1.f / l;
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] *= inv;
  if (p.out_is_bf16) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[e];
    *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + (uint64_t)row * D + dv * 4) = v;
  } else {
    *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + (uint64_t)row * D + dv * 4) = acc;
  }
  if (p.lse && dv == 0) {
    const unsigned tok = row / (unsigned)p.n_q_heads, head = row - tok * (unsigned)p.n_q_heads;
    p.lse[(uint64_t)head * (unsigned)p.n_tokens + tok] = (m + log2f(l)) * 0.6931471805599453f;
  }
}

hipError_t launch_combine(const CombineParams& p, hipStream_t s) {
  if (p.n_rows <= 0) return hipSuccess;
  const int lv = p.head_dim == 128 ? 5 : 4, V = 1 << lv;
  // Split groups (a power of two, at most the number of pieces and what one row's share of a block
  // allows) as far as they are needed to put a thread's pieces into one batch, and about two blocks on every CU: with
  // many rows one thread per (row, column vector) walking the pieces is the cheaper form.
  const int64_t blocks1 = ((int64_t)p.n_rows * V + kCombineThreads - 1) / kCombineThreads;
  int lsg = 0;
  while ((1 << lsg) < p.n_splits && (2 << lsg) * V <= kCombineThreads && ((blocks1 << lsg) < 512 || p.n_splits > kBatch << lsg)) ++lsg;
  const int rows_per_block = kCombineThreads >> (lv + lsg);
  const dim3 grid((unsigned)((p.n_rows + rows_per_block - 1) / rows_per_block)), block(kCombineThreads);
  // More groups for the pieces' sake leave a block one of the sixteen rows that share a line of (m, l): neighbouring rows go to one
  // XCD then.  Whole steps, with blocks as they come / dealt: 1024 rows x 56 pieces 28.1 / 26.4 us, 2048 x 40 48.2 / 46.8.  Nowhere
  // else: blocks of four rows follow the KV heads of groups of four, and find in their L2 what the attention kernel wrote
  // from there (121 tokens, 32 heads on 8, 8 pieces 23.2 / 25.9, 64 wide, 66 tokens, 12 pieces 14.4 / 15.4); 45 tokens, 8 heads on
  // 2, 53 pieces 21.0 / 22.7; 3584 x 18 43.6 / 43.9.
  const bool for_pieces = lsg > 0 && blocks1 << (lsg - 1) >= 512;
  const unsigned dealt = for_pieces && rows_per_block == 1 ? grid.x / kNumXcd * kNumXcd : 0;
  const size_t lds = lsg ? kCombineThreads * 16 + (kCombineThreads >> lv) * 8 : 0;
  if (lv == 5)
    hipLaunchKernelGGL(combine_kernel<5>, grid, block, lds, s, p, lsg, dealt);
  else
    hipLaunchKernelGGL(combine_kernel<4>, grid, block, lds, s, p, lsg, dealt);
  return hipGetLastError();
}

}  // namespace kvfold
