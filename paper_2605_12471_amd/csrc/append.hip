// Cache carry of the fold step (paper Sec. 2 and Fig. 2: the chunk's K/V rows are appended to the
// cache, the prefix is handed on untouched).  Token-major [C][Hkv][d] rows are scattered to the
// head-major cache [Hkv][capacity][d] at rows [len_prev, len_prev + C); a pure bit copy.
//
// HBM-bound: 16 bytes per lane, destination addresses of a wavefront are contiguous (one head's
// rows are adjacent), source addresses are contiguous per row (d * elem_size bytes).
#include "kvfold_internal.h"

namespace kvfold {

// blockIdx.y = 2 * KV head + (0: K, 1: V).  A row is 8, 16 or 32 16-byte vectors (a power of two), so the
// (token, vector) split of an index is a shift and a mask, and one head's destination is one contiguous run.
__global__ void __launch_bounds__(256) append_kernel(AppendParams p, int log2_vpr) {
  const bool is_v = (blockIdx.y & 1) != 0;
  const int64_t g = blockIdx.y >> 1;
  const int64_t vpr = (int64_t)1 << log2_vpr;
  const uint4* __restrict__ src = reinterpret_cast<const uint4*>(is_v ? p.v_new : p.k_new) + g * vpr;
  uint4* __restrict__ dst = reinterpret_cast<uint4*>(is_v ? p.v_cache : p.k_cache) + (g * p.capacity + p.len_prev) * vpr;
  const int64_t per_head = (int64_t)p.n_tokens << log2_vpr;
  const int64_t src_row = (int64_t)p.n_kv_heads << log2_vpr;  // vectors from one token's row to the next
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < per_head; idx += (int64_t)gridDim.x * blockDim.x)
    dst[idx] = src[(idx >> log2_vpr) * src_row + (idx & (vpr - 1))];
}

// The same carry with work on the rows' way into the cache: one pass, where the rotation and the storage round trip after
// it used to be kernels of their own that read the new rows again (1024 tokens, 8 KV heads, both: 5.1 + 5.2 us in two
// launches before, 5.3 us in one now).  A lane owns 16 bytes of a row; launch-latency bound at these sizes.
//
// ROPE, K rows only (Sec. 2: the new tokens' positions continue from the absolute position, so their rotations line up with
// the original sequence).  Element j pairs with element j + d/2 (half-split layout):
//     k'_j = k_j cos_j - k_{j+d/2} sin_j,   k'_{j+d/2} = k_{j+d/2} cos_j + k_j sin_j,
// in fp32 -- the product of the other element with the sine rounded first, then one fused
// multiply-add -- and rounded to the cache's element type (RNE).  The lane reads the 16 bytes half a row away as well.
//
// QUANT, K and V rows: the storage perturbation of the carried cache (Sec. 8, Discussion: a per-step quantisation round
// trip bf16 -> intN -> bf16).  The paper names no quantiser; the reading: one group = the d elements of one (token, KV head)
// row, symmetric,
//   scale = max|x| / (2^(N-1) - 1),  code = round-half-even(x / scale) clamped to +-(2^(N-1) - 1),
//   x' = code * scale,
// all in fp32, stored as bf16 (RNE); an all-zero row stays zero.  The d / 8 lanes of a row agree on the maximum by butterfly
// exchanges inside their lane group.
template <typename T, int E, bool ROPE, bool QUANT>  // element type, elements per 16-byte vector
__global__ void __launch_bounds__(256) append_work_kernel(AppendParams p, int log2_vpr, float qmax) {
  typedef __attribute__((ext_vector_type(E))) T vec_t;
  const bool is_v = (blockIdx.y & 1) != 0;
  const int64_t g = blockIdx.y >> 1;
  const int vpr = 1 << log2_vpr, half = vpr >> 1;
  const vec_t* __restrict__ src = reinterpret_cast<const vec_t*>(is_v ? p.v_new : p.k_new) + g * vpr;
  vec_t* __restrict__ dst = reinterpret_cast<vec_t*>(is_v ? p.v_cache : p.k_cache) + (g * p.capacity + p.len_prev) * vpr;
  const int64_t per_head = (int64_t)p.n_tokens << log2_vpr;  // whole rows: the lanes of a row leave the loop together
  const int64_t src_row = (int64_t)p.n_kv_heads << log2_vpr;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < per_head; idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = idx >> log2_vpr;
    const int c = (int)idx & (vpr - 1);
    const vec_t* row = src + i * src_row;
    vec_t v = row[c];
    if (ROPE && !is_v) {
      const bool lower = c < half;
      const int a = lower ? c : c - half;
      const vec_t other = row[lower ? c + half : a];
      const float* cs = p.rope_cos + (i * half + a) * E;
      const float* sn = p.rope_sin + (i * half + a) * E;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float mine = (float)v[e], theirs = (float)other[e];
        const float t = theirs * sn[e];
        v[e] = (T)__builtin_fmaf(mine, cs[e], lower ? -t : t);
      }
    }
    if (QUANT) {
      float x[E], amax = 0.f;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        x[e] = (float)v[e];
        amax = fmaxf(amax, fabsf(x[e]));
      }
      for (int off = 1; off < vpr; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
      const float scale = amax / qmax;
      if (scale > 0.f) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          float code = rintf(x[e] / scale);
          code = fminf(fmaxf(code, -qmax), qmax);
          v[e] = (T)(code * scale);
        }
      }
    }
    dst[idx] = v;
  }
}

hipError_t launch_append(const AppendParams& p, int storage_bits, hipStream_t s) {
  if (p.n_tokens <= 0 || p.n_kv_heads <= 0) return hipSuccess;
  int log2_vpr = 0;
  while ((16 << log2_vpr) < p.row_bytes) ++log2_vpr;
  if ((16 << log2_vpr) != p.row_bytes || p.n_kv_heads > 32767 || (storage_bits && !p.elem_is_bf16)) return hipErrorInvalidValue;
  const int64_t per_head = (int64_t)p.n_tokens << log2_vpr;
  int64_t bx = (per_head + 255) / 256;
  if (bx > 1024) bx = 1024;
  const dim3 grid((unsigned)bx, (unsigned)(2 * p.n_kv_heads)), block(256);
  const float qmax = storage_bits ? (float)((1 << (storage_bits - 1)) - 1) : 0.f;
  if (p.rope_cos && storage_bits)
    hipLaunchKernelGGL((append_work_kernel<__bf16, 8, true, true>), grid, block, 0, s, p, log2_vpr, qmax);
  else if (storage_bits)
    hipLaunchKernelGGL((append_work_kernel<__bf16, 8, false, true>), grid, block, 0, s, p, log2_vpr, qmax);
  else if (p.rope_cos && p.elem_is_bf16)
    hipLaunchKernelGGL((append_work_kernel<__bf16, 8, true, false>), grid, block, 0, s, p, log2_vpr, qmax);
  else if (p.rope_cos)
    hipLaunchKernelGGL((append_work_kernel<float, 4, true, false>), grid, block, 0, s, p, log2_vpr, qmax);
  else
    hipLaunchKernelGGL(append_kernel, grid, block, 0, s, p, log2_vpr);
  return hipGetLastError();
}

}  // namespace kvfold
