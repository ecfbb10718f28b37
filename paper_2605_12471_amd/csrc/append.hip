// Cache carry of the fold step (paper Sec. 2 and Fig. 2: the chunk's K/V rows are appended to the
// cache, the prefix is handed on untouched).  Token-major [C][Hkv][d] rows are scattered to the
// head-major cache [Hkv][capacity][d] at rows [len_prev, len_prev + C); a pure bit copy.
//
// HBM-bound: 16 bytes per lane, destination addresses of a wavefront are contiguous (one head's
// rows are adjacent), source addresses are contiguous per row (d * elem_size bytes).
#include "append_rows.h"
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
// The arithmetic is in append_rows.h.
template <typename T, int E, bool ROPE, bool QUANT>  // element type, elements per 16-byte vector
__global__ void __launch_bounds__(256) append_work_kernel(AppendParams p, int log2_vpr, float qmax) {
  typedef row_vec<T, E> vec_t;
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
      rotate_vec<T, E>(v, other, p.rope_cos + (i * half + a) * E, p.rope_sin + (i * half + a) * E, lower);
    }
    if (QUANT) round_trip_vec<T, E>(v, vpr, qmax);
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
