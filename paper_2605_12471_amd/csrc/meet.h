// The pieces of a step meet in the attention kernel: the last workgroup of a unit to have stored its partial results merges them all.  For kernels
// of one unit a workgroup, where that is little to read.  Against the combine kernel (captured graphs, one token, 32 heads on 8): 500 keys 6.74 -> 5.75 us,
// 1000 7.03 -> 6.44, 4187 9.48 -> 8.68, 9000 12.4 -> 11.7, 64 wide 1000 6.66 -> 5.36, 4187 8.18 -> 6.60.  The counters of two KV heads lie 256 bytes apart: next
// to one another the atomics of all heads waited for each other, 0.1 us for every piece (17 pieces of 8 heads 9.56 us, apart 8.90).  A
// wavefront has a row, or two (64 heads on 8, 600 keys 6.97 -> 6.17, 64 wide 28 on 4, 1300 6.89 -> 5.95, 6000 8.0 -> 7.2); two of 128 columns with many pieces
// are more than it has registers in flight for (28 on 4, 2331 keys 7.9 / 8.7 us with 19), and 16 rows a second way through memory (10.4 / 11.3).
#pragma once
#include "kvfold_internal.h"
#include "wave_ops.h"

namespace kvfold {

constexpr int kDeviceScope = 16;        // sc1 of a buffer access: past the L2, which another piece's workgroup need not share
constexpr int kRawBuffer = 0x00020000;  // word 3 of a buffer descriptor: untyped

// The partial results of row `at` of [token][query head], column vector c (four floats): O and, from one thread, (m, l).
template <int D>
struct Partials {
  typedef __attribute__((ext_vector_type(4))) unsigned uintx4;
  typedef __attribute__((ext_vector_type(2))) unsigned uintx2;
  typedef __attribute__((ext_vector_type(4))) float floatx4;
  __amdgpu_buffer_rsrc_t o, ml;
  unsigned n_rows;
  __device__ __forceinline__ Partials(const AttnParams& p) : n_rows((unsigned)(p.n_tokens * p.n_q_heads)) {
    o = __builtin_amdgcn_make_buffer_rsrc(p.part_o, 0, (unsigned)p.n_splits * n_rows * (D * 4u), kRawBuffer);
    ml = __builtin_amdgcn_make_buffer_rsrc(p.part_ml, 0, (unsigned)p.n_splits * n_rows * 8u, kRawBuffer);
  }
  __device__ __forceinline__ void store(int piece, unsigned at, int c, const floatx4& x, float m, float l) const {
    const unsigned row = (unsigned)piece * n_rows + at;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, x), o, row * (D * 4u) + (unsigned)c * 16u, 0, kDeviceScope);
    if (c == 0) {
      uintx2 y;
      y[0] = __float_as_uint(m);
      y[1] = __float_as_uint(l);
      __builtin_amdgcn_raw_buffer_store_b64(y, ml, row * 8u, 0, kDeviceScope);
    }
  }
  // The pieces of B rows, at most N * 64 / V of each (V = D / 4 column vectors), by one wavefront: lane (part, c) takes every 64 / V-th of them
  // from the part-th on, then the parts meet; every lane has O, m and l in the end.  Every load is in flight before the first is waited
  // for; those past the last piece lie outside the buffer, cost no traffic and bring zeros: no keys.
  template <int N, int B>
  __device__ __forceinline__ void merge(const unsigned (&at)[B], int part, int c, floatx4 (&acc)[B], float (&m)[B], float (&l)[B]) const {
    constexpr unsigned PARTS = 64 / (D / 4);
    uintx4 x[B][N];
    uintx2 y[B][N];
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const unsigned row = ((unsigned)i * PARTS + (unsigned)part) * n_rows + at[j];
        y[j][i] = __builtin_amdgcn_raw_buffer_load_b64(ml, row * 8u, 0, kDeviceScope);
        x[j][i] = __builtin_amdgcn_raw_buffer_load_b128(o, row * (D * 4u) + (unsigned)c * 16u, 0, kDeviceScope);
      }
#pragma unroll
    for (int j = 0; j < B; ++j) {
      m[j] = -INFINITY;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        // no visible key for the row in this piece, whose O may be NaN: 0 times a value that is not finite
        if (y[j][i][1] == 0u) {
          y[j][i][0] = __float_as_uint(-INFINITY);
          x[j][i] = uintx4{0u, 0u, 0u, 0u};
        }
        m[j] = fmaxf(m[j], __uint_as_float(y[j][i][0]));
      }
      m[j] = pair_max(m[j]);
      if (PARTS == 4) m[j] = row16_max(m[j]);
      const float ref = m[j] == -INFINITY ? 0.f : m[j];
      acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
      l[j] = 0.f;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float b = __builtin_amdgcn_exp2f(__uint_as_float(y[j][i][0]) - ref);
        l[j] = __builtin_fmaf(__uint_as_float(y[j][i][1]), b, l[j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = __builtin_fmaf(__uint_as_float(x[j][i][e]), b, acc[j][e]);
      }
      l[j] = pair_sum(l[j]);
      if (PARTS == 4) l[j] = row16_sum(l[j]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[j][e] = pair_sum(acc[j][e]);
        if (PARTS == 4) acc[j][e] = row16_sum(acc[j][e]);
      }
    }
  }
};

// Whether this workgroup is the last of its unit's n_splits; for all its threads, behind their stores.  The counter is back at zero then, and
// there is one for every number of pieces, so that it is between steps, whatever ran in between.
__device__ __forceinline__ bool last_to_meet(const AttnParams& p, int unit, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *flag = atomicInc(p.meet_count + unit * kMeetStride + p.n_splits, (unsigned)p.n_splits - 1u) == (unsigned)p.n_splits - 1u;
  __syncthreads();
  return *flag != 0;
}

}  // namespace kvfold
