// The chunk's rows on their way into the cache with work on the way: the arithmetic, shared by the append kernel and by the
// few-rows attention kernel, which appends its rows itself.
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
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvfold {

template <typename T, int E>
using row_vec = __attribute__((ext_vector_type(E))) T;

// v: the lane's 16 bytes of the row; other: those half a row away; cs, sn: the pair's E angles; lower: first half of the row
template <typename T, int E>
__device__ __forceinline__ void rotate_vec(row_vec<T, E>& v, const row_vec<T, E>& other, const float* cs, const float* sn, bool lower) {
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float mine = (float)v[e], theirs = (float)other[e];
    const float t = theirs * sn[e];
    v[e] = (T)__builtin_fmaf(mine, cs[e], lower ? -t : t);
  }
}

// qmax: 2^(N-1) - 1; vpr: lanes of a row, neighbours and a power of two
template <typename T, int E>
__device__ __forceinline__ void round_trip_vec(row_vec<T, E>& v, int vpr, float qmax) {
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

// Rows [r0, r1) of the chunk of one KV head (bf16, D wide), rotated (K) and passed through the round trip as asked for, to
// the head's cache rows len_prev + r; 256 threads.  The pieces of the key range are disjoint and each has one workgroup, which
// reads no row of the chunk but those that it has written itself: none waits for another.
template <int D>
__device__ __forceinline__ void append_work_rows(const unsigned char* knew, const unsigned char* vnew, unsigned new_stride, unsigned char* kdst,
                                                 unsigned char* vdst, const float* rope_cos, const float* rope_sin, float qmax, int r0, int r1, int tid) {
  constexpr int CH = D / 8, TURNS = 2;  // turns whose loads are in flight together
  typedef row_vec<__bf16, 8> vec;
  const int n = (r1 - r0) * CH, c = tid % CH, a = c % (CH / 2);  // (256 is a multiple of CH: a thread keeps its column)
  const bool lower = c < CH / 2;
#pragma unroll 1
  for (int i0 = tid; i0 < 2 * n; i0 += TURNS * 256) {
    vec x[TURNS], other[TURNS];
    typedef __attribute__((ext_vector_type(4))) float floatx4;
    floatx4 cs[TURNS][2], sn[TURNS][2];
#pragma unroll
    for (int u = 0; u < TURNS; ++u) {
      const int i = i0 + u * 256;
      if (i >= 2 * n) continue;
      const bool is_v = i >= n;
      const int r = r0 + (is_v ? i - n : i) / CH;
      const unsigned char* row = (is_v ? vnew : knew) + (unsigned)r * new_stride;
      x[u] = *reinterpret_cast<const vec*>(row + c * 16);
      if (rope_cos && !is_v) {
        other[u] = *reinterpret_cast<const vec*>(row + (c ^ (CH / 2)) * 16);
        const floatx4* pc = reinterpret_cast<const floatx4*>(rope_cos + r * (D / 2) + a * 8);
        const floatx4* ps = reinterpret_cast<const floatx4*>(rope_sin + r * (D / 2) + a * 8);
        cs[u][0] = pc[0], cs[u][1] = pc[1];
        sn[u][0] = ps[0], sn[u][1] = ps[1];
      }
    }
#pragma unroll
    for (int u = 0; u < TURNS; ++u) {
      const int i = i0 + u * 256;
      if (i >= 2 * n) continue;
      const bool is_v = i >= n;
      const int r = r0 + (is_v ? i - n : i) / CH;
      if (rope_cos && !is_v) {
        float fc[8], fs[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) fc[e] = cs[u][e / 4][e % 4], fs[e] = sn[u][e / 4][e % 4];
        rotate_vec<__bf16, 8>(x[u], other[u], fc, fs, lower);
      }
      if (qmax > 0.f) round_trip_vec<__bf16, 8>(x[u], CH, qmax);
      *reinterpret_cast<vec*>((is_v ? vdst : kdst) + (unsigned)r * (unsigned)(D * 2) + c * 16) = x[u];
    }
  }
}

}  // namespace kvfold
