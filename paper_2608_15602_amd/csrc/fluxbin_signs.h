// Packed sign entries to matrix-core operand order, shared by the matrix-core kernels that read them without LDS: a
// wavefront loads the entries of 64 rows (one per lane, 128 sign bits of a chunk), four 16-row tiles.
#pragma once

#include <hip/hip_runtime.h>

namespace fluxbin {

typedef uint32_t sign_u32x4 __attribute__((ext_vector_type(4)));
typedef float sign_f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void sign_swap32(uint32_t& u, uint32_t& v) {
  const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
  u = r[0];
  v = r[1];
}

__device__ __forceinline__ void sign_swap16(uint32_t& u, uint32_t& v) {
  const auto r = __builtin_amdgcn_permlane16_swap(u, v, false, false);
  u = r[0];
  v = r[1];
}

// The rotation that puts a row's packed entry into canonical column order (right by -mu row mod 128 bits), as a word
// shift and two select masks.
struct SignRot {
  uint32_t shift, m1, m2;
};

template <int MU>
__device__ __forceinline__ SignRot sign_rot(uint32_t row) {
  const uint32_t rot = uint32_t(-(MU * int(row))) & 127u;
  return SignRot{rot & 31u, (rot & 32u) ? ~0u : 0u, (rot & 64u) ? ~0u : 0u};
}

__device__ __forceinline__ void sign_unrotate(const sign_u32x4& e, const SignRot& r, uint32_t (&w)[4]) {
  uint32_t f[4], h[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) f[m] = __builtin_amdgcn_alignbit(e[(m + 1) & 3], e[m], r.shift);
#pragma unroll
  for (int m = 0; m < 4; ++m) h[m] = (f[(m + 1) & 3] & r.m1) | (f[m] & ~r.m1);
#pragma unroll
  for (int m = 0; m < 4; ++m) w[m] = (h[(m + 2) & 3] & r.m2) | (h[m] & ~r.m2);
}

// 4 x 4 transpose between the words and the 16-lane groups: w[q] of lane (n, g) becomes word g of row 16 q + n.
__device__ __forceinline__ void sign_transpose(uint32_t (&w)[4]) {
  sign_swap32(w[0], w[2]);
  sign_swap32(w[1], w[3]);
  sign_swap16(w[0], w[1]);
  sign_swap16(w[2], w[3]);
}

// v of lane 16 q + n in every lane (n, g) of out[q].
__device__ __forceinline__ void sign_broadcast(uint32_t v, uint32_t (&out)[4]) {
  out[0] = out[2] = v;
  sign_swap32(out[0], out[2]);
  out[1] = out[0];
  out[3] = out[2];
  sign_swap16(out[0], out[1]);
  sign_swap16(out[2], out[3]);
}

// Two words shifted left by a constant s < 16 as one v_lshlrev_b64, which takes the time of one 32-bit shift (the
// compiler would split it). The bits the low word pushes into the high one land below bit s.
__device__ __forceinline__ uint64_t sign_shl64(uint64_t v, int s) {
  uint64_t r;
  asm("v_lshlrev_b64 %0, %1, %2" : "=v"(r) : "i"(s), "v"(v));
  return r;
}

}  // namespace fluxbin
