// Shared device helpers for the gfx950 kernels: bf16 bit conversions, vector
// types, wave64 reductions, and the launch-error check used by the host side.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pallas.h"

namespace pallas {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// bf16 stored as its 16-bit pattern.
__device__ __forceinline__ float bf2f(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// Low / high bf16 of a packed pair.
__device__ __forceinline__ float bflo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bfhi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// float -> bf16 with the hardware conversion (v_cvt_pk_bf16_f32: round to
// nearest, ties to even; NaN stays NaN).
__device__ __forceinline__ uint32_t pack_bf2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

// SwiGLU of one output: silu(gate) * up, silu(g) = g / (1 + e^-g), the
// division taken as a multiply by the hardware reciprocal (v_rcp_f32,
// within 1 ulp): the IEEE division sequence costs a dozen instructions per
// output in the GEMM epilogues, and the result is rounded to bf16.
__device__ __forceinline__ float swiglu(float gate, float up) {
  return gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up;
}

// Butterfly reductions over lane distances 32, 16, 8, 4, 2, 1 (in that
// order), done with register lane exchanges instead of LDS permutes.  Each
// step adds (or takes the max of) the values of lanes i and i ^ m, in one
// operand order or the other, which is exact either way, so the results
// are those of the __shfl_xor butterfly bit for bit:
//   32, 16: v_permlane32_swap / v_permlane16_swap of a value with itself
//           return the pair (v[i], v[i ^ m]) in some order;
//   8:      DPP row_ror:8 reads lane (i + 8) mod 16 = i ^ 8 of the row;
//   4:      DPP row_ror:4 reads lane i ^ 4 or i ^ 4 ^ 8, equal after the
//           8-step;
//   2, 1:   DPP quad permutes [2, 3, 0, 1] and [1, 0, 3, 2].
// Every lane of the group being reduced (the quad, the 16-lane row, the
// wave) must be active: a DPP read from an inactive lane does not return
// that lane's value.
template <int CTRL>
__device__ __forceinline__ float dpp_read(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppXor1 = 0xB1;    // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;    // quad_perm [2, 3, 0, 1]
constexpr int kDppRor4 = 0x124;   // row_ror:4
constexpr int kDppRor8 = 0x128;   // row_ror:8

// Sum of a 16-lane row (distances 8, 4, 2, 1).
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_read<kDppRor8>(v);
  v += dpp_read<kDppRor4>(v);
  v += dpp_read<kDppXor2>(v);
  v += dpp_read<kDppXor1>(v);
  return v;
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_read<kDppRor8>(v));
  v = fmaxf(v, dpp_read<kDppRor4>(v));
  v = fmaxf(v, dpp_read<kDppXor2>(v));
  v = fmaxf(v, dpp_read<kDppXor1>(v));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  return row16_sum(v);
}
__device__ __forceinline__ float wave_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  return row16_max(v);
}

// QK-norm (when `norm`) and rotary embedding of four pairs of a D-wide head:
// a lane holds elements [4j, 4j + 4) in `lo` and [4j + D/2, 4j + D/2 + 4) in
// `hi`, their gains in g0 and g1, and (cos, sin) of pairs 4j .. 4j + 3 in cs01
// and cs23.  The D / 8 lanes of a head are neighbours and all active.
template <int D>
__device__ __forceinline__ void norm_rope4(u32x2& lo, u32x2& hi, bool norm, u32x2 g0, u32x2 g1, float eps, f32x4 cs01,
                                           f32x4 cs23) {
  float x0[4] = {bflo(lo.x), bfhi(lo.x), bflo(lo.y), bfhi(lo.y)};
  float x1[4] = {bflo(hi.x), bfhi(hi.x), bflo(hi.y), bfhi(hi.y)};
  if (norm) {
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += x0[e] * x0[e] + x1[e] * x1[e];
    if constexpr (D / 8 == 16) {
      ss = row16_sum(ss);
    } else {
#pragma unroll
      for (int o = D / 16; o > 0; o >>= 1) ss += __shfl_xor(ss, o, kWave);
    }
    const float inv = rsqrtf(ss / D + eps);
    const float ga[4] = {bflo(g0.x), bfhi(g0.x), bflo(g0.y), bfhi(g0.y)};
    const float gb[4] = {bflo(g1.x), bfhi(g1.x), bflo(g1.y), bfhi(g1.y)};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x0[e] = x0[e] * inv * ga[e];
      x1[e] = x1[e] * inv * gb[e];
    }
  }
  const float cs[4] = {cs01.x, cs01.z, cs23.x, cs23.z};
  const float sn[4] = {cs01.y, cs01.w, cs23.y, cs23.w};
  float y0[4], y1[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    y0[e] = x0[e] * cs[e] - x1[e] * sn[e];
    y1[e] = x1[e] * cs[e] + x0[e] * sn[e];
  }
  lo = u32x2{pack_bf2(y0[0], y0[1]), pack_bf2(y0[2], y0[3])};
  hi = u32x2{pack_bf2(y1[0], y1[1]), pack_bf2(y1[2], y1[3])};
}

}  // namespace pallas
