// Device-side helpers shared by the kernels of the eOptShrinkQ library (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "eoq.h"

namespace eoqdev {

typedef _Float16 half_t;

// ---- cross-lane moves (DPP) -------------------------------------------------------------------
// ctrl: 0xB1 = lane^1 and 0x4E = lane^2 inside groups of 4; 0x120+n = rotate by n inside rows of 16;
// 0x140 = mirror of a row of 16 (lane -> 15 - lane), 0x141 = mirror of each half row (lane -> 7 - lane).
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true);
  hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}

// sum over the 2 / 4 lanes of an aligned group; every lane of the group gets the total
template <typename T>
__device__ __forceinline__ T pair_sum(T v) { return v + dpp_mov<0xB1>(v); }
template <typename T>
__device__ __forceinline__ T quad_sum(T v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  return v;
}
// sum over a row of 16 lanes by a butterfly of commutative pair sums (lane^1, lane^2, 7-lane, 15-lane): bit-identical in all
// 16 lanes
__device__ __forceinline__ double row16_sum_uniform(double v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  return v;
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// ---- number formats ---------------------------------------------------------------------------
// double -> binary16 with a single rounding (round-to-odd into binary32 first)
__device__ __forceinline__ uint16_t double_to_half_bits(double x) {
  float f = __double2float_rz(x);
  if ((double)f != x) f = __int_as_float(__float_as_int(f) | 1);
  half_t h = (half_t)f;
  return *reinterpret_cast<uint16_t*>(&h);
}
// float -> binary16, round to nearest even, saturating at the largest finite value (one median-of-three, then the
// conversion)
__device__ __forceinline__ uint16_t float_to_half_bits(float f) {
  f = __builtin_amdgcn_fmed3f(f, -65504.0f, 65504.0f);
  half_t h = (half_t)f;
  return *reinterpret_cast<uint16_t*>(&h);
}
// Kernels that set the mode bit FP16_OVFL (binary16 results that overflow become the largest finite value instead of
// infinity) get the same saturation from the conversion alone.
__device__ __forceinline__ void set_fp16_overflow_clamp() { __builtin_amdgcn_s_setreg(1 | (23 << 6) | (0 << 11), 1); }
__device__ __forceinline__ uint16_t float_to_half_bits_clamped_by_mode(float f) {
  half_t h = (half_t)f;
  return *reinterpret_cast<uint16_t*>(&h);
}
// two floats -> two binary16 in one word (low half first), round to nearest even: one v_cvt_pk_f16_f32
__device__ __forceinline__ uint32_t pack_half2(float a, float b) {
  typedef _Float16 half2v __attribute__((ext_vector_type(2)));
  typedef float float2v __attribute__((ext_vector_type(2)));
  const float2v v = {a, b};
  const half2v h = __builtin_convertvector(v, half2v);
  return *reinterpret_cast<const uint32_t*>(&h);
}
__device__ __forceinline__ float half_bits_to_float(uint16_t b) {
  half_t h = *reinterpret_cast<half_t*>(&b);
  return (float)h;
}

// Load 8 consecutive elements of a block (binary16 or float32) as floats.
__device__ __forceinline__ void load8(const void* base, int dtype, size_t elem, float (&v)[8]) {
  if (dtype == EOQ_F16) {
    const uint4 raw = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(base) + elem);
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = half_bits_to_float((uint16_t)(w[i] & 0xFFFFu));
      v[2 * i + 1] = half_bits_to_float((uint16_t)(w[i] >> 16));
    }
  } else {
    const float4 a = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + elem);
    const float4 b = *reinterpret_cast<const float4*>(static_cast<const float*>(base) + elem + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}

// The four bytes of each of x0 .. x3, transposed: out[k] = bytes k of x0, x1, x2, x3 (x0 lowest).  Eight byte
// permutes: pairs first (bytes 0/1 and 2/3 of two words interleaved), then the halves of the pairs.
__device__ __forceinline__ void transpose_bytes(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, uint32_t (&out)[4]) {
  const uint32_t a01 = __builtin_amdgcn_perm(x1, x0, 0x05010400u), b01 = __builtin_amdgcn_perm(x1, x0, 0x07030602u);
  const uint32_t a23 = __builtin_amdgcn_perm(x3, x2, 0x05010400u), b23 = __builtin_amdgcn_perm(x3, x2, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
}

// Compile-time loop: every index into a per-lane register array must be a constant before the optimiser
// first looks at the array, otherwise the array is kept in (scratch) memory.
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}
#define EOQ_SFOR(var, n, ...) eoqdev::static_for<0, n>([&](auto var##_ic) __attribute__((always_inline)) { \
  constexpr int var = decltype(var##_ic)::value; __VA_ARGS__ })

// Bit-planes of the cells of a product Pi u^T (32 coordinates by 32 tokens).  A lane of half hf holds rows 8 (v / 4) + 4 hf + v % 4
// of column l32: with Pi's rows in the order of plane_row, coordinate 16 hf + v of its token in register v.
__device__ __forceinline__ int plane_row(int l32) { return 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3); }

// Index of a cell = number of boundaries <= z, found from the top bit down by signs, which are appended from below to words of the
// lane: one instruction for the sign of z, three for every further bit (the boundary with the sign of z, the difference, its sign),
// no mask in scalar registers.  The table is symmetric and its middle boundary 0 (lloyd_max), so the positive half of it is
// enough.  A set bit stands for "below the boundary"; z is a sum that starts from +0 and never -0.  Which half of the remaining
// cells comes next follows from the sign of the difference, not from |z|, or a negative z on a boundary would take the other one.
// The boundaries are separate values, not an array or a vector: the compiler turns a select between two elements into an element
// at a selected index (scratch memory for an array, a chain of sixteen selects for a register vector).
template <int BITS>
struct HalfBounds {
  float c0, c1, c2, c3, c4, c5, c6;   // boundaries 2^(BITS-1) ..
  __device__ __forceinline__ void load(const float* __restrict__ bnd) {
    constexpr int N = (1 << (BITS - 1)) - 1;
    const float* b = bnd + N + 1;
    c0 = 0 < N ? b[0] : 0.0f; c1 = 1 < N ? b[1] : 0.0f; c2 = 2 < N ? b[2] : 0.0f;
    c3 = 3 < N ? b[3] : 0.0f; c4 = 4 < N ? b[4] : 0.0f; c5 = 5 < N ? b[5] : 0.0f; c6 = 6 < N ? b[6] : 0.0f;
  }
  __device__ __forceinline__ void append(float z, uint32_t (&below)[BITS]) const {
    auto push = [](uint32_t& to, float x) __attribute__((always_inline)) { to = __builtin_amdgcn_alignbit(to, __float_as_uint(x), 31); };
    auto outer = [&](float e) __attribute__((always_inline)) { return (int)(__float_as_uint(e) ^ __float_as_uint(z)) >= 0; };
    push(below[BITS - 1], z);
    if constexpr (BITS == 2) {
      push(below[0], z - copysignf(c0, z));
    } else if constexpr (BITS == 3) {
      const float e1 = z - copysignf(c1, z);
      push(below[1], e1);
      push(below[0], z - copysignf(outer(e1) ? c2 : c0, z));
    } else if constexpr (BITS == 4) {
      const float e2 = z - copysignf(c3, z);
      push(below[2], e2);
      const bool o2 = outer(e2);
      const float mid = o2 ? c5 : c1, lo = o2 ? c4 : c0, hi = o2 ? c6 : c2;
      const float e1 = z - copysignf(mid, z);
      push(below[1], e1);
      push(below[0], z - copysignf(outer(e1) ? hi : lo, z));
    }
  }
  // bit v of below[p]: plane p of the lane's coordinate v
  template <typename Acc>
  __device__ __forceinline__ void planes(const Acc& z, uint32_t (&below)[BITS]) const {
    EOQ_SFOR(p, BITS, below[p] = 0u;);
    EOQ_SFOR(v, 16, append(z[15 - v], below););
    const bool nan = z[0] != z[0];   // a token with a NaN: all its coordinates are, and lie in cell 0
    EOQ_SFOR(p, BITS, below[p] = nan ? 0xFFFFu : below[p];);
  }
};
// Half words a and b of the lanes: the lower half of the wave gets the plane's word of a, the upper half that of b.
__device__ __forceinline__ uint32_t plane_words(uint32_t a, uint32_t b) {
  const auto w = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  return ~(w[0] | (w[1] << 16));
}

}  // namespace eoqdev
