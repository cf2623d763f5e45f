// SVD factors of the retained components at 4 bits per entry with per-block data-adaptive codebooks (Alg. 3
// line 3; Sec. 3.1: "SVD factors are quantized at 4 bits via data-adaptive Lloyd-Max codebooks", the shrunk singular
// values stay in binary16).
//
// Per block and factor matrix (U: n x r, V: d x r, both with orthonormal columns) the codebook is {+-m_0 .. +-m_7}:
// eight magnitudes fitted to |entries| by Lloyd's iteration from the Lloyd-Max levels of a Gaussian with the
// entries' root mean square, eight rounds, then rounded to binary16.  A code is 3 bits of magnitude index (nearest
// level, ties up) plus the sign bit (bit 3 set for x >= 0): symmetric, so the arbitrary sign of a singular vector
// only flips sign bits.  Besides the codes the kernel writes what they expand to, lfac = binary16(U_hat phi16) and
// rfac = V_hat, which is what the residual (closed loop), the decoder and the scores use.
#include "eoq_device.h"
#include "eoq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

using namespace eoqdev;

constexpr int D = EOQ_D;
constexpr int THREADS = 256;   // of the expansion
constexpr int LEVELS = 8;
constexpr int LLOYD_ITERS = 8;
constexpr int KEEP = 16;   // entries of a matrix that a lane keeps in registers

struct GaussLevels {
  double c[LEVELS];  // Lloyd-Max magnitudes of N(0,1) at 16 levels
};

__device__ __forceinline__ int code_of(float x, const float (&b)[LEVELS - 1]) {
  int k = 0;
#pragma unroll
  for (int q = 0; q < LEVELS - 1; ++q) k += (fabsf(x) >= b[q]) ? 1 : 0;  // a tie goes to the upper cell
  return k | ((x >= 0.0f) ? 8 : 0);
}

__device__ __forceinline__ double swizzle_xor(double v, int mask) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  if (mask == 4) {
    lo = __builtin_amdgcn_ds_swizzle(lo, 0x101F);
    hi = __builtin_amdgcn_ds_swizzle(hi, 0x101F);
  } else if (mask == 8) {
    lo = __builtin_amdgcn_ds_swizzle(lo, 0x201F);
    hi = __builtin_amdgcn_ds_swizzle(hi, 0x201F);
  } else if (mask == 16) {
    lo = __builtin_amdgcn_ds_swizzle(lo, 0x401F);
    hi = __builtin_amdgcn_ds_swizzle(hi, 0x401F);
  } else {
    lo = __shfl_xor(lo, 32, 64);
    hi = __shfl_xor(hi, 32, 64);
  }
  return __hiloint2double(hi, lo);
}

// Eight per-lane values summed over the wave, the eight totals spread over the lanes: lane l returns the total of
// value number 4 (l & 1) + 2 ((l >> 1) & 1) + ((l >> 2) & 1).  Halving exchange: every step hands the partner lane
// the half of the values it keeps, so 4 + 2 + 1 + 3 exchanges instead of 8 x 6.
__device__ __forceinline__ double wave_reduce8(const double (&v)[8], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  double w[4], x[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = b0 ? v[i + 4] : v[i], send = b0 ? v[i] : v[i + 4];
    w[i] = keep + dpp_mov<0xB1>(send);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = b1 ? w[i + 2] : w[i], send = b1 ? w[i] : w[i + 2];
    x[i] = keep + dpp_mov<0x4E>(send);
  }
  double y = (b2 ? x[1] : x[0]) + swizzle_xor(b2 ? x[0] : x[1], 4);
  y += swizzle_xor(y, 8);
  y += swizzle_xor(y, 16);
  y += swizzle_xor(y, 32);
  return y;
}
// number of the value wave_reduce8 leaves in lane l (l < 8)
__device__ __forceinline__ int reduce8_slot(int l) { return 4 * (l & 1) + 2 * ((l >> 1) & 1) + ((l >> 2) & 1); }

// The boundaries between the levels that the lanes k = lane % 8 hold, as float32 numbers rounded up: a float32 number is at or
// above one of them exactly where it is at or above the midpoint itself.
__device__ __forceinline__ void boundaries(double level, float (&b)[LEVELS - 1]) {
  const double mid = 0.5 * (level + dpp_mov<0x101>(level));   // (row_shl:1: the next lane's)
  float f = (float)mid;
  if ((double)f < mid) f = __uint_as_float(__float_as_uint(f) + 1u);   // (magnitudes: positive)
#pragma unroll
  for (int k = 0; k < LEVELS - 1; ++k) b[k] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), k));
}

// One wave has V (r D entries), UW waves have U (r n entries).  A wave walks its entries, the first sixteen to a lane kept in
// registers, and adds up for itself; its eight levels are all else that it keeps.  With four waves on both matrices each of
// them went through both sums and both moves of the levels, and those, not the entries, were most of its instructions at
// 128 tokens.  Ranks 1 .. 6: 4096 blocks of 128 x 128 took 246 us and take 118, 16 of them 41 and 33; 16384 blocks of 512 x 128
// 1480 and 1065, 4096 of 1024 x 128 770 and 673.  The reads of the rows of S, one to a lane, keep it from more waves: five to a
// SIMD instead of four read them from further away and take 158 where it is 118; on the fp64 matrix cores, sixteen rows
// at a time, the product takes longer (128, 1240 and 710).
template <int RCAP, int UW>
__global__ __launch_bounds__(64 * (UW + 1), 4) void eoq_factor_quant_kernel(
    const uint16_t* __restrict__ blocks, EoqBlockMap map, int64_t B, int n, int r_max, GaussLevels g,
    const int32_t* __restrict__ rank_in,
    const float* __restrict__ phi, const float* __restrict__ sigma, const float* __restrict__ wfac,
    uint16_t* __restrict__ rfac, uint16_t* __restrict__ lfac, uint8_t* __restrict__ lcodes,
    uint8_t* __restrict__ rcodes, uint16_t* __restrict__ fbook, uint16_t* __restrict__ phi16) {
  constexpr int THREADS = 64 * (UW + 1);
  extern __shared__ __align__(16) float dyn[];  // Vs[r][D] then Us[r][n]
  __shared__ __align__(16) double red[2][UW + 1][8];   // [parity][wave]: sums at or above the boundaries, and of all
  __shared__ int redc[2][UW + 1][8];                   // counts
  __shared__ float book[UW + 1][LEVELS];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool is_v = wave == UW;
  // The workgroups walk the batch with the grid's stride.  The launch with the small table has one workgroup per block
  // and takes the blocks of rank 1 .. 8 (and clears the codebook of rank-0 blocks); the launch with the large table is
  // a few persistent workgroups that look for the rest (usually there are none: a grid of B would only spend its
  // time placing workgroups with a large LDS allocation that return at once).
  for (size_t wblk = blockIdx.x; wblk < (size_t)B; wblk += gridDim.x) {   // number in the batch: workspace and input
  __syncthreads();                           // LDS of the previous block has been consumed
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));              // (else every address that follows from it is kept over the blocks)
  const int lane = tid & 63;
  const size_t blk = map.slot(wblk);         // record slot: everything that is stored
  const int r = rank_in[blk];
  if (RCAP == 8) {
    if (r == 0 && tid < 2 * LEVELS) fbook[blk * 2 * LEVELS + tid] = 0;
    if (r == 0 || r > 8) continue;
  } else {
    if (r <= 8) continue;
  }
  float* Vs = dyn;
  float* Us = dyn + (size_t)r * D;
  // right vectors back from the projection operand W = V phi / sigma (float32); where phi = 0 (guarded
  // component) from the stored binary16 vector
  for (int e = tid; e < r * D; e += THREADS) {
    const int i = e >> 7;
    const float ph = phi[blk * r_max + i], sg = sigma[blk * r_max + i];
    Vs[e] = (ph > 0.0f) ? wfac[wblk * (size_t)r_max * D + e] * (sg / ph) : half_bits_to_float(rfac[blk * (size_t)r_max * D + e]);
  }
  __syncthreads();
  // left vectors U = S V / sigma, one token per lane and pass, four components at a time
  for (int t = tid; t < n; t += THREADS) {
    const uint16_t* row = blocks + map.in_base(wblk) + (size_t)t * (size_t)map.token_stride;
    for (int i0 = 0; i0 < r; i0 += 4) {
      const float* vrow[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) vrow[c] = Vs + min(i0 + c, r - 1) * D;
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
      for (int q = 0; q < 16; ++q) {
        const uint4 raw = *reinterpret_cast<const uint4*>(row + 8 * q);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
        double sv[8];
#pragma unroll
        for (int h = 0; h < 8; ++h) sv[h] = (double)half_bits_to_float((uint16_t)(w[h >> 1] >> (16 * (h & 1))));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float4 va = *reinterpret_cast<const float4*>(vrow[c] + 8 * q);
          const float4 vb = *reinterpret_cast<const float4*>(vrow[c] + 8 * q + 4);
          acc[c] = fma(sv[0], (double)va.x, acc[c]);
          acc[c] = fma(sv[1], (double)va.y, acc[c]);
          acc[c] = fma(sv[2], (double)va.z, acc[c]);
          acc[c] = fma(sv[3], (double)va.w, acc[c]);
          acc[c] = fma(sv[4], (double)vb.x, acc[c]);
          acc[c] = fma(sv[5], (double)vb.y, acc[c]);
          acc[c] = fma(sv[6], (double)vb.z, acc[c]);
          acc[c] = fma(sv[7], (double)vb.w, acc[c]);
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (i0 + c < r) {
          const float sg = sigma[blk * r_max + i0 + c];
          Us[(size_t)(i0 + c) * n + t] = (sg > 0.0f) ? (float)(acc[c] / (double)sg) : 0.0f;
        }
    }
  }
  __syncthreads();

  // ---- Lloyd fits of the two codebooks, side by side (one barrier per round, none where each is one wave's) ----
  const float* X = is_v ? Vs : Us;
  const int count = r * (is_v ? D : n), first = is_v ? lane : 64 * wave + lane, step = is_v ? 64 : 64 * UW;
  const int k = lane & 7;   // every eight lanes hold the levels and move them alike
  int par = 0;
  auto meet = [&]() __attribute__((always_inline)) {
    if constexpr (UW > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();   // one wave: its LDS operations complete in order
  };
  auto total = [&](int v) __attribute__((always_inline)) {   // value number v over the waves of the matrix
    double t = red[par][is_v ? UW : 0][v];
#pragma unroll
    for (int w = 1; w < UW; ++w) t += is_v ? 0.0 : red[par][w][v];
    return t;
  };
  auto number = [&](int v) __attribute__((always_inline)) {
    int t = redc[par][is_v ? UW : 0][v];
#pragma unroll
    for (int w = 1; w < UW; ++w) t += is_v ? 0 : redc[par][w][v];
    return t;
  };
  // The first entries of the lane stay in registers (all of them where a wave has the 128 tokens of eight components).
  const int trips = (count + step - 1) / step;
  float x[KEEP];
  auto entry = [&](int j) __attribute__((always_inline)) {   // magnitude; -1 behind the last
    const int e = j * step + first;
    return (e < count) ? fabsf(X[e]) : -1.0f;
  };
#pragma unroll
  for (int j = 0; j < KEEP; ++j) x[j] = (j < trips) ? entry(j) : -1.0f;
  double level, all;
  {
    double st[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    auto add = [&](float f) __attribute__((always_inline)) {
      const double a = (double)fmaxf(f, 0.0f);
      st[0] = fma(a, a, st[0]);
      st[4] += a;                                      // (values 0 and 4 end in the lanes 0 and 1)
    };
#pragma unroll
    for (int j = 0; j < KEEP; ++j)
      if (j < trips) add(x[j]);
    for (int j = KEEP; j < trips; ++j) add(entry(j));
    const double y = wave_reduce8(st, lane);
    if (lane < 2) red[par][wave][lane] = y;
    meet();
    const double rms = sqrt(total(0) / (double)count);
    all = total(1);
    level = 0.0;
#pragma unroll
    for (int q = 0; q < LEVELS; ++q) level = (k == q) ? g.c[q] * rms : level;
    par ^= 1;
  }
  float b[LEVELS - 1];
#pragma unroll 1
  for (int it = 0; it < LLOYD_ITERS; ++it) {
    // sums of the entries at or above every boundary per lane, the counts per wave
    double st[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int cnt[LEVELS - 1] = {0, 0, 0, 0, 0, 0, 0};
    boundaries(level, b);
    auto add = [&](float f) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < LEVELS - 1; ++q) {
        const bool ge = f >= b[q];
        float a = ge ? f : 0.0f;
        asm("" : "+v"(a));   // (else all conversions are kept over the rounds)
        st[q] += (double)a;
        cnt[q] += __popcll(__ballot(ge));
      }
    };
#pragma unroll
    for (int j = 0; j < KEEP; ++j)
      if (j < trips) add(x[j]);
    for (int j = KEEP; j < trips; ++j) add(entry(j));
    const double y = wave_reduce8(st, lane);
    if (lane < 8) red[par][wave][reduce8_slot(lane)] = y;
    int mine = 0;
#pragma unroll
    for (int q = 0; q < LEVELS - 1; ++q) mine = (lane == q) ? cnt[q] : mine;
    if (lane < LEVELS - 1) redc[par][wave][lane] = mine;
    meet();
    // Every lane moves level k (the waves of a matrix repeat the work and agree bit for bit, so no second barrier).  Cell
    // sum = difference of two "at or above" sums, T[0] = all, T[j] = value j - 1, T[8] = 0; counts likewise.
    const int ib = min(k, LEVELS - 2);
    const double sa = (k == 0) ? all : total(max(k - 1, 0)), sb = (k == LEVELS - 1) ? 0.0 : total(ib);
    const int ca = (k == 0) ? count : number(max(k - 1, 0)), cb = (k == LEVELS - 1) ? 0 : number(ib);
    const int ck = ca - cb;
    level = (ck > 0) ? (sa - sb) / (double)ck : level;   // an empty cell keeps its level
    par ^= 1;
  }

  // ---- levels in binary16, codes and what they expand to ----
  const uint16_t bits16 = double_to_half_bits(level);
  const float m16 = half_bits_to_float(bits16);
  if ((wave == 0 || is_v) && lane < LEVELS) fbook[blk * 2 * LEVELS + (is_v ? LEVELS : 0) + lane] = bits16;
  if (lane < LEVELS) book[wave][lane] = m16;
  boundaries((double)m16, b);
  __builtin_amdgcn_wave_barrier();
  if (!is_v) {
    for (int i = 0; i < r; ++i) {
      const uint16_t ph16 = float_to_half_bits(phi[blk * r_max + i]);
      const double p16 = (double)half_bits_to_float(ph16);
      if (tid == 0) phi16[blk * r_max + i] = ph16;
      for (int t = first; t < n / 2; t += step) {   // two tokens per byte
        const float2 x = *reinterpret_cast<const float2*>(Us + (size_t)i * n + 2 * t);
        const int c0 = code_of(x.x, b), c1 = code_of(x.y, b);
        const double l0 = (double)book[wave][c0 & 7], l1 = (double)book[wave][c1 & 7];
        const uint32_t o0 = double_to_half_bits(((c0 & 8) ? l0 : -l0) * p16), o1 = double_to_half_bits(((c1 & 8) ? l1 : -l1) * p16);
        *reinterpret_cast<uint32_t*>(lfac + (blk * r_max + i) * (size_t)n + 2 * t) = o0 | (o1 << 16);
        lcodes[(blk * r_max + i) * (size_t)(n / 2) + t] = (uint8_t)(c0 | (c1 << 4));
      }
    }
  } else {
    for (int i = 0; i < r; ++i) {
      const float2 x = *reinterpret_cast<const float2*>(Vs + i * D + 2 * lane);
      const int c0 = code_of(x.x, b), c1 = code_of(x.y, b);
      const uint32_t o0 = float_to_half_bits((c0 & 8) ? book[wave][c0 & 7] : -book[wave][c0 & 7]);
      const uint32_t o1 = float_to_half_bits((c1 & 8) ? book[wave][c1 & 7] : -book[wave][c1 & 7]);
      *reinterpret_cast<uint32_t*>(rfac + (blk * r_max + i) * (size_t)D + 2 * lane) = o0 | (o1 << 16);
      rcodes[(blk * r_max + i) * (size_t)(D / 2) + lane] = (uint8_t)(c0 | (c1 << 4));
    }
  }
  }  // blocks of this workgroup
}

// codes + codebooks + phi16 -> lfac = binary16(U_hat phi16), rfac = V_hat (rows below the rank)
__global__ __launch_bounds__(THREADS) void eoq_factor_expand_kernel(
    int n, int r_max, const int32_t* __restrict__ rank_in, const uint8_t* __restrict__ lcodes,
    const uint8_t* __restrict__ rcodes, const uint16_t* __restrict__ fbook, const uint16_t* __restrict__ phi16,
    uint16_t* __restrict__ lfac, uint16_t* __restrict__ rfac) {
  const int tid = threadIdx.x;
  const size_t blk = blockIdx.x;
  const int r = min(max(rank_in[blk], 0), r_max);   // a record read back from storage: never index past r_max rows
  __shared__ uint16_t book[2 * LEVELS];
  if (tid < 2 * LEVELS) book[tid] = fbook[blk * 2 * LEVELS + tid];
  __syncthreads();
  for (int e = tid; e < r * (n / 2); e += THREADS) {
    const int i = e / (n / 2), t = 2 * (e - i * (n / 2));
    const double p16 = (double)half_bits_to_float(phi16[blk * r_max + i]);
    const int byte = lcodes[(blk * r_max + i) * (size_t)(n / 2) + (t >> 1)];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int code = (byte >> (4 * u)) & 15;
      const double lev = (double)half_bits_to_float(book[code & 7]);
      lfac[(blk * r_max + i) * (size_t)n + t + u] = double_to_half_bits(((code & 8) ? lev : -lev) * p16);
    }
  }
  for (int e = tid; e < r * (D / 2); e += THREADS) {
    const int i = e / (D / 2), j = 2 * (e - i * (D / 2));
    const int byte = rcodes[(blk * r_max + i) * (size_t)(D / 2) + (j >> 1)];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int code = (byte >> (4 * u)) & 15;
      const uint16_t lev = book[LEVELS + (code & 7)];
      rfac[(blk * r_max + i) * (size_t)D + j + u] = (code & 8) ? lev : (uint16_t)(lev | 0x8000u);
    }
  }
}

}  // namespace

// Calls f(waves of U).  With the one of V they are two, four or eight, alike for the four SIMDs of a unit: at n / 128 waves of U,
// that is five a workgroup at 512 tokens and nine at 1024, one SIMD had two or three of them and the others waited for it (16384
// blocks of 512 x 128 1700 us instead of 1065, 4096 of 1024 x 128 914 instead of 673).
template <typename F>
static hipError_t for_u_waves(int n, F&& f) {
  if (n < 256) return f(std::integral_constant<int, 1>{});
  if (n < 768) return f(std::integral_constant<int, 3>{});
  return f(std::integral_constant<int, 7>{});
}

// Largest LDS tables the two variants are ever launched with (n * r_max <= 32768, n <= 4096): raised once per device
// at context creation, so that the hot call sets no function attribute.
hipError_t eoq_factor_quant_prepare() {
  for (int n = 128; n <= 1024; n *= 2) {
    const hipError_t e = for_u_waves(n, [](auto uw) {
      constexpr int UW = decltype(uw)::value;
      const hipError_t e8 = hipFuncSetAttribute(reinterpret_cast<const void*>(eoq_factor_quant_kernel<8, UW>),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, 8 * (4096 + D) * (int)sizeof(float));
      if (e8 != hipSuccess) return e8;
      return hipFuncSetAttribute(reinterpret_cast<const void*>(eoq_factor_quant_kernel<32, UW>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (32768 + EOQ_RMAX_CAP * D) * (int)sizeof(float));
    });
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t eoq_launch_factor_quant(const EoqLaunch& L, const void* blocks_fp16, int64_t B, const float* wfac,
                                   eoq_packed out, eoq_factor_codes fq, const double* gauss_levels) {
  GaussLevels g;
  for (int k = 0; k < LEVELS; ++k) g.c[k] = gauss_levels[k];
  // two launches over all blocks, each taking the blocks of its rank class: the table of the factors in LDS is
  // sized for 8 components (most blocks: many workgroups per CU) or for r_max
  return for_u_waves(L.n, [&](auto uw) {
    constexpr int UW = decltype(uw)::value;
    const size_t lds8 = (size_t)std::min(8, L.r_max) * (L.n + D) * sizeof(float);
    hipLaunchKernelGGL((eoq_factor_quant_kernel<8, UW>), dim3((unsigned)B), dim3(64 * (UW + 1)), lds8, L.stream,
                       static_cast<const uint16_t*>(blocks_fp16), L.map, B, L.n, L.r_max, g, out.rank, out.phi, out.sigma, wfac,
                       out.rfac, out.lfac, fq.lcodes, fq.rcodes, fq.fbook, fq.phi16);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || L.r_max <= 8) return e;
    const size_t lds = (size_t)L.r_max * (L.n + D) * sizeof(float);
    hipLaunchKernelGGL((eoq_factor_quant_kernel<32, UW>), dim3((unsigned)(B < 512 ? B : 512)), dim3(64 * (UW + 1)), lds, L.stream,
                       static_cast<const uint16_t*>(blocks_fp16), L.map, B, L.n, L.r_max, g, out.rank, out.phi, out.sigma, wfac,
                       out.rfac, out.lfac, fq.lcodes, fq.rcodes, fq.fbook, fq.phi16);
    return hipGetLastError();
  });
}

hipError_t eoq_launch_factor_expand(const EoqLaunch& L, eoq_packed rec, eoq_factor_codes fq, int64_t B) {
  hipLaunchKernelGGL(eoq_factor_expand_kernel, dim3((unsigned)B), dim3(THREADS), 0, L.stream, L.n, L.r_max, rec.rank,
                     fq.lcodes, fq.rcodes, fq.fbook, fq.phi16, rec.lfac, rec.rfac);
  return hipGetLastError();
}
