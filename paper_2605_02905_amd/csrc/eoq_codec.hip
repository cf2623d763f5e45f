// HIP kernels (gfx950) of the residual coder of eOptShrinkQ and its inverse:
//   encode : projection C = S V diag(phi/sigma) = U diag(phi), residual against the stored binary16 factors
//            (Alg. 3), then per row norm, rotation, Lloyd-Max index and bit-plane packing (Alg. 1 lines 3-5).
#include "eoq_device.h"
#include "eoq_internal.h"

namespace {

using namespace eoqdev;

constexpr int D = EOQ_D;

// ---------------------------------------------------------------------------
// encode kernel for float32 blocks: 64 rows of one block per workgroup, float32 arithmetic throughout.
//   rows in LDS -> C = S W^T rounded to the stored binary16 -> R = S - C V^T, its norm and u in registers -> u in LDS
//   -> z^T = Pi u^T with v_mfma_f32_32x32x2_f32, wave w the coordinates 32 w .. 32 w + 31 with its rows of Pi in 64
//   registers -> cells by signs, appended to half words of the bit-planes (HalfBounds).
// Operands of v_mfma_f32_32x32x2_f32 (wave64): lane l supplies A[row = l%32][k = l/32] and B[k = l/32][col = l%32] and
// receives D[row = 8*(v/4) + 4*(l/32) + v%4][col = l%32] in register v.  The contraction index is permuted so that a lane's
// entries of four consecutive instructions are four consecutive floats.
// Float32 products run at twice the vector rate on the matrix cores, and the rotation no longer takes 64 KB of LDS and
// twelve LDS reads per 32 multiply-adds, which left one workgroup per compute unit.  The matrix instructions of a workgroup, 8 k
// cycles, wait for its rows and its residual, so it is workgroups on a unit that fill them: W comes through the scalar cache, C
// lies in LDS in the binary16 it is stored in, and Pi is read when the rows of the block are done with their registers, which
// leaves room for four a unit instead of two.  8192 workgroups of 64 rows at 1 bit 244 -> 200 us, 1000 at 4 bits 41 -> 36.5 (of
// which 13 are the matrix cores' rate and 8 that of memory).
// The product comes out with the coordinates of a row in a lane's registers (HalfBounds): 2 us less of a compress call of 125
// blocks of 512 at 4 bits than with comparison masks dealt out to the rows.
// ---------------------------------------------------------------------------
constexpr int ENC_ROWS = 64;
constexpr int ENC_THREADS = 256;
constexpr int LDS_X = D + 4;                 // row stride in floats: 16-byte reads of 32 rows hit every bank alike
constexpr int LDS_C = EOQ_RMAX_CAP + 1;
typedef float float16v __attribute__((ext_vector_type(16)));

template <int BITS>
__global__ __launch_bounds__(ENC_THREADS, 4) void eoq_encode_kernel(
    const float* __restrict__ blocks, EoqBlockMap map, int64_t b0, int n, int r_max, const float* __restrict__ pi,
    const float* __restrict__ tab, const float* __restrict__ wfac, const int32_t* __restrict__ rank_in,
    const uint16_t* __restrict__ rfac, uint16_t* __restrict__ lfac, uint16_t* __restrict__ norms,
    uint8_t* __restrict__ codes) {
  __shared__ __align__(16) float X[ENC_ROWS * LDS_X];      // rows of S, then sqrt(d) u
  __shared__ uint16_t Cl[ENC_ROWS * LDS_C];                // C as stored
  constexpr int ROWB = BITS * D / 8;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const size_t blk = (size_t)b0 + blockIdx.y;
  const size_t slot = map.slot(blk);
  const int row0 = blockIdx.x * ENC_ROWS;
  const int r = rank_in[slot];

  {
    const float* src = blocks + map.in_base(blk) + (size_t)(row0 + (tid >> 5)) * (size_t)map.token_stride + 4 * (tid & 31);
    float4 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = *reinterpret_cast<const float4*>(src + (size_t)(8 * k) * (size_t)map.token_stride);
#pragma unroll
    for (int k = 0; k < 8; ++k) *reinterpret_cast<float4*>(X + (8 * k + (tid >> 5)) * LDS_X + 4 * (tid & 31)) = x[k];
  }
  HalfBounds<BITS> bnd;
  bnd.load(tab + 16);
  __syncthreads();

  // C = S W^T (= U diag(phi)), rounded to the stored binary16 (Alg. 2 Return, Alg. 3 Store)
  for (int i = wave; i < r; i += 4) {
    const float* w = wfac + (blk * r_max + i) * D;   // V diag(phi/sigma): the same for every lane, through the scalar cache
    float s0 = 0.0f, s1 = 0.0f;
#pragma unroll 8
    for (int j = 0; j < D; j += 4) {
      const float4 x = *reinterpret_cast<const float4*>(X + lane * LDS_X + j);
      s0 = fmaf(x.x, w[j], s0);
      s1 = fmaf(x.y, w[j + 1], s1);
      s0 = fmaf(x.z, w[j + 2], s0);
      s1 = fmaf(x.w, w[j + 3], s1);
    }
    const uint16_t hb = float_to_half_bits(s0 + s1);
    lfac[(slot * r_max + i) * (size_t)n + row0 + lane] = hb;
    Cl[lane * LDS_C + i] = hb;
  }
  __syncthreads();

  // R = S - C V^T (Alg. 3; the whole block when r = 0), rho_t = |R_t|, sqrt(d) u_t = sqrt(d) R_t / rho_t (Alg. 1 line 3):
  // a half wave takes eight rows, a lane the columns 4 l32 .. + 3 of them
  {
    const int tr = tid >> 5;
    float4 x[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) x[a] = *reinterpret_cast<const float4*>(X + (8 * tr + a) * LDS_X + 4 * l32);
    const uint16_t* vrow = rfac + slot * r_max * D + 4 * l32;
#pragma unroll 2
    for (int i = 0; i < r; ++i) {
      const uint2 h = *reinterpret_cast<const uint2*>(vrow + i * D);
      const float v0 = half_bits_to_float((uint16_t)(h.x & 0xFFFFu)), v1 = half_bits_to_float((uint16_t)(h.x >> 16));
      const float v2 = half_bits_to_float((uint16_t)(h.y & 0xFFFFu)), v3 = half_bits_to_float((uint16_t)(h.y >> 16));
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const float c = half_bits_to_float(Cl[(8 * tr + a) * LDS_C + i]);
        x[a].x = fmaf(-c, v0, x[a].x);
        x[a].y = fmaf(-c, v1, x[a].y);
        x[a].z = fmaf(-c, v2, x[a].z);
        x[a].w = fmaf(-c, v3, x[a].w);
      }
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      float ss = fmaf(x[a].x, x[a].x, fmaf(x[a].y, x[a].y, fmaf(x[a].z, x[a].z, x[a].w * x[a].w)));
      ss += dpp_mov<0xB1>(ss);
      ss += dpp_mov<0x4E>(ss);
      ss += dpp_mov<0x141>(ss);
      ss += dpp_mov<0x140>(ss);
      ss += __shfl_xor(ss, 16, 64);
      const float rho = sqrtf(ss);
      const float sc = (rho > 0.0f) ? sqrtf((float)D) / rho : 0.0f;
      if (l32 == 0) norms[slot * (size_t)n + row0 + 8 * tr + a] = float_to_half_bits(rho);
      *reinterpret_cast<float4*>(X + (8 * tr + a) * LDS_X + 4 * l32) = make_float4(x[a].x * sc, x[a].y * sc, x[a].z * sc, x[a].w * sc);
    }
  }
  __syncthreads();

  // z = Pi u (Alg. 1 line 4) and index of the nearest centroid (line 5): two tiles of 32 rows
  float4 P[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) P[m] = *reinterpret_cast<const float4*>(pi + (32 * wave + plane_row(l32)) * D + 8 * m + 4 * hf);
  float16v acc[2];
  EOQ_SFOR(t, 2, EOQ_SFOR(v, 16, acc[t][v] = 0.0f;););
  EOQ_SFOR(m, 16,
    const float4 u0 = *reinterpret_cast<const float4*>(X + l32 * LDS_X + 8 * m + 4 * hf);
    const float4 u1 = *reinterpret_cast<const float4*>(X + (32 + l32) * LDS_X + 8 * m + 4 * hf);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].x, u0.x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].x, u1.x, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].y, u0.y, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].y, u1.y, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].z, u0.z, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].z, u1.z, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].w, u0.w, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(P[m].w, u1.w, acc[1], 0, 0, 0);
  );
  // bit-planes of row 32 t + l32, two half words at a time: the lower half of the wave stores the first, the upper half the second
  uint32_t held = 0u;
  EOQ_SFOR(t, 2,
    uint32_t below[BITS];
    bnd.planes(acc[t], below);
    EOQ_SFOR(p, BITS,
      constexpr int item = t * BITS + p;
      if constexpr (item % 2 == 0) {
        held = below[p];
      } else {
        constexpr int at_a = (item - 1) / BITS * 32 * ROWB + (item - 1) % BITS * 16; constexpr int at_b = 32 * t * ROWB + 16 * p;
        uint8_t* dst = codes + (slot * (size_t)n + row0 + l32) * ROWB + 4 * wave + (hf ? at_b : at_a);
        *reinterpret_cast<uint32_t*>(dst) = plane_words(held, below[p]);
      }
    );
  );
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t eoq_launch_encode(const EoqLaunch& L, const void* blocks, int dtype, int64_t B, const float* wfac,
                             eoq_packed out) {
  if (L.ev) (void)hipEventRecord(L.ev[2], L.stream);
  if (dtype == EOQ_F16) {  // binary16 blocks go to the matrix-core kernel
    const hipError_t e = eoq_launch_encode_f16(L, blocks, B, wfac, out);
    if (L.ev) (void)hipEventRecord(L.ev[3], L.stream);
    return e;
  }
  // gridDim.y is limited to 65535: split long batches
  for (int64_t b0 = 0; b0 < B; b0 += 32768) {
    const int64_t nb = (B - b0 < 32768) ? B - b0 : 32768;
#define EOQ_ENCODE(BITS)                                                                                               \
  hipLaunchKernelGGL(eoq_encode_kernel<BITS>, dim3(L.n / ENC_ROWS, (unsigned)nb), dim3(ENC_THREADS), 0, L.stream,     \
                     static_cast<const float*>(blocks), L.map, b0, L.n, L.r_max, L.pi, L.tab, wfac, out.rank,          \
                     out.rfac, out.lfac, out.norms, out.codes)
    switch (L.bits) {
      case 1: EOQ_ENCODE(1); break;
      case 2: EOQ_ENCODE(2); break;
      case 3: EOQ_ENCODE(3); break;
      default: EOQ_ENCODE(4); break;
    }
#undef EOQ_ENCODE
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (L.ev) (void)hipEventRecord(L.ev[3], L.stream);
  return hipSuccess;
}

