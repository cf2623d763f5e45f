// Decode scoring on compressed keys (Sec. 2.1 attention logits, Remark 6.5): scores[s][h][t] = <q_h, x_hat_t>/sqrt(d)
// from the record, without forming x_hat.  With x_hat_t = rho_t Pi^T z_hat_t + C_t V_r:
//     <q, x_hat_t> = rho_t <Pi q, z_hat_t> + <C_t, V_r^T q>.
//
// The first term runs on the integer matrix cores.  The codebook is symmetric, so a centroid is its sign times a
// magnitude that is a multilinear function of the magnitude bits m_p (index bit p of the code, inverted on the negative
// half):  z_hat_j = s_j sum_M coef[M] prod_{p in M} m_pj over the subsets M of the b-1 magnitude bits (b = 2: c_0 + (c_1 -
// c_0) m_0).  Every term is an inner product of q' = Pi q with a vector of entries in {-1, 0, +1}: exact in int8.  q' is
// multiplied by the coefficient of its term and held in 32-bit fixed point per head (a power-of-two unit, four balanced
// signed bytes): the 32 rows of the A operand of v_mfma_i32_32x32x32_i8 are the four byte planes of eight query heads,
// the terms of a coordinate sit side by side along k (one int32 accumulator takes the whole sum, exactly) and the
// columns are 32 tokens.
// Operand convention of v_mfma_i32_32x32x32_i8 (wave64): lane l supplies A[row = l%32][k = 16*(l/32) .. +15] and
// B[k = 16*(l/32) .. +15][col = l%32] and receives D[row = 8*(v/4) + 4*(l/32) + v%4][col = l%32] in accumulator
// register v.  Row 8 q + 4 f + e is byte plane e of head 2 q + f: lane (token, f) receives all four planes of the heads
// f, 2 + f, 4 + f, 6 + f of ITS token, joins them, scales by its own stored norm and stores -- nothing changes lanes.
// The low-rank term rides the f16 matrix cores the same way: rows e = 0 / 1 of head 2 q + f hold the binary16 hi / lo
// parts of w_h = V_r^T q_h / sqrt(d), the B operand the token's stored coefficients.
// The {-1, 0, +1} operands come out of tables in LDS.  Up to 2 bits one table of 256 entries, indexed by a nibble of the sign plane
// and one of the magnitude plane: four coordinates of two terms per 8-byte read, in the order the matrix instruction takes
// them.  From 3 bits on two tables of 16 words, the signs of a nibble and the byte mask of a nibble of a magnitude plane, and
// an AND: sixteen words lie in sixteen banks, so the lanes' lookups, which collide at random in the large table, never do
// (3 and 4 bits, one to eight heads: logits of 1 M to 8.4 M tokens 10 to 16 % shorter, with the correction 8 to 13 %, of 262144
// tokens 4 to 8 % and 3 to 5 %; 4.2 M tokens at four heads, us: 95.9 -> 83.8 and 149 -> 131, corrected 125 -> 109 and 170 -> 152.  At 2 bits the additional lookups and
// ANDs cost more than the collisions, 3 %; and with the correction at 4 bits and more than four heads, where 268 registers leave
// one wave to a SIMD, the chain of lookup and AND does, 1 to 3 %: those have the table of pairs).  The
// lane that owns a token reads its 8 bytes of every bit-plane straight from the record (lane half f: coordinates 64 f ..
// 64 f + 63).
#include "eoq_device.h"
#include "eoq_internal.h"

namespace {

using namespace eoqdev;

constexpr int D = EOQ_D;
constexpr int THREADS = 256;
constexpr int SC_MAXG = 8;      // most query heads per KV head
constexpr int SC_RUN_MAX = 16;  // most blocks per workgroup (the run is shortened until the grid fills the chip)

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
union H8 {
  half8 h;
  uint4 u;
  uint32_t w[4];
  uint16_t s[8];
};

// Buffer descriptor over `bytes` bytes at `base` (raw addressing: loads past the end return zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes > 0x7FFFFFFFu ? 0x7FFFFFFFu : bytes),
                                           0x00020000);
}
__device__ __forceinline__ float4v mfma32(const H8& a, const H8& b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) { return (mask & a) | (~mask & b); }

// out[h][c] = sum_j table[c][j] q[h][j] for the heads of one group (rows above the group are zero), the table given as
// binary16 hi + lo parts [c][j] (LO = false: it is binary16 to begin with): the query side of the rotation (<q, Pi^T z> =
// <Pi q, z>) and of the projection Phi q.  q is binary16, so every product is exact; v_mfma_f32_16x16x32_f16, A operand
// `a` = q: lane (l16, g) holds q[l16][32 ks + 8 g .. + 7].  The loads are a step of their own so that they are in flight
// together.  `out` is LDS, [SC_MAXG][D]; the caller synchronises.
template <bool LO>
struct TableRows {
  H8 hi[2][4], lo[2][LO ? 4 : 1];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ tab_hi, const uint16_t* __restrict__ tab_lo, int wave, int l16, int g) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int at = (16 * (2 * wave + tt) + l16) * D + 32 * ks + 8 * g;
        hi[tt][ks].u = *reinterpret_cast<const uint4*>(tab_hi + at);
        if constexpr (LO) lo[tt][ks].u = *reinterpret_cast<const uint4*>(tab_lo + at);
      }
  }
  __device__ __forceinline__ void rotate(const H8 (&a)[4], float* out, int wave, int l16, int g) const {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int c = 16 * (2 * wave + tt) + l16;
      float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        acc = mfma32(a[ks], hi[tt][ks], acc);
        if constexpr (LO) acc = mfma32(a[ks], lo[tt][ks], acc);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (4 * g + v < SC_MAXG) out[(4 * g + v) * D + c] = acc[v];
    }
  }
};

// Rows of `rows` ([SC_MAXG][D] float, LDS), each multiplied by the NT coefficients coef[0 .. NT-1], to 32-bit fixed
// point: per row the unit is 2^(E - 29) with E the exponent of the largest |coef| |entry| of the row, so |integer| <=
// 2^30; the integer is cut into four balanced signed bytes (the bytes of I + 0x80808080 with the top bit of each flipped)
// and byte plane p of row h goes to dig[(4 h + p) * dig_stride(NT) + ...] with the NT terms of four consecutive coordinates side
// by side: byte ((c / 4) * NT + term) * 4 + c % 4 -- the order of k in the matrix instructions.  unit[h] = value of one
// integer unit (0 for a row that is zero, below 2^-87 or not finite).  All 256 lanes, 32 per row; the caller synchronises.
// 16 bytes more than the row has: the lanes of an operand read, a row each, meet all banks (a multiple of 256 bytes put
// them all on the same four: 8.5 of 55 thousand cycles of a workgroup at 4 bits)
constexpr int dig_stride(int terms) { return terms * D + 16; }
template <int NT>
__device__ __forceinline__ void fixed_point_rows(const float* rows, const float (&coef)[NT], unsigned char* dig, float* unit,
                                                 int tid) {
  const int h = tid >> 5, c0 = 4 * (tid & 31);
  float cmax = 0.0f;
#pragma unroll
  for (int t = 0; t < NT; ++t) cmax = fmaxf(cmax, fabsf(coef[t]));
  float v[4];
  int m = 0;   // bits of the largest magnitude
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = rows[h * D + c0 + e];
    m = max(m, __float_as_int(fabsf(v[e]) * cmax));
  }
  m = max(m, dpp_mov<0xB1>(m));
  m = max(m, dpp_mov<0x4E>(m));
  m = max(m, dpp_mov<0x141>(m));
  m = max(m, dpp_mov<0x140>(m));
  m = max(m, __shfl_xor(m, 16, 64));
  const int eb = m >> 23;   // biased exponent of the row maximum
  const bool live = eb >= 40 && eb < 255;
  const double up = live ? (double)__uint_as_float((unsigned)(283 - eb) << 23) : 0.0;   // 2^(29 - (eb - 127))
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    uint32_t dg[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int I = live ? __double2int_rn((double)v[e] * (double)coef[t] * up) : 0;   // one rounding, |I| <= 2^30
      dg[e] = ((uint32_t)I + 0x80808080u) ^ 0x80808080u;
    }
    uint32_t pl[4];
    transpose_bytes(dg[0], dg[1], dg[2], dg[3], pl);
#pragma unroll
    for (int p = 0; p < 4; ++p) *reinterpret_cast<uint32_t*>(dig + (4 * h + p) * dig_stride(NT) + ((c0 >> 2) * NT + t) * 4) = pl[p];
  }
  if ((tid & 31) == 0) unit[h] = live ? __uint_as_float((unsigned)(eb - 29) << 23) : 0.0f;
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float float16v __attribute__((ext_vector_type(16)));
constexpr int CTLD = 32 + 8;   // row stride (halfs) of a tile's coefficient rows in LDS, [component][token]

// What a lane requests of a tile of 32 consecutive tokens: lane (l32, hf) owns token l32.
template <int BITS, bool QJL>
struct TileFetch {
  u32x2 pl[BITS];            // bytes 8 hf .. 8 hf + 7 of every bit-plane of the token
  uint32_t rho;              // the token's stored norm (binary16 in the low half)
  u32x4 cf;                  // lane L: stored coefficients C[tokens 8 (L % 4) .. + 7][component L / 4]; zero at and above the rank
  u32x2 sg[QJL ? 1 : 0];     // the same bytes of sign(Phi r_x)
  uint32_t gam[QJL ? 1 : 0]; // the token's stored residual norm
};

// Scores of the uncompressed tail (the newest tokens of every head, binary16, not yet a full block):
// row[h][t] = <q[h], tail[t]> / sqrt(d) for the tokens t0 .. t0 + TAIL_TOK - 1 of one (sequence, KV head).  16 lanes share a
// token (16 bytes each), float32 accumulation of exact binary16 products.  These are further workgroups of the scores
// kernel, 64 tokens each: a kernel of their own cost a launch, and with one workgroup per head 32 us at 12 heads and 389
// tokens.
constexpr int TAIL_TOK = 64;
constexpr int QUAD = 128;   // tokens of one tile of each of the four waves
__device__ __forceinline__ void tail_scores(const uint16_t* __restrict__ tail, int t0, int tail_len,
                                            const uint16_t* __restrict__ q, int group, float* __restrict__ row, size_t T, float* qs,
                                            int tid) {
  const int l16 = tid & 15;
  float x[TAIL_TOK / 16][8];
#pragma unroll
  for (int i = 0; i < TAIL_TOK / 16; ++i) {
    const int t = t0 + 16 * i + (tid >> 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[i][e] = 0.0f;
    if (t < tail_len) load8(tail, EOQ_F16, (size_t)t * D + 8 * l16, x[i]);
  }
  for (int e = tid; e < group * D; e += THREADS) qs[e] = half_bits_to_float(q[e]);
  __syncthreads();
  const float inv_sqrt_d = 1.0f / sqrtf((float)D);
  for (int h = 0; h < group; ++h) {
    const float4 q0 = *reinterpret_cast<const float4*>(qs + h * D + 8 * l16), q1 = *reinterpret_cast<const float4*>(qs + h * D + 8 * l16 + 4);
    const float qv[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
    for (int i = 0; i < TAIL_TOK / 16; ++i) {
      const int t = t0 + 16 * i + (tid >> 4);
      float acc = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(x[i][e], qv[e], acc);
      acc += dpp_mov<0xB1>(acc);
      acc += dpp_mov<0x4E>(acc);
      acc += dpp_mov<0x141>(acc);
      acc += dpp_mov<0x140>(acc);
      if (l16 == 0 && t < tail_len) row[h * T + t] = acc * inv_sqrt_d;
    }
  }
}

// One workgroup per (sequence, KV head, run of tokens); every wave works on 32-token tiles of its own (wave w takes the tiles
// w, w + 4, ... of the run), the record bytes of the next tile on their way while this one is worked on.  A run is a number of
// steps of 128 tokens, a tile for each wave, and may begin and end inside a block (eoq_scores_run).  NQ = query heads a lane
// finishes per token (2 for groups up to 4).
// QJL: the logits get the correction of Eq. (qjl), |r_x| sqrt(pi/2)/d <Phi q, sign(Phi r_x)>, from one more bit plane
// (the signs) and the stored residual norm; Phi q goes through the same fixed-point form as Pi q.
// (With the correction at 3 bits the compiler is told that two workgroups on a unit are what to schedule for: it went for a third,
// which the registers do not allow, and gave every product of a tile the same operand registers, so that each waited for its own
// reads of the table: one head of 1000 blocks of 512 26.5 us and now 24.4, 3 x 64 blocks 13.1 and 11.6.)
template <int BITS, bool QJL, int NQ>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu((BITS <= 2 && !QJL) ? 4 : 1, (QJL && BITS == 3) ? 2 : 8)))
void eoq_scores_i8_kernel(
    int n, int r_max, int n_kv_heads, int group, int64_t blocks_per_head, int64_t block_capacity, int64_t score_stride,
    int run, const uint16_t* __restrict__ pih,
    const float* __restrict__ tab, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ norms,
    const int32_t* __restrict__ rank_in, const uint16_t* __restrict__ lfac, const uint16_t* __restrict__ rfac,
    const uint16_t* __restrict__ q, float* __restrict__ scores, const uint16_t* __restrict__ phih,
    const uint8_t* __restrict__ qsigns, const uint16_t* __restrict__ qnorms, int run_heads, const uint16_t* __restrict__ tail,
    int64_t tail_capacity, int tail_len, int heads) {
  constexpr int TYPES = 1 << (BITS - 1);
  constexpr int NMM = 4 * TYPES;   // matrix instructions per tile: 64 coordinates x TYPES bytes per lane, 16 at a time
  // One pool, used in turn: during the set-up the rotated query and the byte planes of coef[M] Pi q ([head][plane][k])
  // and of Phi q; in the tile loop the four waves' coefficient tiles.
  constexpr int ROT_BYTES = SC_MAXG * D * 4 * (QJL ? 2 : 1);
  constexpr int SETUP_BYTES = ROT_BYTES + SC_MAXG * 4 * dig_stride(TYPES) + (QJL ? SC_MAXG * 4 * dig_stride(1) : 0);
  constexpr int CS_BYTES = 4 * 2 * 16 * CTLD * 2;
  __shared__ __align__(16) unsigned char pool[SETUP_BYTES > CS_BYTES ? SETUP_BYTES : CS_BYTES];
  float* qrot = reinterpret_cast<float*>(pool);
  float* prot = qrot + SC_MAXG * D;
  unsigned char* qdig = pool + ROT_BYTES;
  unsigned char* pdig = qdig + SC_MAXG * 4 * dig_stride(TYPES);
  // A operands of the low-rank product, components 16 k2 .. + 15 of every block of the run: entry (16 f + 2 h + part) of a
  // block are components 8 f .. + 7 of head h, part 0 binary16(w), part 1 what that rounding lost
  __shared__ __align__(16) uint4 wop[2][SC_RUN_MAX * 32];
  constexpr bool PAIRS = BITS <= 2 || (BITS == 4 && QJL && NQ == 4);   // one table of pairs
  __shared__ __align__(PAIRS ? 16 : 64) uint2 nib_tab[PAIRS ? 256 : 16];   // PAIRS: signs, masked signs; else sign and mask words of a nibble: sign_tab, mask_tab
  uint32_t* sign_tab = reinterpret_cast<uint32_t*>(nib_tab);
  uint32_t* mask_tab = sign_tab + 16;
  __shared__ float qunit[SC_MAXG], punit[SC_MAXG];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave: scalar
  const int l16 = lane & 15, g = lane >> 4;
  const int l32 = lane & 31, hf = lane >> 5;
  const int n_q_heads = n_kv_heads * group;
  const size_t T = (size_t)score_stride;   // entries per score row (>= blocks_per_head * n)
  constexpr int ROWB = BITS * D / 8;
  const float inv_sqrt_d = 1.0f / sqrtf((float)D);
  if ((int)blockIdx.y >= run_heads) {   // a workgroup of the tail, or none: see scores_grid
    const uint32_t id = (blockIdx.y - (uint32_t)run_heads) * gridDim.x + blockIdx.x;
    const uint32_t per_head = (uint32_t)(tail_len + TAIL_TOK - 1) / TAIL_TOK, head = id / per_head;
    if (head >= (uint32_t)heads) return;
    const size_t first = (size_t)(head / n_kv_heads) * n_q_heads + (head % n_kv_heads) * group;   // query head
    tail_scores(tail + head * (size_t)tail_capacity * D, TAIL_TOK * (int)(id - head * per_head), tail_len, q + first * D, group,
                scores + first * T + (size_t)blocks_per_head * n, T, qrot, tid);
    return;
  }
  const size_t sg = blockIdx.y;
  const size_t sq = sg / n_kv_heads, kv = sg % n_kv_heads;
  const size_t q0 = (sq * n_q_heads + kv * group) * D;

  // the run: `run` steps of QUAD tokens from step number blockIdx.x * run of the head, which is token tok0 of block jb0; the
  // blocks it touches are numbers 0 .. nblk - 1 of the run (B n < 2^39: a step number fits 32 bits)
  const uint32_t steps_per_block = (uint32_t)n / QUAD;
  const uint32_t step0 = blockIdx.x * (uint32_t)run;
  const int count = (int)min((uint32_t)run, (uint32_t)blocks_per_head * steps_per_block - step0);   // tiles of every wave
  const uint32_t first_block = step0 / steps_per_block, in_block = step0 - first_block * steps_per_block;
  const int64_t jb0 = first_block;
  const int tok0 = QUAD * (int)in_block;
  const int nblk = (int)((in_block + (uint32_t)count - 1) / steps_per_block) + 1;
  const size_t blk0 = sg * (size_t)block_capacity + jb0;   // the store holds block_capacity slots per head

  // ---- set-up.  It is paid once per workgroup and is latency: everything that depends on nothing is requested first
  // (ranks, query, tables), then the first tile and the right factors of the wave's share of the blocks, which travel while
  // the rotated query is cut into bytes.  (One table row after the other behind a branch, and the products with the
  // right factors as a loop of loads and sums over lanes, took 65 of 213 thousand cycles of a workgroup at 16 blocks of 512.)
  int rk_all = rank_in[blk0 + min(lane & 15, nblk - 1)];   // ranks of the run's blocks, one per lane
  H8 aq[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    aq[ks].u = (l16 < group) ? *reinterpret_cast<const uint4*>(q + q0 + l16 * D + 32 * ks + 8 * g) : make_uint4(0u, 0u, 0u, 0u);
  TableRows<true> pi_rows;
  pi_rows.load(pih, pih + D * D, wave, l16, g);
  {
    const int tn = tid & 15, xn = tid >> 4;
    uint32_t sd = 0u, td = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t sb = ((tn >> e) & 1) ? 0x01u : 0xFFu;   // sign plane bit set: +1
      sd |= sb << (8 * e);
      if constexpr (PAIRS) {
        if ((xn >> e) & 1) td |= sb << (8 * e);
      } else {
        if ((tn >> e) & 1) td |= 0xFFu << (8 * e);
      }
    }
    if constexpr (PAIRS) nib_tab[tid] = make_uint2(sd, td);
    else if (tid < 32) sign_tab[tid] = tid < 16 ? sd : td;
  }
  // coefficients of the multilinear form of the magnitudes: level number sum_p m_p 2^p is centroid L/2 + level of the
  // ascending N(0,1) table; coef[M] = sum over subsets S of M of (-1)^(|M| - |S|) centroid[L/2 + S]
  float coef[TYPES];
#pragma unroll
  for (int M = 0; M < TYPES; ++M) {
    float c = 0.0f;
#pragma unroll
    for (int S = 0; S < TYPES; ++S)
      if ((S & M) == S) c += ((__builtin_popcount(M ^ S) & 1) ? -1.0f : 1.0f) * tab[TYPES + S];
    coef[M] = c;
  }
  // Buffer addressing: a resource descriptor in scalar registers, a scalar byte offset that moves from tile to tile and
  // a per-lane 32-bit offset that never changes -- no vector arithmetic per load.  The coefficients get a descriptor per
  // block that ends behind row rank - 1, and the range check covers the per-lane part of the offset, which holds the
  // row: rows at and above the rank read zero.
  const uint8_t* codes0 = codes + blk0 * (size_t)n * ROWB;
  const uint16_t* norms0 = norms + blk0 * (size_t)n;
  const uint8_t* qsigns0 = QJL ? qsigns + blk0 * (size_t)n * (D / 8) : nullptr;
  const uint16_t* qnorms0 = QJL ? qnorms + blk0 * (size_t)n : nullptr;
  // score rows of this (sequence, KV head): row h at h T floats; lane (token, hf) stores head 2 qq + hf
  float* scores0 = scores + (sq * n_q_heads + kv * group) * T;
  const uint32_t vo_code = (uint32_t)(l32 * ROWB + 8 * hf);
  const uint32_t vo_sign = (uint32_t)(l32 * (D / 8) + 8 * hf);
  const uint32_t vo_norm = (uint32_t)(2 * l32);
  const uint32_t vo_cf = (uint32_t)(((lane >> 2) * n + (lane & 3) * 8) * 2);
  const uint32_t vo_out = (uint32_t)((hf * T + l32) * 4);
  uint16_t* cs = reinterpret_cast<uint16_t*>(pool) + wave * (2 * 16 * CTLD);

  // The scalar unit is shared by the whole compute unit, so what a tile costs in scalar instructions counts: the
  // descriptors of the run are built once, a tile is addressed by its first token counted from the start of the run
  // (the wave's tiles are 128 tokens apart, also across a block boundary), the ranks of the run's blocks sit in the
  // lanes of one register, and the descriptor of a block's coefficients is rebuilt only when the block changes.
  const __amdgpu_buffer_rsrc_t bcodes = buffer_of(codes0, (size_t)nblk * n * ROWB);
  const __amdgpu_buffer_rsrc_t bnorms = buffer_of(norms0, (size_t)nblk * n * 2);
  const __amdgpu_buffer_rsrc_t bsigns = buffer_of(qsigns0, QJL ? (size_t)nblk * n * (D / 8) : 0);
  const __amdgpu_buffer_rsrc_t bgam = buffer_of(qnorms0, QJL ? (size_t)nblk * n * 2 : 0);
  const __amdgpu_buffer_rsrc_t bout = buffer_of(scores0 + (size_t)jb0 * n, ((size_t)group * T - (size_t)jb0 * n) * 4);
  rk_all = min(max(rk_all, 0), r_max);   // records may come from storage: never index past r_max rows
  auto rank_of = [&](int b) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(rk_all, b); };
  auto coef_buffer = [&](int b) __attribute__((always_inline)) {
    return buffer_of(lfac + (blk0 + b) * (size_t)r_max * n, (size_t)rank_of(b) * n * 2);
  };
  // the tile whose first token is number tok of the run, in block b (first token b n), coefficients through cfd
  auto request = [&](TileFetch<BITS, QJL>& f, int tok, int b, __amdgpu_buffer_rsrc_t cfd) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < BITS; ++p) f.pl[p] = __builtin_amdgcn_raw_buffer_load_b64(bcodes, vo_code + 16 * p, tok * ROWB, 0);
    f.rho = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bnorms, vo_norm, tok * 2, 0);
    f.cf = __builtin_amdgcn_raw_buffer_load_b128(cfd, vo_cf, (tok - b * n) * 2, 0);
    if constexpr (QJL) {
      f.sg[0] = __builtin_amdgcn_raw_buffer_load_b64(bsigns, vo_sign, tok * (D / 8), 0);
      f.gam[0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bgam, vo_norm, tok * 2, 0);
    }
  };
  // A operand of the low-rank product for block b of the run, components 16 k2 + 8 hf + e: row 8 qq + 4 f of the matrix
  // instruction holds binary16(w) of head 2 qq + f, the row after it what that rounding lost, the other two rows are zero
  auto w_operand = [&](int b, int k2) __attribute__((always_inline)) {
    H8 x;
    x.u = ((l32 & 3) < 2) ? wop[k2][b * 32 + 16 * hf + 2 * (l32 >> 2) + (l32 & 1)] : make_uint4(0u, 0u, 0u, 0u);
    return x;
  };
  // C[token l32][16 k2 + 8 hf + e] of the rows staged in the wave's coefficient tile: the B operand of that product
  auto c_operand = [&](int k2) __attribute__((always_inline)) {
    H8 x;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t a = cs[(16 * k2 + 8 * hf + 2 * w) * CTLD + l32], b = cs[(16 * k2 + 8 * hf + 2 * w + 1) * CTLD + l32];
      x.w[w] = a | (b << 16);
    }
    return x;
  };

  // the first tile's record bytes
  TileFetch<BITS, QJL> f0, f1;
  const int tok_last = tok0 + 32 * wave + QUAD * (count - 1);
  int tok_r = tok0 + 32 * wave, b_r = 0, end_r = n;           // next tile to request: first token, block, end of the block
  __amdgpu_buffer_rsrc_t cfd = coef_buffer(0);
#define EOQ_SC_REQUEST(F)                    \
  if (tok_r >= end_r) {                      \
    ++b_r;                                   \
    end_r += n;                              \
    cfd = coef_buffer(b_r);                  \
  }                                          \
  request(F, tok_r, b_r, cfd);               \
  tok_r = min(tok_r + QUAD, tok_last);
  // q' = Pi q (the rotation moved to the query side: <q, Pi^T z> = <Pi q, z>), and Phi q
  pi_rows.rotate(aq, qrot, wave, l16, g);
  if constexpr (QJL) {
    TableRows<false> phi_rows;
    phi_rows.load(phih, nullptr, wave, l16, g);
    phi_rows.rotate(aq, prot, wave, l16, g);
  }
  EOQ_SC_REQUEST(f0)
  // w[i][h] = <v_i, q_h> / sqrt(d) of the run's blocks (the low-rank term is <C_t, w_h>): the same matrix product with the
  // right factors as table, block b by wave b % 4, rows at and above the rank zero by the descriptor; component 16 k2 + l16
  constexpr int VB = SC_RUN_MAX / 4;
  H8 vrow[VB][4];
  auto load_v = [&](H8 (&v)[4], int b, int k2) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t vb = buffer_of(rfac + (blk0 + b) * (size_t)r_max * D, (size_t)rank_of(b) * D * 2);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(vb, (uint32_t)(((16 * k2 + l16) * D + 32 * ks + 8 * g) * 2), 0, 0);
      v[ks].u = make_uint4(x[0], x[1], x[2], x[3]);
    }
  };
  auto put_w = [&](const H8 (&v)[4], int b, int k2) __attribute__((always_inline)) {
    float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = mfma32(aq[ks], v[ks], acc);
    uint16_t* dst = reinterpret_cast<uint16_t*>(&wop[k2][b * 32 + 16 * (l16 >> 3)]) + (l16 & 7);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int h = 4 * g + e;
      if (h < SC_MAXG) {
        const float w = acc[e] * inv_sqrt_d;
        const uint16_t hi = float_to_half_bits(w);
        dst[16 * h] = hi;
        dst[16 * h + 8] = float_to_half_bits(w - half_bits_to_float(hi));
      }
    }
  };
#pragma unroll
  for (int k = 0; k < VB; ++k)
    if (4 * k + wave < nblk) load_v(vrow[k], 4 * k + wave, 0);   // uniform
  __syncthreads();   // qrot (and prot) written
  fixed_point_rows<TYPES>(qrot, coef, qdig, qunit, tid);
  if constexpr (QJL) {
    const float one[1] = {1.0f};
    fixed_point_rows<1>(prot, one, pdig, punit, tid);
  }
#pragma unroll
  for (int k = 0; k < VB; ++k)
    if (4 * k + wave < nblk) {
      put_w(vrow[k], 4 * k + wave, 0);
      if (rank_of(4 * k + wave) > 16) {   // rare
        load_v(vrow[k], 4 * k + wave, 1);
        put_w(vrow[k], 4 * k + wave, 1);
      }
    }
  __syncthreads();   // byte planes and low-rank operands written
  // A operands: row l32 = byte plane l32 % 4 of head 2 (l32 / 8) + (l32 / 4) % 2; instruction i covers the 16 bytes of k
  // from 16 i of lane half hf's 64 coordinates (64 TYPES bytes: per nibble of four coordinates the TYPES terms).  Kq / Kp:
  // what one integer unit of head 2 qq + hf is worth in the logit.
  const int arow = 4 * (2 * (l32 >> 3) + ((l32 >> 2) & 1)) + (l32 & 3);   // row of the byte planes: 4 head + plane
  v4i Aq[NMM], Ap[QJL ? 4 : 1];
  float Kq[NQ], Kp[QJL ? NQ : 1];
  const float qjl_scale = sqrtf(1.5707963267948966f) / (float)D;
#pragma unroll
  for (int i = 0; i < NMM; ++i) Aq[i] = *reinterpret_cast<const v4i*>(qdig + arow * dig_stride(TYPES) + 64 * TYPES * hf + 16 * i);
#pragma unroll
  for (int qq = 0; qq < NQ; ++qq) Kq[qq] = qunit[2 * qq + hf] * (1.0f / (float)D);   // z_hat = centroid / sqrt(d), logit = <q, x_hat> / sqrt(d)
  if constexpr (QJL) {
#pragma unroll
    for (int i = 0; i < 4; ++i) Ap[i] = *reinterpret_cast<const v4i*>(pdig + arow * dig_stride(1) + 64 * hf + 16 * i);
#pragma unroll
    for (int qq = 0; qq < NQ; ++qq) Kp[qq] = punit[2 * qq + hf] * (qjl_scale * inv_sqrt_d);
  }

  __syncthreads();   // the pool changes hands

  int wb = -1;   // block of the run whose w operand the wave holds
  H8 Aw;
  Aw.u = make_uint4(0u, 0u, 0u, 0u);
  auto work = [&](TileFetch<BITS, QJL>& cur, int tok, int b, int r) __attribute__((always_inline)) {
    if (b != wb) {   // uniform
      Aw = w_operand(b, 0);
      wb = b;
    }
    // ---- the integer term: the lane's 64 coordinates, byte kk of every plane at a time ----
    const uint32_t top0 = cur.pl[BITS - 1][0], top1 = cur.pl[BITS - 1][1];
    v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
    // byte j of the words made of a plane's word: four times the low / the high nibble of its byte j, a place in a table of words
    auto places = [](uint32_t w, uint32_t (&at)[2]) __attribute__((always_inline)) {
      at[0] = (w << 2) & 0x3C3C3C3Cu;
      at[1] = (w >> 2) & 0x3C3C3C3Cu;
      // opaque: otherwise every lookup shifts and masks the plane's word (two instructions) instead of taking a byte of these
      asm("" : "+v"(at[0]), "+v"(at[1]));
    };
    auto entry = [](const uint32_t* table, const uint32_t (&at)[2], int nibble) __attribute__((always_inline)) {
      return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(table) + __builtin_amdgcn_ubfe(at[nibble & 1], 8 * (nibble >> 1), 8));
    };
    if constexpr (BITS <= 2) {
      // even / odd: byte j = (sign nibble | magnitude nibble << 4) of the low / high nibbles of byte j of the planes;
      // one table read gives the four sign bytes and the same bytes where the magnitude bit is set: 8 of the 16 bytes
      // of an instruction (BITS = 1: the sign bytes alone, 4 of 16)
      uint32_t even[2], odd[2];
#pragma unroll
      for (int wq = 0; wq < 2; ++wq) {
        const uint32_t t = wq ? top1 : top0;
        const uint32_t x = (BITS == 2) ? ~(cur.pl[0][wq] ^ t) : 0u;   // magnitude bit: plane 0 where the sign plane is set, its complement elsewhere
        even[wq] = bfi(0x0F0F0F0Fu, t, x << 4);
        odd[wq] = bfi(0x0F0F0F0Fu, t >> 4, x);
      }
      if constexpr (BITS == 2) {
        EOQ_SFOR(kk, 8,
          const uint2 lo = nib_tab[(even[kk >> 2] >> (8 * (kk & 3))) & 0xFFu], hi = nib_tab[(odd[kk >> 2] >> (8 * (kk & 3))) & 0xFFu];
          const v4i B = {(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
          acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Aq[kk], B, acc, 0, 0, 0);
        );
      } else {
        EOQ_SFOR(i, 4,
          const v4i B = {(int)nib_tab[(even[i >> 1] >> (16 * (i & 1))) & 0xFFu].x, (int)nib_tab[(odd[i >> 1] >> (16 * (i & 1))) & 0xFFu].x,
                         (int)nib_tab[(even[i >> 1] >> (16 * (i & 1) + 8)) & 0xFFu].x, (int)nib_tab[(odd[i >> 1] >> (16 * (i & 1) + 8)) & 0xFFu].x};
          acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Aq[i], B, acc, 0, 0, 0);
        );
      }
    } else if constexpr (PAIRS) {
      // per nibble of four coordinates the TYPES terms, four bytes each: term 0 the signs, term 2^p from the table read
      // of magnitude plane p, the other terms (products of magnitude bits) as bitwise ANDs of those
      EOQ_SFOR(nb, 16,
        constexpr int wq = nb >> 3, sh = 4 * (nb & 7);
        const uint32_t t = wq ? top1 : top0;
        uint32_t term[TYPES];
        EOQ_SFOR(p, BITS - 1,
          const uint32_t x = ~(cur.pl[p][wq] ^ t);
          const uint2 e = nib_tab[((t >> sh) & 0xFu) | (((x >> sh) & 0xFu) << 4)];
          term[0] = e.x;
          term[1 << p] = e.y;
        );
        EOQ_SFOR(M, TYPES,
          if constexpr ((M & (M - 1)) != 0) term[M] = term[M & -M] & term[M ^ (M & -M)];
        );
        EOQ_SFOR(i, TYPES / 4,
          const v4i B = {(int)term[4 * i], (int)term[4 * i + 1], (int)term[4 * i + 2], (int)term[4 * i + 3]};
          acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Aq[nb * (TYPES / 4) + i], B, acc, 0, 0, 0);
        );
      );
    } else {
      // the same from the two small tables: term 2^p is the signs under the mask of magnitude plane p
      EOQ_SFOR(wq, 2,
        const uint32_t t = wq ? top1 : top0;
        uint32_t sat[2], mat[BITS - 1][2];
        places(t, sat);
        EOQ_SFOR(p, BITS - 1, places(~(cur.pl[p][wq] ^ t), mat[p]););
        EOQ_SFOR(nb, 8,
          uint32_t term[TYPES];
          term[0] = entry(sign_tab, sat, nb);
          EOQ_SFOR(p, BITS - 1, term[1 << p] = term[0] & entry(mask_tab, mat[p], nb););
          EOQ_SFOR(M, TYPES,
            if constexpr ((M & (M - 1)) != 0) term[M] = term[M & -M] & term[M ^ (M & -M)];
          );
          EOQ_SFOR(i, TYPES / 4,
            const v4i B = {(int)term[4 * i], (int)term[4 * i + 1], (int)term[4 * i + 2], (int)term[4 * i + 3]};
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Aq[(8 * wq + nb) * (TYPES / 4) + i], B, acc, 0, 0, 0);
          );
        );
      );
    }
    // ---- the planes of a head meet in the lane: registers 4 qq .. 4 qq + 3 are head 2 qq + hf; planes 0-1 and 2-3
    // are joined exactly in int32 (|register| < 2^18), the halves in float32 ----
    const float rho = half_bits_to_float((uint16_t)cur.rho);
    float res[NQ];
#pragma unroll
    for (int qq = 0; qq < NQ; ++qq) {
      const int lo = acc[4 * qq] + (acc[4 * qq + 1] << 8), hi = acc[4 * qq + 2] + (acc[4 * qq + 3] << 8);
      res[qq] = fmaf((float)hi, 65536.0f, (float)lo) * (Kq[qq] * rho);
    }
    if constexpr (QJL) {
      // sign(Phi r_x) is one more plane of +-1: in the table of pairs the first entry kind with the magnitude nibble at zero
      v16i ac2;
#pragma unroll
      for (int v = 0; v < 16; ++v) ac2[v] = 0;
      if constexpr (PAIRS) {
        EOQ_SFOR(i, 4,
          const uint32_t sw = cur.sg[0][i >> 1] >> (16 * (i & 1));
          const v4i B = {(int)nib_tab[sw & 0xFu].x, (int)nib_tab[(sw >> 4) & 0xFu].x, (int)nib_tab[(sw >> 8) & 0xFu].x, (int)nib_tab[(sw >> 12) & 0xFu].x};
          ac2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Ap[i], B, ac2, 0, 0, 0);
        );
      } else {
        EOQ_SFOR(wq, 2,
          uint32_t sat[2];
          places(cur.sg[0][wq], sat);
          EOQ_SFOR(i, 2,
            v4i B;
            EOQ_SFOR(e, 4, B[e] = (int)entry(sign_tab, sat, 4 * i + e););
            ac2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Ap[2 * wq + i], B, ac2, 0, 0, 0);
          );
        );
      }
      const float gam = half_bits_to_float((uint16_t)cur.gam[0]);
#pragma unroll
      for (int qq = 0; qq < NQ; ++qq) {
        const int lo = ac2[4 * qq] + (ac2[4 * qq + 1] << 8), hi = ac2[4 * qq + 2] + (ac2[4 * qq + 3] << 8);
        res[qq] = fmaf(fmaf((float)hi, 65536.0f, (float)lo), Kp[qq] * gam, res[qq]);
      }
    }
    // ---- low-rank term sum_i C[i][token] w[i][head] on the f16 matrix cores: the coefficients change lanes through the
    // wave's LDS tile (one wave's LDS operations complete in order) ----
    if (r > 0) {   // uniform
      *reinterpret_cast<u32x4*>(cs + (lane >> 2) * CTLD + (lane & 3) * 8) = cur.cf;
      __builtin_amdgcn_wave_barrier();
      float16v lr;
#pragma unroll
      for (int v = 0; v < 16; ++v) lr[v] = 0.0f;
      lr = __builtin_amdgcn_mfma_f32_32x32x16_f16(Aw.h, c_operand(0).h, lr, 0, 0, 0);
      if (r > 16) {
        // components 16 .. 31 (rare): fetched and prepared here, nothing of them is kept
        const u32x4 c2 = __builtin_amdgcn_raw_buffer_load_b128(coef_buffer(b), vo_cf + (uint32_t)(16 * n * 2), (tok - b * n) * 2, 0);
        *reinterpret_cast<u32x4*>(cs + (16 + (lane >> 2)) * CTLD + (lane & 3) * 8) = c2;
        __builtin_amdgcn_wave_barrier();
        lr = __builtin_amdgcn_mfma_f32_32x32x16_f16(w_operand(b, 1).h, c_operand(1).h, lr, 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();   // the tile is rewritten by the next one
#pragma unroll
      for (int qq = 0; qq < NQ; ++qq) res[qq] += lr[4 * qq] + lr[4 * qq + 1];
    }
    // head 2 qq + hf of the group: lanes of a head that the group does not have aim behind the descriptor
#pragma unroll
    for (int qq = 0; qq < NQ; ++qq) {
      const bool live = 2 * qq + hf < group;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(res[qq]), bout, live ? vo_out : 0xFFFFFFF0u,
                                            (int)((2 * qq * T + tok) * 4), 0);
    }
  };

  // Two register sets in turn: the next tile is on its way while this one is worked on.  The loop body has no branch
  // around a memory instruction (a wait can then name exactly the loads it needs): behind the wave's last tile a
  // request fetches that tile once more.  The last tile of an odd number has a body of its own.  (With a pass that stored
  // nothing there, runs of five steps took as long as runs of six; with an exit in the middle of the loop its trip count and
  // its addresses passed through vector registers, 90 vector instructions a tile instead of 82 at 2 bits: 8 heads x 23 blocks
  // of 128 5.88 us where it is 5.78, 8 heads x 64 blocks of 512 with the correction 13.8 and 13.7.)
  int tok_w = tok0 + 32 * wave, b_w = 0, end_w = n, r_w = rank_of(0);   // next tile to work on
#define EOQ_SC_WORK(F)                       \
  if (tok_w >= end_w) {                      \
    ++b_w;                                   \
    end_w += n;                              \
    r_w = rank_of(b_w);                      \
  }                                          \
  work(F, tok_w, b_w, r_w);                  \
  tok_w += QUAD;
#pragma unroll 1
  for (int it = 1; it < count; it += 2) {
    EOQ_SC_REQUEST(f1)
    EOQ_SC_WORK(f0)
    EOQ_SC_REQUEST(f0)
    EOQ_SC_WORK(f1)
  }
  if (count & 1) {   // uniform
    EOQ_SC_WORK(f0)
  }
#undef EOQ_SC_REQUEST
#undef EOQ_SC_WORK
}

}  // namespace

constexpr int64_t GRID_Y = 65535;
struct ScoresGrid {
  int64_t x, y, run_heads;   // workgroups (x, y): run x of head y below row run_heads, behind it the tail's in turn
};
// The launches for `runs` runs and `tail_groups` workgroups of the tail of each of `heads` heads: one, or two where the rows of a
// grid do not suffice.  The runs come first: workgroups go to the eight XCDs in turn, and with each head's tail behind its
// runs the runs of all heads met on one XCD in eight, four or two wherever runs and tail of a head were together a multiple of
// eight and so on (128 heads, 23 blocks of 256 and 255 tokens, 4 bits: 2 runs and 4 tail workgroups a head 57 us, 4 and 4 65).
extern "C" int eoq_scores_grids(int64_t heads, int64_t runs, int64_t tail_groups, ScoresGrid* out) {
  const int64_t rows = runs > 0 ? (heads * tail_groups + runs - 1) / runs : 0;
  if (runs > 0 && heads + rows <= GRID_Y) {
    out[0] = {runs, heads + rows, heads};
    return 1;
  }
  int k = 0;
  if (runs > 0) out[k++] = {runs, heads, heads};
  if (tail_groups > 0) out[k++] = {tail_groups, heads, 0};
  return k;
}

namespace {

template <int BITS>
const void* scores_kernel(bool qjl, bool wide) {
  if (qjl) return wide ? (const void*)eoq_scores_i8_kernel<BITS, true, 4> : (const void*)eoq_scores_i8_kernel<BITS, true, 2>;
  return wide ? (const void*)eoq_scores_i8_kernel<BITS, false, 4> : (const void*)eoq_scores_i8_kernel<BITS, false, 2>;
}

hipError_t launch_scores_impl(const EoqLaunch& L, eoq_packed keys, const eoq_qjl* qjl, int64_t n_seq, int n_kv_heads,
                              int64_t blocks_per_head, const void* q_fp16, int n_q_heads, float* scores,
                              int64_t block_capacity, int64_t score_stride, const void* tail_fp16,
                              int64_t tail_capacity, int tail_len) {
  const int64_t sg_total = n_seq * n_kv_heads;
  if (block_capacity <= 0) block_capacity = blocks_per_head;
  if (score_stride <= 0) score_stride = blocks_per_head * L.n;
  if (L.ev) (void)hipEventRecord(L.ev[6], L.stream);
  const int64_t tail_groups = (tail_len + TAIL_TOK - 1) / TAIL_TOK;
  const int group = n_q_heads / n_kv_heads;
  const int64_t spb = L.n / QUAD, steps = blocks_per_head * spb;
  const int64_t run = eoq_scores_run(L.bits, L.score_places[qjl ? 1 : 0][group <= 4 ? 0 : 1], L.units, sg_total, steps, spb, sg_total * tail_groups);
  const int64_t runs = (steps + run - 1) / run;
  if (sg_total > GRID_Y || runs + tail_groups > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 block(THREADS);
  const uint16_t* q = static_cast<const uint16_t*>(q_fp16);
#define EOQ_SCORES_ARGS                                                                                              \
  dim3((unsigned)G.x, (unsigned)G.y), block, 0, L.stream, L.n, L.r_max, n_kv_heads, group, blocks_per_head, block_capacity, score_stride, (int)run, \
      L.pih, L.tab, keys.codes, keys.norms, keys.rank, keys.lfac, keys.rfac, q, scores
#define EOQ_SCORES(BITS, NQ)                                                                                         \
  do {                                                                                                               \
    if (qjl)                                                                                                         \
      hipLaunchKernelGGL((eoq_scores_i8_kernel<BITS, true, NQ>), EOQ_SCORES_ARGS, L.phih, qjl->signs, qjl->norms,  \
                         (int)G.run_heads, (const uint16_t*)nullptr, (int64_t)0, 0, (int)sg_total);                  \
    else                                                                                                             \
      hipLaunchKernelGGL((eoq_scores_i8_kernel<BITS, false, NQ>), EOQ_SCORES_ARGS, (const uint16_t*)nullptr,      \
                         (const uint8_t*)nullptr, (const uint16_t*)nullptr, (int)G.run_heads,                       \
                         static_cast<const uint16_t*>(tail_fp16), tail_capacity, tail_len, (int)sg_total);           \
  } while (0)
#define EOQ_SCORES_BITS(NQ)                 \
  switch (L.bits) {                         \
    case 1: EOQ_SCORES(1, NQ); break;    \
    case 2: EOQ_SCORES(2, NQ); break;    \
    case 3: EOQ_SCORES(3, NQ); break;    \
    default: EOQ_SCORES(4, NQ); break;   \
  }
  ScoresGrid grids[2];
  const int launches = eoq_scores_grids(sg_total, runs, tail_groups, grids);
  for (int i = 0; i < launches; ++i) {
    const ScoresGrid& G = grids[i];
    if (group <= 4) {
      EOQ_SCORES_BITS(2)
    } else {
      EOQ_SCORES_BITS(4)
    }
  }
#undef EOQ_SCORES_BITS
#undef EOQ_SCORES
#undef EOQ_SCORES_ARGS
  if (L.ev) (void)hipEventRecord(L.ev[7], L.stream);
  return hipGetLastError();
}

}  // namespace

// Steps of 128 tokens (a tile for each of the four waves) that a workgroup takes, for `heads` (sequence, KV head) pairs of `steps`
// steps each in blocks of `steps_per_block`, beside `tails` workgroups of the tail, on a device of `units` compute units that
// holds `places` workgroups of the kernel.  A second, partly filled round of workgroups costs a set-up and a run, so the grid has
// no more than w workgroups for each unit, w up to what a unit holds (more where heads of up to 16 blocks each are more than
// that); the tail's workgroups are among them, or, a layer of one to each unit at a time, beside them, where a layer costs what
// a set-up does (8 heads x 23 blocks of 512 and 171 tokens, 24 workgroups of the tail, 2 bits: 7.5 us with 184 runs and 9.4 with
// 248; 128 heads x 5 blocks of 1024 and 342 tokens, 768 of the tail, 1 bit: 17.8 with 512 runs and 27.6 with 256).  The unit that
// has w of them decides.  Calls of one head with exactly w workgroups of `run` steps to a unit take, within 8 % from four steps on,
//   (run (w + 2.2) + s w) e + 4 us,  e = 0.13, 0.19, 0.35, 0.51 us and s = 15, 11, 6, 6 at 1 .. 4 bits
// (with the correction e = 0.26, 0.60 and s = 12, 7 at 2 and 4): the waves of a unit work their steps off side by side, their
// set-ups pass one behind the other.  The w with the least of it, in fifths, with s = 12 up to 2 bits and 6 above.  Against as
// many workgroups as there are places wherever that leaves six steps to a run, else as few as it takes for six (us before and
// now): 24 heads x 64 blocks of 512, 2 bits 20.0, 18.5 (3 of 8 steps to a unit, not 4 of 7); 8 x 64 of 1024, 1 bit 13.4, 11.8 (2
// of 8, not 3 of 6); 8 x 64 of 512, 3 bits 16.6, 15.6 (2 of 4, not 1 of 8).  Whole blocks are too coarse a measure: 12 x 204
// steps on 512 places at 4 bits 28 us with runs of two blocks (8 steps), 24 with 6.
extern "C" int64_t eoq_scores_run(int bits, int64_t places, int64_t units, int64_t heads, int64_t steps, int64_t steps_per_block,
                                  int64_t tails) {
  const int64_t most = SC_RUN_MAX * steps_per_block, setup = bits <= 2 ? 12 : 6;
  const int64_t layers = (tails + units - 1) / units;   // of one tail workgroup to a unit
  int64_t run = most, least = INT64_MAX;
  for (int64_t w = places / units; w >= 1; --w) {
    for (int64_t beside = 0; beside <= layers && beside <= 4; ++beside) {
      const int64_t among = (beside < 4 && tails > beside * units) ? tails - beside * units : 0;
      const int64_t per_head = (w * units - among) / heads;
      if (w * units - among < heads) continue;
      int64_t r = (steps + per_head - 1) / per_head;                             // the shortest run that does not exceed the grid
      if (r > most) continue;                                                    // more than one round
      r = r < 1 ? 1 : r;                                                         // no block at all: the tail's workgroups only
      if (r % steps_per_block != 0 && r > most - steps_per_block + 1) r = most;  // begun inside a block it touches one block more
      const int64_t cost = r * (5 * w + 11) + 5 * setup * (w + beside);
      if (cost < least) {
        least = cost;
        run = r;
      }
    }
  }
  return run;
}

// Workgroups of the kernel for `bits` that the current device holds at a time, by the compiled kernel's own registers and LDS
// (a table of numbers beside the kernels was wrong at 4 bits with the correction, one per unit where two fit: 2048 blocks of
// 512 for groups of three 57 us, now 49; 512 blocks for groups of four 21 either way).
extern "C" int eoq_scores_places(int bits, int corrected, int group) {
  const bool qjl = corrected != 0, wide = group > 4;
  const void* f = bits == 1 ? scores_kernel<1>(qjl, wide) : (bits == 2 ? scores_kernel<2>(qjl, wide) : (bits == 3 ? scores_kernel<3>(qjl, wide) : scores_kernel<4>(qjl, wide)));
  int device = 0, units = 0, per_unit = 0;
  if (hipGetDevice(&device) != hipSuccess || hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_unit, f, THREADS, 0) != hipSuccess)
    return 0;
  return units * per_unit;
}

hipError_t eoq_launch_scores(const EoqLaunch& L, eoq_packed keys, int64_t n_seq, int n_kv_heads,
                             int64_t blocks_per_head, const void* q_fp16, int n_q_heads, float* scores,
                             int64_t block_capacity, int64_t score_stride, const void* tail_fp16,
                             int64_t tail_capacity, int tail_len) {
  return launch_scores_impl(L, keys, nullptr, n_seq, n_kv_heads, blocks_per_head, q_fp16, n_q_heads, scores,
                            block_capacity, score_stride, tail_fp16, tail_capacity, tail_len);
}

hipError_t eoq_launch_scores_prod(const EoqLaunch& L, eoq_packed keys, eoq_qjl qjl, int64_t n_seq, int n_kv_heads,
                                  int64_t blocks_per_head, const void* q_fp16, int n_q_heads, float* scores) {
  return launch_scores_impl(L, keys, &qjl, n_seq, n_kv_heads, blocks_per_head, q_fp16, n_q_heads, scores, 0, 0, nullptr,
                            0, 0);
}
