// The normalisation layer in front of a quantized linear layer with the channel reorder absorbed
// into it (paper App. C): RMSNorm, or LayerNorm followed by a per-sample scale and shift, emitting
// y_P[m, j] = y[m, pi(j)] as a bf16 tensor, as the activation operand of the GEMM (the dynamic
// quantizer of Eq. 1-2 applied to those bf16 values), or both.
//
// One wave, or the two or four waves of a workgroup, own one token row from load to store:
//   1. the row is read as it lies in memory (16 bytes per lane and access, whole lines) and stays in
//      registers; its sum and sum of squares come from v_dot2c_f32_bf16 on the packed pairs;
//   2. it is normalised, the channel-wise vectors -- read as they lie too -- are applied, and the values,
//      rounded to bf16, go into the row's slab of LDS in their own order.  All of that is element-wise,
//      so it need not wait for the reorder: no vector is ever gathered, and a row of any sample takes
//      its own sample's vectors;
//   3. lane l then produces chunks l, l + 64, ... (8 consecutive positions j each) of the reordered row:
//      it loads pi(j) for its positions, gathers y[pi(j)] from the slab with 2-byte LDS reads -- where
//      the paper's kernel issues indexed global loads -- and the chunk is stored (consecutive lanes,
//      consecutive 16 bytes) and / or quantized: a group of G positions is G / 8 consecutive lanes, so
//      the group maximum is a lane reduction and the per-row power of two of the INT operand layout a
//      reduction over the row's waves.
// What bounds it: few rows the chain of loads, sums, LDS and gathers (RMSNorm + NVFP4, 512 x 3072: 4.5 us; 6.3 when each
// workgroup first reordered the vectors into LDS), many rows the vector unit beside the traffic: modulated LayerNorm +
// NVFP4, 4608 x 3072, 36 MB: 14.7 us (20.4 before), RMSNorm 13.4 (16.3).
//
// The same skeleton runs the Hadamard variant (paper App. D, x H P): steps 1 and 2 become a fast
// Hadamard transform of the row in the slab (fp32), step 3 reads the transformed row at pi(j) -- the
// reorder is the order in which the transform's output is consumed.
#include <math.h>

#include <algorithm>

#include "pq_qgemm_common.h"

namespace pq {

namespace {

enum Norm : int { kNormRms = 0, kNormAdaLn = 1, kHadamard = 2 };
constexpr int kFmtNone = -1;                  // normalise and reorder only, no quantization
constexpr int kNormMaxWaves = 8;

struct NormArgs {
  const int32_t* perm;          // pi, or null for the identity
  const uint16_t* gamma;        // RMSNorm: bf16 [K], or null for ones
  const uint16_t* mod_scale;    // AdaLN: bf16 [n_mod][K] s (the factor is 1 + s), or null for zeros
  const uint16_t* mod_shift;    // AdaLN: bf16 [n_mod][K] b, or null for zeros
  int64_t rows_per_mod;         // token row m uses modulation row m / rows_per_mod
  float eps;
  uint16_t* y;                  // bf16 [rows][ldy] normalised, reordered output, or null
  int64_t ldy;
  int had_pow2, had_m;          // Hadamard: K = had_pow2 * had_m, had_m in {1, 12, 20}
  float had_scale;              // 1 / sqrt(K)
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// the sum over the wave, in every lane: halves, rows of 16 lanes, then inside a row by DPP rotations and quad permutes (the
// values are equal in lanes 8 apart when lanes 4 apart meet, so the rotation gives the partner's)
__device__ __forceinline__ float wave_sum_f32(float v) {
  const auto h = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
  v = as_f32(h[0]) + as_f32(h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
  v = as_f32(r[0]) + as_f32(r[1]);
  v += dpp_f32<0x128>(v);                                    // row_ror:8
  v += dpp_f32<0x124>(v);                                    // row_ror:4
  v += dpp_f32<0x4E>(v);                                     // quad_perm [2,3,0,1]
  return v + dpp_f32<0xB1>(v);                               // quad_perm [1,0,3,2]
}

__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){lo, hi}, bf16x2_t));
}

struct Idx8 {
  int4 lo, hi;
};


// ---- fast Hadamard transform of one row held in LDS as fp32, by one wave -------------------
// H = S_{2^k} (x) P_m / sqrt(K), channel i = a * m + b (a: Sylvester index, natural order; b: Paley
// index).  Kronecker factors act on separate index digits, so the transform is a sequence of
// passes, each applying a small matrix along one digit: every lane takes whole fibres (all elements
// that differ only in that digit), transforms them in registers and writes them back.

// between passes: the wave's LDS writes are complete and visible to its other lanes
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A row is worked on by a team of TEAM waves: one wave, which only has to order its own LDS
// traffic, or (wide rows) all waves of the workgroup, which meet at a workgroup barrier.
template <int TEAM>
__device__ __forceinline__ void team_sync() {
  if constexpr (TEAM == 1) wave_lds_sync();
  else __syncthreads();
}

// Sylvester matrix of order R along a digit of weight `inner` elements; n_fibres = K / R
template <int R, int TEAM>
__device__ __forceinline__ void sylvester_pass(float* slab, int inner, int n_fibres, int lane) {
  // f / inner through a float reciprocal: f < 2^13 and the quotient's fractional part is at least
  // 1 / (2 inner) away from an integer, far more than the rounding error of the product
  const float inv_inner = 1.0f / (float)inner;
  for (int f = lane; f < n_fibres; f += 64 * TEAM) {
    const int hi = (int)(((float)f + 0.5f) * inv_inner), lo = f - hi * inner;
    float* base = slab + hi * (R * inner) + lo;
    float v[R];
#pragma unroll
    for (int t = 0; t < R; ++t) v[t] = base[t * inner];
#pragma unroll
    for (int h = 1; h < R; h <<= 1)
#pragma unroll
      for (int i = 0; i < R; i += 2 * h)
#pragma unroll
        for (int j = i; j < i + h; ++j) {
          const float a = v[j], b = v[j + h];
          v[j] = a + b;
          v[j + h] = a - b;
        }
#pragma unroll
    for (int t = 0; t < R; ++t) base[t * inner] = v[t];
  }
  team_sync<TEAM>();
}

// quadratic character mod Q (Q prime): +1 for a non-zero square, -1 otherwise, 0 for 0
template <int Q>
__host__ __device__ constexpr int legendre(int r) {
  r = ((r % Q) + Q) % Q;
  if (r == 0) return 0;
  for (int t = 1; t < Q; ++t)
    if ((t * t) % Q == r) return 1;
  return -1;
}

// entry (b, b2) of the Paley type I Hadamard matrix of order M = Q + 1:  I + [[0, 1^T], [-1, chi(i - j)]]
template <int M>
__host__ __device__ constexpr int paley_entry(int b, int b2) {
  if (b == b2) return 1;
  if (b == 0) return 1;
  if (b2 == 0) return -1;
  return legendre<M - 1>((b - 1) - (b2 - 1));
}

// y[b2] = sum_b x[b] P[b][b2] along the last digit (M contiguous elements per fibre)
template <int M, int TEAM>
__device__ __forceinline__ void paley_pass(float* slab, int n_fibres, int lane) {
  for (int f = lane; f < n_fibres; f += 64 * TEAM) {
    float* base = slab + f * M;
    float v[M], o[M];
#pragma unroll
    for (int b = 0; b < M; ++b) v[b] = base[b];
    // a pair of inputs enters every output as +-(v0 + v1) or +-(v0 - v1): form both once, then each
    // output is a signed sum of M / 2 terms instead of M
    float sum[M / 2], dif[M / 2];
#pragma unroll
    for (int j = 0; j < M / 2; ++j) {
      sum[j] = v[2 * j] + v[2 * j + 1];
      dif[j] = v[2 * j] - v[2 * j + 1];
    }
#pragma unroll
    for (int b2 = 0; b2 < M; ++b2) {
      float acc = 0.0f;
#pragma unroll
      for (int j = 0; j < M / 2; ++j) {
        const int s0 = paley_entry<M>(2 * j, b2), s1 = paley_entry<M>(2 * j + 1, b2);
        const float term = s0 == s1 ? sum[j] : dif[j];
        acc = s0 > 0 ? acc + term : acc - term;
      }
      o[b2] = acc;
    }
#pragma unroll
    for (int b = 0; b < M; ++b) base[b] = o[b];
  }
  team_sync<TEAM>();
}

// The Paley pass of order 12 on the matrix unit, straight from the bf16 row in memory into the fp32 slab:
// sixteen fibres (16 x 12 contiguous values) times P_12 padded to 16 x 16 is one v_mfma_f32_16x16x16_bf16.
// Inputs and the +-1 entries are exact in bf16 and the products are accumulated in fp32, as on the
// vector unit.  Operand layout of the instruction: lane l holds A[l % 16][4 (l / 16) + i] (a fibre's
// values 4j .. 4j + 3: eight contiguous bytes), B[4 (l / 16) + i][l % 16] and D[4 (l / 16) + i][l % 16].
// negative entries of rows 4j .. 4j + 3 of P_12: bit 16 i + n for entry (4j + i, n)
constexpr uint64_t paley12_negatives(int j) {
  uint64_t mask = 0;
  for (int i = 0; i < 4; ++i)
    for (int n = 0; n < 12; ++n)
      if (paley_entry<12>(4 * j + i, n) < 0) mask |= (uint64_t)1 << (16 * i + n);
  return mask;
}
template <int TEAM>
__device__ __forceinline__ void paley12_pass_from_memory(const uint16_t* __restrict__ xr, float* slab, int n_fibres,
                                                         int tl) {
  typedef short bf16x4_bits __attribute__((ext_vector_type(4)));
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int lane = tl & 63, wv = tl >> 6;
  const int n = lane & 15, j = lane >> 4;
  constexpr uint64_t kNeg0 = paley12_negatives(0), kNeg1 = paley12_negatives(1), kNeg2 = paley12_negatives(2);
  const uint64_t neg = j == 0 ? kNeg0 : j == 1 ? kNeg1 : kNeg2;
  const bool in_matrix = j < 3 && n < 12;                    // the padding rows and columns are zero
  uint32_t bw[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t e0 = ((neg >> (32 * h + n)) & 1) ? 0xBF80u : 0x3F80u;
    const uint32_t e1 = ((neg >> (32 * h + 16 + n)) & 1) ? 0xBF80u : 0x3F80u;
    bw[h] = in_matrix ? (e0 | (e1 << 16)) : 0u;
  }
  const bf16x4_bits b = __builtin_bit_cast(bf16x4_bits, make_uint2(bw[0], bw[1]));
  const int groups = n_fibres / 16;
  constexpr int kInFlight = 8;
  for (int g0 = wv; g0 < groups; g0 += TEAM * kInFlight) {
    uint2 a[kInFlight];
#pragma unroll
    for (int t = 0; t < kInFlight; ++t) {
      const int g = g0 + t * TEAM;
      a[t] = make_uint2(0u, 0u);
      if (g < groups && j < 3) a[t] = *reinterpret_cast<const uint2*>(xr + (size_t)(g * 16 + n) * 12 + 4 * j);
    }
#pragma unroll
    for (int t = 0; t < kInFlight; ++t) {
      const int g = g0 + t * TEAM;
      if (g >= groups) break;                                // wave-uniform
      const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4_bits, a[t]), b,
                                                                (f32x4){0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
      if (n < 12) {
        float* out = slab + (size_t)(g * 16 + 4 * j) * 12 + n;
        out[0] = d[0];
        out[12] = d[1];
        out[24] = d[2];
        out[36] = d[3];
      }
    }
  }
  team_sync<TEAM>();
}

// `lane` is the thread's index inside its team (0 .. 64 TEAM - 1); paley_done: the Paley pass has been applied
template <int TEAM>
__device__ __forceinline__ void hadamard_row(float* slab, int K, int pow2, int m, int lane, bool paley_done = false) {
  if (m == 12 && !paley_done) paley_pass<12, TEAM>(slab, pow2, lane);
  if (m == 20) paley_pass<20, TEAM>(slab, pow2, lane);
  int inner = m;                       // weight of the current Sylvester digit, in elements
  int rem = pow2;
  while (rem >= 16) {
    sylvester_pass<16, TEAM>(slab, inner, K / 16, lane);
    inner *= 16;
    rem /= 16;
  }
  if (rem == 8) sylvester_pass<8, TEAM>(slab, inner, K / 8, lane);
  if (rem == 4) sylvester_pass<4, TEAM>(slab, inner, K / 4, lane);
  if (rem == 2) sylvester_pass<2, TEAM>(slab, inner, K / 2, lane);
}

constexpr int kHold = 6;        // chunks of a row that a thread holds between the statistics and the normalisation

// eight channels of the normalised row, rounded to bf16
template <bool ADA>
__device__ __forceinline__ uint4 normalised(const uint4& x, const uint4& g0, const uint4& g1, float rstd, float nmr) {
  uint32_t d[4] = {x.x, x.y, x.z, x.w};
  const uint32_t s[4] = {g0.x, g0.y, g0.z, g0.w};
  const uint32_t h[4] = {g1.x, g1.y, g1.z, g1.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo, hi;
    if constexpr (ADA) {
      const float l0 = fmaf(bf16_lo(d[e]), rstd, nmr), l1 = fmaf(bf16_hi(d[e]), rstd, nmr);
      lo = fmaf(bf16_lo(s[e]), l0, bf16_lo(h[e])) + l0;      // (1 + s) ln + b
      hi = fmaf(bf16_hi(s[e]), l1, bf16_hi(h[e])) + l1;
    } else {
      lo = (bf16_lo(d[e]) * rstd) * bf16_lo(s[e]);
      hi = (bf16_hi(d[e]) * rstd) * bf16_hi(s[e]);
    }
    d[e] = pack_bf16_rne(lo, hi);
  }
  return make_uint4(d[0], d[1], d[2], d[3]);
}

// sum / maximum over the team, the same value in every thread (fixed order of the waves); `red`: a word per wave
template <int TEAM, int N>
__device__ __forceinline__ void team_sums(float (&v)[N], float* red, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_sum_f32(v[i]);
  if constexpr (TEAM > 1) {
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) red[wave * N + i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
      v[i] = 0.0f;
#pragma unroll
      for (int w = 0; w < TEAM; ++w) v[i] += red[w * N + i];
    }
    __syncthreads();
  }
}
template <int TEAM, int N>
__device__ __forceinline__ void team_maxima(float (&v)[N], float* red, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_max(v[i]);
  if constexpr (TEAM > 1) {
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) red[wave * N + i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
      v[i] = 0.0f;
#pragma unroll
      for (int w = 0; w < TEAM; ++w) v[i] = fmaxf(v[i], red[w * N + i]);
    }
    __syncthreads();
  }
}

constexpr int kBatch = 3;                                    // chunks whose indices and gathers a thread has in flight

// indices pi(j) of chunk c (clamped to an existing chunk: the address is always valid)
__device__ __forceinline__ Idx8 load_idx(const int32_t* __restrict__ perm, int c, int k_chunks) {
  const int cc = min(c, k_chunks - 1);
  Idx8 ix;
  if (perm) {
    ix.lo = *reinterpret_cast<const int4*>(perm + (size_t)cc * 8);
    ix.hi = *reinterpret_cast<const int4*>(perm + (size_t)cc * 8 + 4);
  } else {
    ix.lo = make_int4(cc * 8, cc * 8 + 1, cc * 8 + 2, cc * 8 + 3);
    ix.hi = make_int4(cc * 8 + 4, cc * 8 + 5, cc * 8 + 6, cc * 8 + 7);
  }
  return ix;
}

// What a team's second half needs: the outputs, the sizes and the team's place
struct Emit {
  int64_t rows, row;            // all rows; the team's
  int k_chunks, n_chunks;       // chunks that exist; chunks the panel holds (a half step past K included)
  int n_units;
  uint8_t* codes;
  uint16_t* scales;
  float* mul;
  uint16_t* y;                  // or null
  int64_t ldy;
  float T, encT, scale;         // NVFP4; the factor of an fp32 slab
  float* h_lds;                 // INT: n_units group maxima
  float* red;
  int wave, lane, tl;
};

// Chunks tl, tl + 64 TEAM, ... (8 positions j each) of the reordered row: the values at pi(j) are read from the slab (bf16,
// or fp32 to be scaled and rounded), stored and / or quantized.
template <int FMT, int G, int TEAM, bool F32>
__device__ __forceinline__ void emit_row(const void* slab, const int32_t* __restrict__ perm, Idx8 (&ix_cur)[kBatch],
                                          const Emit& em) {
  constexpr bool QUANT = FMT != kFmtNone;
  constexpr bool IS_INT = FMT == kInt4 || FMT == kInt3;
  constexpr int LPG = G / 8;                                 // lanes that share a group
  constexpr int TL = 64 * TEAM;
  static_assert(LPG >= 1 && LPG <= 64, "a group lies inside one wave-wide run of chunks");
  const int n_iter = (em.n_chunks + TL - 1) / TL;
  float row_max[1] = {0.0f};
  for (int it0 = 0; it0 < n_iter; it0 += kBatch) {
    // next batch's indices while this one is worked on
    Idx8 ix_next[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix_next[q] = load_idx(perm, em.tl + TL * (it0 + kBatch + q), em.k_chunks);
    // gathers of the whole batch in flight together
    uint32_t got[kBatch][8];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      if (it0 + q >= n_iter) break;                          // wave-uniform
      const int idx[8] = {ix_cur[q].lo.x, ix_cur[q].lo.y, ix_cur[q].lo.z, ix_cur[q].lo.w,
                          ix_cur[q].hi.x, ix_cur[q].hi.y, ix_cur[q].hi.z, ix_cur[q].hi.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (F32) got[q][e] = as_u32(static_cast<const float*>(slab)[idx[e]]);
        else got[q][e] = static_cast<const uint16_t*>(slab)[idx[e]];
      }
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      const int c = em.tl + TL * (it0 + q);
      if (it0 + q >= n_iter) break;                          // wave-uniform
      const bool in_row = c < em.k_chunks;
      uint4 yb;                                              // eight bf16 values
      if constexpr (F32) {
        float yv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) yv[e] = as_f32(got[q][e]) * em.scale;
        yb = make_uint4(pack_bf16_rne(yv[0], yv[1]), pack_bf16_rne(yv[2], yv[3]), pack_bf16_rne(yv[4], yv[5]),
                        pack_bf16_rne(yv[6], yv[7]));
      } else {
        yb = make_uint4(got[q][0] | (got[q][1] << 16), got[q][2] | (got[q][3] << 16), got[q][4] | (got[q][5] << 16),
                        got[q][6] | (got[q][7] << 16));
      }
      if (!in_row) yb = make_uint4(0u, 0u, 0u, 0u);          // the half step past K holds zeros
      if (em.y && in_row) *reinterpret_cast<uint4*>(em.y + em.row * em.ldy + (size_t)c * 8) = yb;

      if constexpr (QUANT) {
        // the quantizer of pq_quantize.hip on the rounded values
        const float v[8] = {bf16_lo(yb.x), bf16_hi(yb.x), bf16_lo(yb.y), bf16_hi(yb.y),
                            bf16_lo(yb.z), bf16_hi(yb.z), bf16_lo(yb.w), bf16_hi(yb.w)};
        float a = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) a = fmaxf(a, fabsf(v[j]));
        a = group_max<LPG>(a);
        uint32_t codes;
        if constexpr (FMT == kNvfp4) {
          const Nv4Scale sc = nv4_scale(a, em.T, em.encT);
          codes = 0;
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, v[0] * sc.inv, v[1] * sc.inv, 1.0f, 0);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, v[2] * sc.inv, v[3] * sc.inv, 1.0f, 1);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, v[4] * sc.inv, v[5] * sc.inv, 1.0f, 2);
          codes = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(codes, v[6] * sc.inv, v[7] * sc.inv, 1.0f, 3);
          // a scale unit is the two bytes of 32 positions = four lanes; the first lane of the quad
          // collects the byte of the second pair
          const uint32_t other = dpp_u32<0x4E>(sc.byte);       // lane ^ 2
          const int u = c >> 2;
          if ((em.lane & 3) == 0 && u < em.n_units)
            em.scales[(int64_t)u * em.rows + em.row] = (uint16_t)(sc.byte | (other << 8));
        } else {
          constexpr int FI = IS_INT ? FMT : kInt4;
          const IntScale sc = int_scale<FI>(a);
          codes = int_codes8(v, sc.inv);
          row_max[0] = fmaxf(row_max[0], a);
          const int g = c / LPG;
          if (em.lane % LPG == 0 && g < em.n_units) em.h_lds[g] = a;
        }
        if (c < em.n_chunks)
          *reinterpret_cast<uint32_t*>(em.codes + ((int64_t)(c >> 3) * em.rows + em.row) * 32 + (c & 7) * 4) = codes;
      }
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix_cur[q] = ix_next[q];
  }

  if constexpr (IS_INT) {
    // the per-row power of two of the operand layout: E = exponent(row maximum) - 10 puts the
    // largest group maximum in [2^10, 2^11) (see pack_operand_kernel); scale units are the fp16
    // group maxima times 2^-E, the row factor 2^E / Q
    constexpr float Q = qmax_of(FMT);
    team_maxima<TEAM>(row_max, em.red, em.wave, em.lane);      // (with TEAM > 1 also the barrier after the h_lds writes)
    int e = (int)((as_u32(row_max[0]) >> 23) & 0xFF) - 127;
    if (row_max[0] == 0.0f) e = 0;
    const int E = max(-120, min(120, e - 10));
    const float down = as_f32((uint32_t)(127 - E) << 23);
    if (em.tl == 0) em.mul[em.row] = as_f32((uint32_t)(127 + E) << 23) / Q;
    for (int u = em.tl; u < em.n_units; u += TL) {             // the team's own LDS writes, ordered above
      const _Float16 hn = (_Float16)(em.h_lds[u] * down);
      em.scales[(int64_t)u * em.rows + em.row] = __builtin_bit_cast(uint16_t, hn);
    }
  }
}

// Workgroups go round the eight chiplets in turn: the row block that gives each chiplet a contiguous run of them, so that
// the lines that neighbouring rows share (32 bytes of codes and 2 of a scale unit a row) meet in one L2 (RMSNorm + NVFP4
// 2048 x 6144 14.6 -> 10.7 us, 4608 x 3072 15.7 -> 13.4)
__device__ __forceinline__ int64_t block_by_chiplet(int b, int n) {
  const int per = n >> 3, extra = n & 7, chiplet = b & 7;
  return (int64_t)chiplet * per + min(chiplet, extra) + (b >> 3);
}

template <int FMT, int G, int NORM, int TEAM>
__global__ __launch_bounds__(64 * kNormMaxWaves) void norm_rows_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t K, int64_t ld, const float* __restrict__ tensor_scale,
    int64_t steps, int64_t units, uint8_t* __restrict__ p_codes, uint16_t* __restrict__ p_scales,
    float* __restrict__ p_mul, NormArgs na) {
  constexpr bool IS_INT = FMT == kInt4 || FMT == kInt3;
  // dynamic LDS: [per team: K bf16 (Hadamard: fp32) slab] [per team, INT: `units` fp32 group maxima]
  //              [per wave: 4 floats for team reductions]
  // TEAM == 1: every wave owns a row.  TEAM > 1: the workgroup is one team of TEAM waves and owns one row.
  constexpr int TL = 64 * TEAM;                              // threads of a team
  constexpr int kSlabBytes = NORM == kHadamard ? 4 : 2;      // per channel
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, n_waves = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tl = TEAM == 1 ? lane : tid;                     // index inside the team
  const int slot = TEAM == 1 ? wave : 0;                     // the team's place inside the workgroup
  const int teams = TEAM == 1 ? n_waves : 1;
  const int Ki = (int)K;
  const int k_chunks = Ki / 8;
  const int n_units = (int)units;
  const int64_t row = block_by_chiplet(blockIdx.x, gridDim.x) * teams + slot;
  if (TEAM == 1 && row >= rows) return;                      // wave-uniform; a team stays together to the end

  unsigned char* slab = lds_raw + (size_t)slot * Ki * kSlabBytes;
  float* h_all = reinterpret_cast<float*>(lds_raw + (size_t)teams * Ki * kSlabBytes);
  Emit em;
  em.rows = rows;
  em.row = row;
  em.k_chunks = k_chunks;
  em.n_chunks = (int)steps * 8;
  em.n_units = n_units;
  em.codes = p_codes;
  em.scales = p_scales;
  em.mul = p_mul;
  em.y = na.y;
  em.ldy = na.ldy;
  em.T = em.encT = em.scale = 0.0f;
  em.h_lds = h_all + (size_t)slot * n_units;
  em.red = h_all + (size_t)(IS_INT ? teams * n_units : 0);
  em.wave = wave;
  em.lane = lane;
  em.tl = tl;
  if constexpr (FMT == kNvfp4) {
    em.T = *tensor_scale;
    em.encT = nv4_enc_scale(em.T);
  }
  const uint16_t* xr = x + row * ld;

  if constexpr (NORM == kHadamard) {
    // ---- 1. the row as fp32 in the team's slab, transformed in place
    Idx8 ix[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix[q] = load_idx(na.perm, tl + TL * q, k_chunks);
    float* slab_f = reinterpret_cast<float*>(slab);
    constexpr int kInFlight = 8;
    const bool paley_on_mfma = na.had_m == 12 && na.had_pow2 >= 16;      // uniform
    if (paley_on_mfma) paley12_pass_from_memory<TEAM>(xr, slab_f, na.had_pow2, tl);
    for (int c0 = 0; c0 < (paley_on_mfma ? 0 : k_chunks); c0 += kInFlight * TL) {
      uint4 lines[kInFlight];
#pragma unroll
      for (int t = 0; t < kInFlight; ++t) {
        const int c = min(c0 + t * TL + tl, k_chunks - 1);
        lines[t] = *reinterpret_cast<const uint4*>(xr + (size_t)c * 8);
      }
#pragma unroll
      for (int t = 0; t < kInFlight; ++t) {
        const int c = c0 + t * TL + tl;
        if (c < k_chunks) {
          const uint4 p = lines[t];
          *reinterpret_cast<float4*>(slab_f + c * 8) = make_float4(bf16_lo(p.x), bf16_hi(p.x), bf16_lo(p.y), bf16_hi(p.y));
          *reinterpret_cast<float4*>(slab_f + c * 8 + 4) = make_float4(bf16_lo(p.z), bf16_hi(p.z), bf16_lo(p.w), bf16_hi(p.w));
        }
      }
    }
    team_sync<TEAM>();
    hadamard_row<TEAM>(slab_f, Ki, na.had_pow2, na.had_m, tl, paley_on_mfma);
    em.scale = na.had_scale;
    emit_row<FMT, G, TEAM, true>(slab, na.perm, ix, em);
  } else {
    constexpr bool ADA = NORM == kNormAdaLn;
    // ---- 1. the row as it lies (buffer loads: past its end they give zeros, which add nothing), a block of kHold chunks
    // a thread; the last block stays in registers, blocks before it (rows wider than kHold * 8 * TL) are parked in the
    // slab.  A chunk that no thread of the team has is skipped.
    const int n_blocks = (k_chunks + kHold * TL - 1) / (kHold * TL);
    const int last_turns = (k_chunks - (n_blocks - 1) * kHold * TL + TL - 1) / TL;     // chunks of the last block: 1 .. kHold
    const auto buffer = [&](const uint16_t* p) {
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, p ? Ki * 2 : 0, 0x00027000);
    };
    const auto chunk_of = [&](auto buf, int c) {
      return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(buf, c * 16, 0, 0));
    };
    uint4 lines[kHold];
    float st[ADA ? 2 : 1] = {};                              // sum of squares and (LayerNorm) sum
    const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3F803F80u);
    const auto xb = buffer(xr);
    uint4* parked = reinterpret_cast<uint4*>(slab);
    for (int b = 0; b < n_blocks; ++b) {
      const int c0 = b * kHold * TL + tl;
      const int turns = b + 1 < n_blocks ? kHold : last_turns;
#pragma unroll
      for (int t = 0; t < kHold; ++t)
        if (t < turns) lines[t] = chunk_of(xb, c0 + t * TL);
#pragma unroll
      for (int t = 0; t < kHold; ++t) {
        if (t >= turns) break;
        const uint32_t d[4] = {lines[t].x, lines[t].y, lines[t].z, lines[t].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf16x2_t v = __builtin_bit_cast(bf16x2_t, d[e]);
          if constexpr (ADA) st[1] = __builtin_amdgcn_fdot2_f32_bf16(v, ones, st[1], false);
          st[0] = __builtin_amdgcn_fdot2_f32_bf16(v, v, st[0], false);
        }
        if (b + 1 < n_blocks) parked[c0 + t * TL] = lines[t];
      }
    }
    // the channel-wise vectors of the last block and the first indices do not depend on the sums
    const uint16_t* vec0 = na.gamma;
    const uint16_t* vec1 = nullptr;
    if constexpr (ADA) {
      const int64_t mod = na.rows_per_mod >= rows ? 0 : row / na.rows_per_mod;
      vec0 = na.mod_scale ? na.mod_scale + mod * K : nullptr;
      vec1 = na.mod_shift ? na.mod_shift + mod * K : nullptr;
    }
    const auto b0 = buffer(vec0), b1 = buffer(vec1);
    constexpr int kVec = ADA ? kHold / 2 : kHold;            // chunks of the vectors held at a time
    uint4 g0[kVec], g1[kVec];
    const auto load_vectors = [&](int c0, int turns) {
#pragma unroll
      for (int t = 0; t < kVec; ++t) {
        if (t >= turns) break;
        g0[t] = chunk_of(b0, c0 + t * TL);
        if constexpr (ADA) g1[t] = chunk_of(b1, c0 + t * TL);
        else if (!vec0) g0[t] = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
      }
    };
    load_vectors((n_blocks - 1) * kHold * TL + tl, last_turns);
    Idx8 ix[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) ix[q] = load_idx(na.perm, tl + TL * q, k_chunks);

    team_sums<TEAM>(st, em.red, wave, lane);
    const float k_f = (float)Ki;
    float mean = 0.0f;
    if constexpr (ADA) {
      mean = st[1] / k_f;
      // variance = mean square - mean^2 loses accuracy when the mean dominates; then (rare, uniform
      // over the team) it is recomputed from the deviations
      const float mean_sq = st[0] / k_f;
      const float var = mean_sq - mean * mean;
      if (mean_sq > 16.0f * var) {
        float s3[1] = {0.0f};
        const auto add = [&](const uint4& p) {
          const uint32_t d[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = bf16_lo(d[e]) - mean, hi = bf16_hi(d[e]) - mean;
            s3[0] = fmaf(hi, hi, fmaf(lo, lo, s3[0]));
          }
        };
        const int c_last = (n_blocks - 1) * kHold * TL + tl;
        for (int c = tl; c < c_last; c += TL) add(parked[c]);
#pragma unroll
        for (int t = 0; t < kHold; ++t)
          if (c_last + t * TL < k_chunks) add(lines[t]);
        team_sums<TEAM>(s3, em.red, wave, lane);
        st[0] = s3[0];
      } else {
        st[0] = var * k_f;
      }
    }
    const float rstd = 1.0f / sqrtf(st[0] / k_f + na.eps);
    const float nmr = -mean * rstd;                          // LN(x) = x * rstd + nmr

    // ---- 2. normalised, the vectors applied, rounded to bf16, into the slab in the row's own order
    for (int b = n_blocks - 1; b >= 0; --b) {
      const int c0 = b * kHold * TL + tl;
      const int turns = b + 1 < n_blocks ? kHold : last_turns;
      if (b + 1 < n_blocks) {
#pragma unroll
        for (int t = 0; t < kHold; ++t) lines[t] = parked[c0 + t * TL];
        load_vectors(c0, kHold);
      }
#pragma unroll
      for (int h = 0; h < kHold; h += kVec) {
        if (h >= turns) break;
        if (h > 0) {
          asm volatile("" ::: "memory");                     // not earlier: the registers are those of the part before
          load_vectors(c0 + h * TL, turns - h);
        }
#pragma unroll
        for (int t = h; t < h + kVec; ++t) {
          if (t >= turns) break;
          const uint4 y = normalised<ADA>(lines[t], g0[t - h], g1[t - h], rstd, nmr);
          if (c0 + t * TL < k_chunks) parked[c0 + t * TL] = y;
        }
      }
    }
    team_sync<TEAM>();

    // ---- 3. gathered at pi(j), stored and / or quantized
    emit_row<FMT, G, TEAM, false>(slab, na.perm, ix, em);
  }
}

constexpr size_t kNormLdsLimit = 160 * 1024 - 1024;      // dynamic LDS a workgroup may ask for

size_t norm_lds_bytes(int norm, bool is_int, int teams, int n_waves, int64_t K, int64_t units) {
  const size_t tail = (is_int ? (size_t)teams * units * 4 : 0) + (size_t)n_waves * 16;
  return (size_t)teams * K * (norm == kHadamard ? 4 : 2) + tail;
}

// Waves (= rows) per workgroup: as many as still let the launch run in one round of resident
// workgroups, without leaving a tail of workgroups that start when the others are done.  How many workgroups of a given size a
// compute unit holds (registers, LDS, wave slots) is asked of the runtime.
template <typename Kern>
int hadamard_waves_per_group(Kern kern, bool is_int, int64_t rows, int64_t K, int64_t units) {
  int best = 1;
  double best_cost = 1e30;
  for (int w = 1; w <= kNormMaxWaves; ++w) {
    const size_t lds = norm_lds_bytes(kHadamard, is_int, w, w, K, units);
    if (lds > kNormLdsLimit) break;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * w, lds) != hipSuccess || per_cu < 1)
      per_cu = 1;
    const int64_t groups = (rows + w - 1) / w;
    const int64_t rounds = (groups + 256 * (int64_t)per_cu - 1) / (256 * (int64_t)per_cu);
    // time ~ rounds x (row work + a share of the workgroup's), in units of one row's work, plus what the rows that meet on
    // the busiest of the 256 units cost each other (the transform's passes share the unit's LDS: 512 x 4096 takes 26 us
    // with eight rows a workgroup on 64 units, 13 with two on 256; 1024 x 3072 10.6 and 8.9); among equal costs prefer more
    // waves in flight per compute unit
    const double crowd = 0.06 * (double)((groups + 255) / 256 * w);
    const double cost = (double)rounds * (1.0 + 0.35 / w) + crowd - 1e-3 * (double)std::min(per_cu * w, 32);
    if (cost < best_cost) best_cost = cost, best = w;
  }
  return best;
}

template <int FMT, int G, int NORM, int TEAM>
int launch_norm_team(const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts, const OperandLayout& L,
                     uint8_t* operand, const NormArgs& na, hipStream_t st) {
  constexpr bool is_int = FMT == kInt4 || FMT == kInt3;
  auto kern = norm_rows_kernel<FMT, G, NORM, TEAM>;
  // the choice depends on the shape only: remembered from the previous launch of this kernel
  static thread_local struct { int64_t rows, K; int n_waves; } memo = {0, 0, 0};
  if (memo.rows != rows || memo.K != K) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kNormLdsLimit);
    if (e != hipSuccess) return check_hip(e, "hipFuncSetAttribute(norm_rows_kernel)");
    // waves that own a row each: one a workgroup spreads few rows best (RMSNorm 256 x 2048 4.9 us, four 5.4), four write
    // more of a line together (3072 x 512 4.4 -> 4.3, LayerNorm 3072 x 2048 8.3 -> 8.0)
    memo.n_waves = TEAM > 1 ? TEAM : NORM == kHadamard ? hadamard_waves_per_group(kern, is_int, rows, K, L.units) : rows > 1024 ? 4 : 1;
    memo.rows = rows;
    memo.K = K;
  }
  const int n_waves = memo.n_waves;
  const int teams = TEAM == 1 ? n_waves : 1;
  const size_t shmem = norm_lds_bytes(NORM, is_int, teams, n_waves, K, L.units);
  const int64_t groups = (rows + teams - 1) / teams;
  hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(64 * n_waves), shmem, st, (const uint16_t*)x, rows, K, ld, ts,
                     L.steps, L.units, operand ? operand + L.codes : nullptr,
                     (uint16_t*)(operand ? operand + L.scales : nullptr),
                     (float*)(operand ? operand + L.mul : nullptr), na);
  return check_hip(hipGetLastError(), "norm_rows_kernel");
}

// Waves that share a row.  Norms: a row's chain of loads, sums, stores and gathers is what few rows take, and more waves walk
// it faster; with many rows it is the work, and each wave more costs its own sums and divisions.  Up to kHold chunks a thread
// (3072 channels a wave) no part of a row is parked in LDS and read back.  Measured with 1, 2, 4 waves, us, RMSNorm + NVFP4:
// 512 x 3072 6.3, 5.0, 4.6; 1024 x 3072 6.7, 5.3, 6.0; 2048 x 3072 7.6, 7.2, 9.0; 8192 x 3072 20.6, 20.2, 27.3; 4608 x 1536
// 7.7, 9.6, 12.4; 1024 x 768 4.0, 3.8, 4.8; 2048 x 6144 13.1, 10.9, 11.4; 2048 x 12288 39.9, 29.3, 21.4; modulated LayerNorm
// 512 x 3072 6.6, 5.5, 5.1; 8192 x 3072 21.9, 22.7, 30.6; 4608 x 1536 8.6, 10.9, 14.0; 1024 x 2048 5.7, 5.0, 5.6.
// Hadamard: up to 4096 channels a wave's own LDS traffic is all that a row waits for; wider rows leave a unit with two or
// three in flight, and few rows wait for their chain: four waves there.  Hadamard + INT4, one wave -> four, us: K = 3072,
// 256 rows 10.8 -> 5.8, 512 rows 10.9 -> 6.5, 768 rows 11.0 -> 7.6, 1024 rows 11.0 (9.5 with fewer rows a workgroup) -> 10.6;
// K = 1024, 768 rows 9.0 -> 7.2.
int waves_per_row(int norm, int64_t rows, int64_t K) {
  if (norm == kHadamard) return K > 4096 || (rows <= 768 && K >= 1024) ? 4 : 1;
  if (K > 6144) return 4;
  if (K >= 4096) return rows <= 768 ? 4 : 2;
  if (K >= 1280) return rows <= 512 ? 4 : rows <= (K >= 2560 ? 2048 : K >= 2048 ? 1024 : 0) ? 2 : 1;
  return K >= 768 && rows <= 1024 ? 2 : 1;
}

template <int FMT, int G, int NORM>
int launch_norm_rows(const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts, const OperandLayout& L,
                     uint8_t* operand, const NormArgs& na, hipStream_t st) {
  // the widths that are taken, more than a row alone needs for the norms: K and the vectors' 2 K or 4 K bytes beside the row
  constexpr bool is_int = FMT == kInt4 || FMT == kInt3;
  const int team = waves_per_row(NORM, rows, K);
  const size_t least = (size_t)K * (NORM == kNormAdaLn ? 6 : 4) + (is_int ? L.units * 4 : 0) + (size_t)(K > 4096 ? 4 : 1) * 16;
  if (least > kNormLdsLimit)
    return fail(PQ_ERR_SHAPE, "K=%lld needs %zu bytes of LDS for one row and the vectors, more than the %zu available",
                (long long)K, least, kNormLdsLimit);
  if (team == 4) return launch_norm_team<FMT, G, NORM, 4>(x, rows, K, ld, ts, L, operand, na, st);
  if constexpr (NORM != kHadamard)
    if (team == 2) return launch_norm_team<FMT, G, NORM, 2>(x, rows, K, ld, ts, L, operand, na, st);
  return launch_norm_team<FMT, G, NORM, 1>(x, rows, K, ld, ts, L, operand, na, st);
}

template <int FMT, int G>
int launch_norm(int norm, const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts,
                const OperandLayout& L, uint8_t* operand, const NormArgs& na, hipStream_t st) {
  if (norm == kNormRms) return launch_norm_rows<FMT, G, kNormRms>(x, rows, K, ld, ts, L, operand, na, st);
  if (norm == kHadamard) return launch_norm_rows<FMT, G, kHadamard>(x, rows, K, ld, ts, L, operand, na, st);
  return launch_norm_rows<FMT, G, kNormAdaLn>(x, rows, K, ld, ts, L, operand, na, st);
}

NormArgs norm_args(const pq_norm_params& p, void* y, int64_t ldy) {
  NormArgs na;
  na.perm = p.perm;
  na.gamma = (const uint16_t*)p.gamma;
  na.mod_scale = (const uint16_t*)p.mod_scale;
  na.mod_shift = (const uint16_t*)p.mod_shift;
  na.rows_per_mod = p.rows_per_mod > 0 ? p.rows_per_mod : INT64_MAX;
  na.eps = p.eps;
  na.y = (uint16_t*)y;
  na.ldy = ldy;
  na.had_pow2 = na.had_m = 0;
  na.had_scale = 0.0f;
  return na;
}

// K = 2^k * m with m in {1, 12, 20} (the smallest such m): false if there is none
bool hadamard_factor(int64_t K, int* pow2, int* m) {
  const int ms[3] = {1, 12, 20};
  for (int i = 0; i < 3; ++i) {
    if (K % ms[i]) continue;
    const int64_t p = K / ms[i];
    if (p >= 1 && (p & (p - 1)) == 0) {
      *pow2 = (int)p;
      *m = ms[i];
      return true;
    }
  }
  return false;
}

NormArgs hadamard_args(const int32_t* perm, int64_t K, void* y, int64_t ldy, int pow2, int m) {
  NormArgs na = {};
  na.perm = perm;
  na.rows_per_mod = INT64_MAX;
  na.y = (uint16_t*)y;
  na.ldy = ldy;
  na.had_pow2 = pow2;
  na.had_m = m;
  na.had_scale = (float)(1.0 / sqrt((double)K));
  return na;
}

}  // namespace

int run_norm_reorder(const pq_norm_params& p, const void* x, int64_t rows, int64_t K, int64_t ld, void* y,
                     int64_t ldy, hipStream_t st) {
  OperandLayout L = {};
  L.steps = (K + 63) / 64;
  const int norm = p.kind == PQ_NORM_RMS ? kNormRms : kNormAdaLn;
  return launch_norm<kFmtNone, 64>(norm, x, rows, K, ld, nullptr, L, nullptr, norm_args(p, y, ldy), st);
}

int run_norm_quantize_packed(const pq_norm_params& p, pq_format fmt, int group, const void* x, int64_t rows,
                             int64_t K, int64_t ld, const float* ts, void* operand, void* y, int64_t ldy,
                             hipStream_t st) {
  const OperandLayout L = operand_layout(fmt, group, rows, K);
  const int norm = p.kind == PQ_NORM_RMS ? kNormRms : kNormAdaLn;
  const NormArgs na = norm_args(p, y, ldy);
  uint8_t* o = (uint8_t*)operand;
  if (fmt == PQ_FMT_NVFP4) return launch_norm<kNvfp4, 16>(norm, x, rows, K, ld, ts, L, o, na, st);
#define PQ_INT_CASE(F, FE)                                                      \
  if (fmt == F) {                                                               \
    switch (group) {                                                            \
      case 32: return launch_norm<FE, 32>(norm, x, rows, K, ld, ts, L, o, na, st);   \
      case 64: return launch_norm<FE, 64>(norm, x, rows, K, ld, ts, L, o, na, st);   \
      case 128: return launch_norm<FE, 128>(norm, x, rows, K, ld, ts, L, o, na, st); \
      case 256: return launch_norm<FE, 256>(norm, x, rows, K, ld, ts, L, o, na, st); \
    }                                                                           \
  }
  PQ_INT_CASE(PQ_FMT_INT4, kInt4)
  PQ_INT_CASE(PQ_FMT_INT3, kInt3)
#undef PQ_INT_CASE
  return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
}

bool hadamard_width_ok(int64_t K) {
  int p, m;
  return hadamard_factor(K, &p, &m);
}

int run_hadamard_reorder(const int32_t* perm, const void* x, int64_t rows, int64_t K, int64_t ld, void* y,
                         int64_t ldy, hipStream_t st) {
  int p, m;
  if (!hadamard_factor(K, &p, &m)) return fail(PQ_ERR_SHAPE, "no Hadamard construction for K=%lld", (long long)K);
  OperandLayout L = {};
  L.steps = (K + 63) / 64;
  return launch_norm<kFmtNone, 64>(kHadamard, x, rows, K, ld, nullptr, L, nullptr, hadamard_args(perm, K, y, ldy, p, m), st);
}

int run_hadamard_quantize_packed(const int32_t* perm, pq_format fmt, int group, const void* x, int64_t rows,
                                 int64_t K, int64_t ld, const float* ts, void* operand, void* y, int64_t ldy,
                                 hipStream_t st) {
  int p, m;
  if (!hadamard_factor(K, &p, &m)) return fail(PQ_ERR_SHAPE, "no Hadamard construction for K=%lld", (long long)K);
  const OperandLayout L = operand_layout(fmt, group, rows, K);
  const NormArgs na = hadamard_args(perm, K, y, ldy, p, m);
  uint8_t* o = (uint8_t*)operand;
  if (fmt == PQ_FMT_NVFP4) return launch_norm<kNvfp4, 16>(kHadamard, x, rows, K, ld, ts, L, o, na, st);
#define PQ_INT_CASE(F, FE)                                                           \
  if (fmt == F) {                                                                    \
    switch (group) {                                                                 \
      case 32: return launch_norm<FE, 32>(kHadamard, x, rows, K, ld, ts, L, o, na, st);   \
      case 64: return launch_norm<FE, 64>(kHadamard, x, rows, K, ld, ts, L, o, na, st);   \
      case 128: return launch_norm<FE, 128>(kHadamard, x, rows, K, ld, ts, L, o, na, st); \
      case 256: return launch_norm<FE, 256>(kHadamard, x, rows, K, ld, ts, L, o, na, st); \
    }                                                                                \
  }
  PQ_INT_CASE(PQ_FMT_INT4, kInt4)
  PQ_INT_CASE(PQ_FMT_INT3, kInt3)
#undef PQ_INT_CASE
  return fail(PQ_ERR_FORMAT, "unsupported (format, group) = (%d, %d)", (int)fmt, group);
}

}  // namespace pq
