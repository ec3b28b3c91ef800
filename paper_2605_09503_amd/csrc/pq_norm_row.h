// What the front of a quantized linear layer -- normalisation or Hadamard rotation -- does once a row lies in LDS: the
// reordered row gathered, stored and / or quantized; and the reductions over the waves that share a row.
#pragma once

#include "pq_qgemm_common.h"

namespace pq {

namespace {

constexpr int kFmtNone = -1;                  // normalise and reorder only, no quantization

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
// or fp32 to be scaled and rounded), stored and / or quantized.  kBatch: chunks whose indices and gathers a thread has in
// flight; ix_cur: the indices of the first.
template <int FMT, int G, int TEAM, bool F32, int kBatch>
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
    // the per-row power of two of the operand layout (see int_row_scale): scale units are the fp16 group maxima times 2^-E,
    // the row factor 2^E / Q
    constexpr float Q = qmax_of(FMT);
    team_maxima<TEAM>(row_max, em.red, em.wave, em.lane);      // (with TEAM > 1 also the barrier after the h_lds writes)
    const RowScale scale = int_row_scale(row_max[0]);
    if (em.tl == 0) em.mul[em.row] = scale.up / Q;
    for (int u = em.tl; u < em.n_units; u += TL)               // the team's own LDS writes, ordered above
      em.scales[(int64_t)u * em.rows + em.row] = int_unit(em.h_lds[u], scale.down);
  }
}

constexpr size_t kNormLdsLimit = 160 * 1024 - 1024;      // dynamic LDS a workgroup may ask for

}  // namespace

}  // namespace pq
