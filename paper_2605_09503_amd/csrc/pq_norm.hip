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
#include <math.h>

#include <atomic>

#include "pq_norm_row.h"

namespace pq {

namespace {

enum Norm : int { kNormRms = 0, kNormAdaLn = 1 };
struct NormArgs {
  const int32_t* perm;          // pi, or null for the identity
  const uint16_t* gamma;        // RMSNorm: bf16 [K], or null for ones
  const uint16_t* mod_scale;    // AdaLN: bf16 [n_mod][K] s (the factor is 1 + s), or null for zeros
  const uint16_t* mod_shift;    // AdaLN: bf16 [n_mod][K] b, or null for zeros
  int64_t rows_per_mod;         // token row m uses modulation row m / rows_per_mod
  float eps;
  uint16_t* y;                  // bf16 [rows][ldy] normalised, reordered output, or null
  int64_t ldy;
};

constexpr int kNormMaxWaves = 4;        // of a workgroup: one team of up to four waves, or four rows of a wave each
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

template <int FMT, int G, int NORM, int TEAM>
__global__ __launch_bounds__(64 * kNormMaxWaves) void norm_rows_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t K, int64_t ld, const float* __restrict__ tensor_scale,
    int64_t steps, int64_t units, uint8_t* __restrict__ p_codes, uint16_t* __restrict__ p_scales,
    float* __restrict__ p_mul, NormArgs na) {
  constexpr bool IS_INT = FMT == kInt4 || FMT == kInt3;
  // dynamic LDS: [per team: K bf16 slab] [per team, INT: `units` fp32 group maxima]
  //              [per wave: 4 floats for team reductions]
  // TEAM == 1: every wave owns a row.  TEAM > 1: the workgroup is one team of TEAM waves and owns one row.
  constexpr int TL = 64 * TEAM;                              // threads of a team
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

  unsigned char* slab = lds_raw + (size_t)slot * Ki * 2;
  float* h_all = reinterpret_cast<float*>(lds_raw + (size_t)teams * Ki * 2);
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
  // Without a quantizer a thread asks for one chunk at a time: 67 registers and seven waves a SIMD instead of 83 and five.
  // RMSNorm and reorder, us, three at a time and so: 4608 x 3072 13.6, 12.6, 5126 x 3200 17.9, 14.9, 4096 x 4096 17.6, 13.9,
  // 256 x 2048 3.3, 3.0; 7000 shapes 0.92, three above 1.02.
  constexpr int kBatch = FMT == kFmtNone ? 1 : 3;
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

size_t norm_lds_bytes(bool is_int, int teams, int n_waves, int64_t K, int64_t units) {
  const size_t tail = (is_int ? (size_t)teams * units * 4 : 0) + (size_t)n_waves * 16;
  return (size_t)teams * K * 2 + tail;
}

template <int FMT, int G, int NORM, int TEAM>
int launch_norm_team(const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts, const OperandLayout& L,
                     uint8_t* operand, const NormArgs& na, hipStream_t st) {
  constexpr bool is_int = FMT == kInt4 || FMT == kInt3;
  auto kern = norm_rows_kernel<FMT, G, NORM, TEAM>;
  // waves that own a row each: one a workgroup spreads few rows best (RMSNorm 256 x 2048 4.9 us, four 5.4), four write
  // more of a line together (3072 x 512 4.4 -> 4.3, LayerNorm 3072 x 2048 8.3 -> 8.0)
  const int n_waves = TEAM > 1 ? TEAM : rows > 1024 && K <= 4096 ? 4 : 1;
  const int teams = TEAM == 1 ? n_waves : 1;
  const size_t shmem = norm_lds_bytes(is_int, teams, n_waves, K, L.units);
  static std::atomic<uint64_t> raised{0};
  if (shmem > 48 * 1024) {
    if (int rc = allow_lds(reinterpret_cast<const void*>(kern), kNormLdsLimit, raised, "hipFuncSetAttribute(norm_rows_kernel)"))
      return rc;
  }
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
// The same with and without a quantizer, and not two waves a row wherever the latter is faster so (more than 3072 channels: 0.83
// to 1.0 of the time, with a quantizer 0.81 to 1.18): the statistics' sums take their order from it, and the quantizing call
// equals norm followed by quantizer bit for bit.
int waves_per_row(int64_t rows, int64_t K) {
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
  int team = waves_per_row(rows, K);
  if (rows * 64 * team > UINT32_MAX) team = 1;               // more threads than a grid holds
  const size_t least = (size_t)K * (NORM == kNormAdaLn ? 6 : 4) + (is_int ? L.units * 4 : 0) + (size_t)(K > 4096 ? 4 : 1) * 16;
  if (least > kNormLdsLimit)
    return fail(PQ_ERR_SHAPE, "K=%lld needs %zu bytes of LDS for one row and the vectors, more than the %zu available",
                (long long)K, least, kNormLdsLimit);
  if (team == 4) return launch_norm_team<FMT, G, NORM, 4>(x, rows, K, ld, ts, L, operand, na, st);
  if (team == 2) return launch_norm_team<FMT, G, NORM, 2>(x, rows, K, ld, ts, L, operand, na, st);
  return launch_norm_team<FMT, G, NORM, 1>(x, rows, K, ld, ts, L, operand, na, st);
}

template <int FMT, int G>
int launch_norm(int norm, const void* x, int64_t rows, int64_t K, int64_t ld, const float* ts,
                const OperandLayout& L, uint8_t* operand, const NormArgs& na, hipStream_t st) {
  if (norm == kNormRms) return launch_norm_rows<FMT, G, kNormRms>(x, rows, K, ld, ts, L, operand, na, st);
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

}  // namespace pq
